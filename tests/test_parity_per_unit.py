"""One unit at a time: the oracle's backward pass of a single unit, fed the GPU's own stored tensors, against the GPU.

A gradient depends only on the layers after it (Sec. 1 of the paper), so the backward pass of unit u is a function
of the unit's input and of the gradient entering it from above.  Both lie in the caller's workspace after a step
(spb_unit_io says where).  Feeding the oracle exactly those bfloat16 values removes what the end-to-end comparison
cannot: two correct bfloat16 implementations drift apart from layer to layer (a pre-activation that rounds to the
other side of zero switches a whole term of a sum), and that drift, not the kernels, is what the end-to-end bound
has to absorb on the deep perceptron.  Here every tensor must meet the stated tolerance flat: 2e-2 (bfloat16
storage) or 1e-4 (float32), as max |g - ref| / max |ref| and as a Frobenius ratio, for
  * every parameter gradient of the unit, and
  * the gradient the unit hands to the unit below (compared with what the GPU stored for that unit; for the CNN
    units the max measure may be missed at isolated entries, see _check).
Full-size configurations run selected units, which reaches every product at its real shape, element by element.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2111_10672_amd as spb
import workloads as wl
from oracle import spb as oracle_step
from parity import TOL, rel_fro, rel_max

pytestmark = pytest.mark.gpu


def _shapes(cfg, unit, n_units):
    """(input shape, output shape) of a unit as the oracle lays tensors out; None = 2-D as stored."""
    fam = cfg["family"]
    if not fam.startswith("resnet"):
        return None, None
    lay = wl.resnet_layout(cfg)
    n = cfg["batch"]
    if unit == 0:
        st = lay["stem"]
        out_hw = lay["blocks"][0]["in_hw"]
        return (n, cfg["image"][0], cfg["image"][1], st["cin"]), (n, out_hw[0], out_hw[1], st["cout"])
    if unit == n_units - 1:
        return (n, lay["final_hw"][0], lay["final_hw"][1], lay["features"]), None
    b = lay["blocks"][unit - 1]
    return (n, b["in_hw"][0], b["in_hw"][1], b["cin"]), (n, b["out_hw"][0], b["out_hw"][1], b["cout"])


MASK_FLIP_FRACTION = 1e-4


def _check(name, got, ref, tol, report, allow_mask_flips=False):
    """Both measures within tol.  allow_mask_flips (activation gradients of the CNN units only): up to
    MASK_FLIP_FRACTION of the entries may miss the max-measure bound.  Inside a residual block the oracle recomputes
    the inner activations in float64 and the GPU in float32; where a pre-activation lies within that rounding of
    zero the two ReLU masks differ, which switches single terms of the gradient at isolated pixels (seen: 4 to 281
    entries of 1 to 6 million).  The Frobenius measure stays flat, and a wrong tile edge or index would miss the
    bound on whole rows or columns, thousands of times that many entries."""
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (name, got.shape, ref.shape)
    assert np.isfinite(got).all(), name
    em, ef = rel_max(got, ref), rel_fro(got, ref)
    beyond = int((np.abs(got - ref) > tol * np.abs(ref).max()).sum())
    report.append((name, em, ef, beyond))
    assert ef <= tol, f"{name}: rel_fro {ef:.3e} > {tol:.1e}"
    if allow_mask_flips and beyond:
        print(f"  {name}: {beyond} of {got.size} entries beyond {tol:.0e} of the largest magnitude (mask flips), rel_fro {ef:.2e}", flush=True)
        assert beyond <= MASK_FLIP_FRACTION * got.size, f"{name}: {beyond} of {got.size} entries beyond the bound"
    else:
        assert em <= tol, f"{name}: rel_max {em:.3e} > {tol:.1e}"


def _teacher_forced(name, units_to_run=None, seed=0, perturbed=True, check_handed_down=True):
    cfg = wl.get_config(name)
    params, batch = wl.make_params(cfg, seed, perturbed), wl.make_batch(cfg, seed)
    model = spb.SpbModel(cfg, params)
    dev = {n: t.cuda() for n, t in batch.items()}
    L = model.n_units
    tol = TOL[cfg["dtype"]]
    q = oracle.round_to_bf16 if cfg["dtype"] == "bf16" else oracle.identity
    p64 = {n: oracle_step._as_f64(v) for n, v in params.items()}
    b64 = {n: oracle_step._as_f64(v) for n, v in batch.items()}
    o_units = oracle_step.build_units(cfg)
    units_to_run = list(range(L - 1, -1, -1)) if units_to_run is None else units_to_run
    report = []
    try:
        model.forward(dev, L)
        for u in units_to_run:
            print(f"case {name} unit {u} of {L}", flush=True)
            for g in model.grads:
                g.fill_(float("nan"))
            model.backward(L - u)
            torch.cuda.synchronize()
            v_in, v_g = spb.spb_unit_io(model.handle, L, u)
            in_shape, out_shape = _shapes(cfg, u, L)
            x_u = model.read_view(v_in, batch).numpy()
            if in_shape is not None:
                x_u = x_u.reshape(in_shape)
            g_u = model.read_view(v_g)
            if g_u is not None:
                g_u = g_u.numpy()
                if out_shape is not None:
                    g_u = g_u.reshape(out_shape)
            else:
                assert u == L - 1
            gpu_grads = {info["name"]: g.double().cpu().numpy() for info, g in zip(model.infos, model.grads) if info["unit"] == u}
            # the oracle's unit, from the GPU's input and the GPU's incoming gradient
            o_units[u].forward(x_u, p64, q, b64)
            want_dx = check_handed_down and u > 0
            ref_grads, dx = o_units[u].backward(g_u, p64, q, need_input_grad=want_dx)
            assert set(ref_grads) == set(gpu_grads), (sorted(ref_grads), sorted(gpu_grads))
            for pname, ref in ref_grads.items():
                _check(f"{name} unit {u} {pname}", gpu_grads[pname], ref, tol, report)
            if want_dx:
                model.backward(L - u + 1)              # one unit deeper: unit u now forms the gradient it hands down
                torch.cuda.synchronize()
                _, v_below = spb.spb_unit_io(model.handle, L, u - 1)
                handed = model.read_view(v_below).numpy()
                if v_below["relu_applied"]:            # perceptron: the mask of the unit below (its output = this input) is fused in
                    dx = q(np.asarray(dx) * (x_u > 0))
                _check(f"{name} unit {u} gradient handed to unit {u - 1}", handed, np.asarray(dx).reshape(handed.shape), tol, report,
                       allow_mask_flips=cfg["family"].startswith("resnet"))
    finally:
        model.close()
    flat = [r for r in report if r[3] == 0]
    worst = max(flat, key=lambda r: max(r[1], r[2]))
    print(f"  {name}: {len(report)} tensors, {len(flat)} within {tol:.0e} on both measures (worst {worst[0]}: rel_max {worst[1]:.2e} "
          f"rel_fro {worst[2]:.2e}), {len(report) - len(flat)} activation gradients with isolated mask flips", flush=True)
    return report


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "ragged_mlp_bf16", "ragged_mlp_f32", "many_class_mlp_bf16", "tall_mlp_bf16",
                                  "part_wave_mlp_bf16"])
def test_every_unit_of_the_perceptrons(name):
    _teacher_forced(name, perturbed=(name != "cfg2"))
    if name == "cfg2":
        _teacher_forced(name, seed=1, perturbed=True)


@pytest.mark.parametrize("name", ["small_resnet_basic_bf16", "small_resnet_bottleneck_bf16", "small_resnet101_bf16", "mid_resnet_bottleneck_bf16"])
def test_every_unit_of_the_small_cnns(name):
    _teacher_forced(name)


@pytest.mark.parametrize("name", ["small_encoder_bf16", "fused_attention_encoder_bf16", "wide_encoder_512_bf16", "big_vocab_encoder_bf16"])
def test_every_unit_of_the_small_encoders(name):
    _teacher_forced(name)


@pytest.mark.parametrize("name", ["odd_resnet_basic_bf16", "pixel_resnet_basic_bf16"])
def test_every_unit_of_the_cnns_on_odd_images(name):
    _teacher_forced(name)


@pytest.mark.parametrize("name,units", [("odd_tiles_128x64_resnet_basic_bf16", [2, 1]), ("odd_tiles_stride2_resnet_basic_bf16", [2, 1]),
                                        ("odd_tiles_256x64_resnet_basic_bf16", [1]), ("odd_tiles_128x128_resnet_basic_bf16", [1]),
                                        ("odd_tiles_64x128_resnet_basic_bf16", [1])])
def test_part_filled_large_tiles_of_convolutions(name, units):
    _teacher_forced(name, units_to_run=units)


# 3x3 weight gradients of more pixels than a workgroup's table holds at a time
@pytest.mark.parametrize("name", ["long_slice_resnet_basic_bf16"])
def test_weight_gradients_over_several_tables(name):
    _teacher_forced(name, units_to_run=[1], check_handed_down=False)


@pytest.mark.parametrize("name", ["rows_attention_136_bf16", "rows_attention_256_bf16", "rows_attention_328_bf16", "rows_attention_512_bf16",
                                  "rows_attention_chain_bf16", "rows_attention_chain2_bf16", "long_attention_520_bf16"])
def test_encoder_layers_of_more_than_128_positions(name):
    _teacher_forced(name, units_to_run=[1])


# The logits of a wave that holds 26 of its 32 columns: their weights are scaled up until they take most of the
# softmax, so that a few rows of that wave stored in each other's place show in the gradients of those columns.
@pytest.mark.parametrize("name", ["part_wave_encoder_bf16"])
def test_vocabulary_columns_of_a_part_filled_wave(name):
    cfg = wl.get_config(name)
    whole = cfg["vocab"] // 32 * 32
    params, batch = wl.make_params(cfg, 0, True), wl.make_batch(cfg, 0)
    batch["labels"] = batch["labels"] % whole
    params["head.vocab.weight"][whole:] *= 64.0
    model = spb.SpbModel(cfg, params)
    u = model.n_units - 1
    try:
        model.step({n: t.cuda() for n, t in batch.items()}, 1)
        torch.cuda.synchronize()
        x_u = model.read_view(spb.spb_unit_io(model.handle, 1, u)[0], batch).numpy()
        got = {n: g.double().cpu().numpy() for n, g in model.grad_dict(1).items()}
    finally:
        model.close()
    p64 = {n: oracle_step._as_f64(v) for n, v in params.items()}
    unit = oracle_step.build_units(cfg)[u]
    unit.forward(x_u, p64, oracle.round_to_bf16, {n: oracle_step._as_f64(v) for n, v in batch.items()})
    ref, _ = unit.backward(None, p64, oracle.round_to_bf16, need_input_grad=False)
    for n in ("head.vocab.weight", "head.vocab.bias"):
        _check(f"{name} {n}, columns from {whole}", got[n][whole:], ref[n][whole:], TOL["bf16"], [])


# Full size: the classifier, the top units, and one unit of every kind of shape further down (a stride-2 block with a
# projection, the first block behind the stem, the stem itself / the embedding).
@pytest.mark.parametrize("name,units", [("cfg3", [9, 8, 7, 5, 3, 1, 0]), ("cfg4", [17, 16, 14, 10]), ("cfg5", [13, 12, 11, 1, 0])])
def test_selected_units_at_full_size(name, units):
    _teacher_forced(name, units_to_run=units, perturbed=False)
