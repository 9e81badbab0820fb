"""GPU parity of the encoder step where attention runs without the [seq, seq] matrices (heads of 64 features), against the
CPU oracle: sequences around the tile (64) and workgroup (128) sizes, and one of several workgroups."""
import pytest
import torch

import oracle
import paper_2111_10672_amd as spb
import workloads as wl
from parity import check_gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,seq,heads", [(2, 8, 1), (1, 64, 2), (2, 72, 1), (3, 128, 1), (2, 136, 3), (1, 192, 1), (1, 248, 2), (1, 256, 1), (2, 328, 1), (1, 520, 2)])
def test_attention_lengths(batch, seq, heads):
    cfg = dict(family="encoder", dtype="bf16", batch=batch, seq=seq, layers=1, hidden=64 * heads, heads=heads, ffn=128, vocab=96,
               loss_rows=max(1, batch * seq // 4))
    params, data = wl.make_params(cfg, 0, True), wl.make_batch(cfg, 0)
    for name, t in params.items():
        if "attn.qkv.weight" in name:
            t.mul_(12.0)            # scores far enough apart that a wrong key or statistic shows
    n_units = wl.unit_count(cfg)
    _, exact = oracle.spb_step(cfg, params, data, n_units)
    ref_loss, ref = oracle.spb_step(cfg, params, data, n_units, oracle.round_to_bf16)
    print(f"case batch={batch} seq={seq} heads={heads}", flush=True)
    model = spb.SpbModel(cfg, params)
    model.step({n: t.cuda() for n, t in data.items()}, n_units)
    torch.cuda.synchronize()
    assert abs(model.loss.item() - ref_loss) <= 5e-3 * abs(ref_loss)
    check_gradients({n: g.double().cpu().numpy() for n, g in model.grad_dict(n_units).items()}, ref, "bf16", exact)
    model.close()
