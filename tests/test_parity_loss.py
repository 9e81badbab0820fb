"""GPU parity of the loss and its gradient against the CPU oracle at the edges of each way a row is laid over lanes: up to
64 classes in one workgroup or many, then one row per wave or workgroup in ever more registers, then rows longer than
any of those."""
import hashlib

import numpy as np
import pytest
import torch

import oracle
import paper_2111_10672_amd as spb
import workloads as wl
from parity import check_gradients

pytestmark = pytest.mark.gpu

# one workgroup while rows x (classes up to a power of two) <= 2048; rows of 256, 1024, ..., 32768 columns per register file
CASES = [(1, 2), (1024, 2), (1025, 2), (128, 10), (129, 9), (32, 64), (33, 64), (257, 33), (4097, 5),
         (5, 65), (7, 256), (3, 257), (3, 1024), (3, 1025), (2, 2048), (2, 2049), (2, 4096), (2, 4097), (2, 8192), (2, 8193), (2, 16384),
         (2, 16385), (2, 32768), (2, 32769)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,classes", CASES)
def test_rows_and_classes(rows, classes, dtype):
    cfg = dict(family="mlp", dtype=dtype, batch=rows, dims=[16, classes])
    print(f"case rows={rows} classes={classes} {dtype}", flush=True)
    params, batch = wl.make_params(cfg, 0, True), wl.make_batch(cfg, 0)
    exact_loss, exact = oracle.spb_step(cfg, params, batch, 1)
    ref_loss, ref = oracle.spb_step(cfg, params, batch, 1, oracle.round_to_bf16) if dtype == "bf16" else (exact_loss, exact)
    model = spb.SpbModel(cfg, params)
    try:
        for g in model.grads:
            g.fill_(float("nan"))
        model.step({n: t.cuda() for n, t in batch.items()}, 1)
        torch.cuda.synchronize()
        # float32 logits and sums on both types: the sum over up to 32769 exponentials and 4097 rows stays below 1e-4
        assert abs(model.loss.item() - ref_loss) <= (1e-4 if dtype == "f32" else 5e-3) * abs(ref_loss)
        check_gradients({n: g.double().cpu().numpy() for n, g in model.grad_dict(1).items()}, ref, dtype, exact)
    finally:
        model.close()


# SHA-256 (first 16 digits) of the loss and the gradients' bytes.  Up to 2048 classes a lane adds the exponentials of columns
# lane + 64 i, beyond them those of its 16-byte vectors, and the lanes are added as a tree: the size of the register
# file a row is held in must not show, because one rounding of a bfloat16 dZ moves a whole gradient.
BITS = {
    (256, 100, "f32"): "63137afa61375d7e", (256, 100, "bf16"): "1305330bb0643a5e",
    (5, 65, "f32"): "fe2e4e3d71a4c697", (5, 65, "bf16"): "476a1fc712039c43",
    (5, 128, "f32"): "681cdd82d61af650", (5, 128, "bf16"): "dc1a453c6fb23151",
    (7, 129, "f32"): "bd21184ff1ca87ba", (7, 129, "bf16"): "8b94b6be380c656b",
    (64, 1000, "f32"): "331e14683e253b52", (64, 1000, "bf16"): "c5c95418d24571cd",
    (3, 1025, "f32"): "e2d4aab09cdc0681", (3, 1025, "bf16"): "64e8e25b508c8f90",
    (2, 2048, "f32"): "62a443ca319ef535", (2, 2048, "bf16"): "70aaebf242b1c1fb",
    (2, 2049, "f32"): "97c6918ba0b97db0", (2, 2049, "bf16"): "772b0b8b376f6ed1",
    (2, 4999, "f32"): "bd9347d72835a7df", (2, 4999, "bf16"): "e1ff98d2a8f52ca1",
    (2, 32769, "f32"): "2a96d7d46c0f1ef8", (2, 32769, "bf16"): "efa754e15f89ee27",
}


def _digest(rows, classes, dtype):
    cfg = dict(family="mlp", dtype=dtype, batch=rows, dims=[16, classes])
    print(f"case rows={rows} classes={classes} {dtype}", flush=True)
    model = spb.SpbModel(cfg, wl.make_params(cfg, 3, True))
    try:
        model.step({n: t.cuda() for n, t in wl.make_batch(cfg, 3).items()}, 1)
        torch.cuda.synchronize()
        h = hashlib.sha256(model.loss.cpu().numpy().tobytes())
        for _, g in sorted(model.grad_dict(1).items()):
            h.update(g.cpu().numpy().tobytes())
        return h.hexdigest()[:16]
    finally:
        model.close()


@pytest.mark.parametrize("rows,classes,dtype", sorted(BITS))
def test_the_order_of_the_sums_stays(rows, classes, dtype):
    assert _digest(rows, classes, dtype) == BITS[rows, classes, dtype]


@pytest.mark.parametrize("rows,classes", [(6, 9), (300, 33), (6, 65), (6, 2046), (6, 2049), (6, 32769)])
def test_labels_outside_the_classes_add_no_target_term(rows, classes):
    """-1, the first column of the pitch padding and a far one, in every layout of a row; the other rows keep theirs."""
    cfg = dict(family="mlp", dtype="f32", batch=rows, dims=[16, classes])
    print(f"case rows={rows} classes={classes}", flush=True)
    params, batch = wl.make_params(cfg, 0, True), wl.make_batch(cfg, 0)
    labels = batch["labels"].clone()
    labels[:4] = torch.tensor([-1, classes, classes + 1, 2 ** 31 - 1], dtype=torch.int32)
    x = batch["x"].double().numpy()
    w, b = (params[n].double().numpy() for n in sorted(params, key=lambda n: -params[n].dim()))
    z = x @ w.T + b
    m = z.max(1, keepdims=True)
    lse = m[:, 0] + np.log(np.exp(z - m).sum(1))
    y = labels.numpy()
    kept = [r for r in range(rows) if 0 <= y[r] < classes]
    assert len(kept) == rows - 4
    dz = np.exp(z - lse[:, None])
    dz[kept, y[kept]] -= 1.0
    dz /= rows
    want_loss = (lse.sum() - z[kept, y[kept]].sum()) / rows
    model = spb.SpbModel(cfg, params)
    try:
        model.step({"x": batch["x"].cuda(), "labels": labels.cuda()}, 1)
        torch.cuda.synchronize()
        assert abs(model.loss.item() - want_loss) <= 1e-4 * abs(want_loss)
        got = {n: g.double().cpu().numpy() for n, g in model.grad_dict(1).items()}
        check_gradients(got, {n: (dz.T @ x if g.ndim == 2 else dz.sum(0)) for n, g in got.items()}, "f32")
    finally:
        model.close()
