"""GPU parity of the loss and its gradient against the CPU oracle at the edges of each way a row is laid over lanes: up to
64 classes in one workgroup or many, then one row per wave or workgroup in ever more registers, then rows longer than
any of those."""
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
