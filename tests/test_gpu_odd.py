"""Rows of any length on the vector paths: odd column counts, and stacks whose
matrices therefore start at any address, for both selections and all storage
types, bitwise against the oracle (selection, norms, momentum, W given O), at
the edges of the vectors, row buffers and the fused update."""
import pytest
import torch

from paper_2512_16928_amd import binding, workloads
from paper_2512_16928_amd.binding import AXIS_COLS, AXIS_ROWS, MASTER_FP32, NS_DIRECT, SELECT_RANDOM
from test_gpu_parity import check_matrix, one_group_workload, run_gpu

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def stack(rows, cols, batch, axis, wdt, gdt, device):
    wl = one_group_workload(rows, cols, count=batch, axis=axis, name=f"odd{rows}x{cols}")
    W, M, G = workloads.make_group(wl, 0, device)
    return W.to(DT[wdt]), M, G.to(DT[gdt])


@pytest.mark.parametrize("wdt,gdt", [("bf16", "bf16"), ("f32", "f32"), ("bf16", "f32"), ("f32", "bf16")])
@pytest.mark.parametrize("axis", [AXIS_ROWS, AXIS_COLS])
@pytest.mark.parametrize("cols", [1, 3, 5, 7, 8, 9, 15, 16, 17, 31, 259, 1021, 1026])
def test_any_column_count(hip_device, cols, axis, wdt, gdt):
    W, M, G = stack(70, cols, 3, axis, wdt, gdt, hip_device)
    alpha = 0.3 if cols > 16 else 1.0   # (small: every line, a compact matrix of a few lines is ill-conditioned)
    # steps: 2 keeps matrices of a few lines within the bound, where five may not
    res = run_gpu(W, M, G, alpha, ns_steps=2, axis=axis)
    for b in (0, 2):
        check_matrix(res, b, alpha, ns_steps=2, axis=axis)
    res = run_gpu(W, M, G, alpha, ns_steps=0, axis=axis)   # no product: the gather's O and the apply pass
    check_matrix(res, 1, alpha, ns_steps=0, axis=axis)


@pytest.mark.parametrize("rows,cols,alpha,axis,wdt,batch,kw", [
    (300, 2047, 0.4, AXIS_ROWS, "f32", 2, {}),                                  # momentum: one partial chunk
    (300, 2051, 0.4, AXIS_ROWS, "bf16", 2, {}),                                 # a full chunk, then 3 columns
    (300, 2051, 0.4, AXIS_ROWS, "f32", 1, dict(master=MASTER_FP32)),            # three passes into fp32 W
    (700, 701, 0.5, AXIS_ROWS, "f32", 2, dict(form=NS_DIRECT)),                 # one pass into fp32 W
    (1024, 2560, 0.25, AXIS_ROWS, "f32", 12, {}),                               # fp32 W on 128 x 128 tiles
    (1024, 2555, 0.25, AXIS_ROWS, "bf16", 12, {}),                              # ragged bf16 W on them
    (1024, 2555, 0.25, AXIS_ROWS, "f32", 9, dict(master=MASTER_FP32)),
    (2048, 2301, 1.0, AXIS_ROWS, "f32", 1, {}),                                 # Direct with X^T rows into fp32 W
    (513, 4093, 0.1, AXIS_COLS, "bf16", 1, {}),                                 # a row buffer's last partial chunk
    (130, 4097, 0.1, AXIS_COLS, "bf16", 2, {}),                                 # wider than the row buffer
    (130, 4104, 0.1, AXIS_COLS, "bf16", 1, {}),                                 # ... in whole chunks
    (257, 2047, 0.2, AXIS_COLS, "f32", 2, {}),
    (130, 2051, 0.2, AXIS_COLS, "f32", 1, {}),
    (515, 771, 0.5, AXIS_COLS, "bf16", 3, dict(rand=(5, 6, 7), norms=False)),   # the single column pass
])
def test_odd_shapes(hip_device, rows, cols, alpha, axis, wdt, batch, kw):
    W, M, G = stack(rows, cols, batch, axis, wdt, wdt, hip_device)
    res = run_gpu(W, M, G, alpha, axis=axis, **kw)
    for b in sorted({0, batch - 1}):
        check_matrix(res, b, alpha, axis=axis, rand=kw.get("rand"))


def test_odd_decay_all_and_pointer_tables(hip_device):
    """The decay-all ablation on odd rows, and matrices whose own start is all
    that is aligned (pointer tables)."""
    for axis in (AXIS_ROWS, AXIS_COLS):
        W, M, G = stack(90, 133, 2, axis, "bf16", "bf16", hip_device)
        res = run_gpu(W, M, G, 0.5, axis=axis, decay_all=True)
        check_matrix(res, 1, 0.5, axis=axis, decay_all=True)
    W, M, G = stack(90, 133, 3, AXIS_ROWS, "bf16", "bf16", hip_device)
    Ws, Ms, Gs = ([t[i].clone() for i in range(3)] for t in (W, M, G))
    binding.dion2_step_batched(Ws, Ms, Gs, 0.5)
    binding.dion2_step_strided(W, M, G, 0.5)
    torch.cuda.synchronize()
    for i in range(3):
        assert torch.equal(Ws[i].view(torch.int16), W[i].view(torch.int16)) and torch.equal(Ms[i], M[i])
