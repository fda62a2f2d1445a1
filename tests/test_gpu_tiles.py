"""The Newton-Schulz products' tile and split choices, at the sizes where they change.

A launch of few tiles runs on 64 x 64 tiles, a long K is split over blocks, and
larger launches keep the bigger tiles. Without a split every choice computes
each entry's sum in one order, so a matrix's step is bitwise the same whatever
the batch it is in. With one it is checked against the oracle, within the
bound every Newton-Schulz path has. The workspace starts as NaN bits: tiles
past the compact matrix's real side are not written, and nothing in them may
reach a real entry.
"""
import pytest
import torch

from paper_2512_16928_amd import binding, workloads
from paper_2512_16928_amd.binding import AXIS_AUTO, AXIS_COLS, AXIS_ROWS, CHAIN_F16, MASTER_FP32, NS_DIRECT, NS_GRAM, SELECT_RANDOM
from test_gpu_parity import check_matrix, one_group_workload, run_gpu

pytestmark = pytest.mark.gpu


def nan_workspace(batch, rows, cols, alpha, device, **kw):
    n = binding.dion2_workspace_size_ex(batch, rows, cols, alpha, AXIS_AUTO, 5, **kw)
    return torch.full((n,), 0xFF, dtype=torch.uint8, device=device)


def gram_launches(call):
    """Kernels that the call's Gram products take: two each where K is split."""
    binding.dion2_profile_reset()
    binding.dion2_profile_enable(True)
    call()
    torch.cuda.synchronize()
    prof = binding.dion2_profile_read()
    binding.dion2_profile_enable(False)
    return prof["ns_gram"]["launches"]


def gram_products(batch, rows, cols, alpha, **kw):
    """How many Gram products a call of five steps has: one per step in the DIRECT form."""
    kw.pop("select_rule", None)
    return 5 if binding.dion2_plan_form(batch, rows, cols, alpha, **kw)[0] == NS_DIRECT else 1


@pytest.mark.parametrize("rows,cols,alpha,batches,kw", [
    (260, 1030, 0.25, (1, 2, 90), {}),                           # s = 65: one 64-tile more than s fills
    (1030, 516, 0.5, (1, 17, 18, 38), dict(ns_form=NS_GRAM)),    # s = 258, columns: 15 tiles each, 255 to 570 blocks
    (1000, 1000, 0.25, (1, 25, 26, 56, 57), dict(ns_form=NS_GRAM)),   # s = 250: 250, 260, 560 and 570 blocks
    (1000, 1000, 0.25, (1, 51, 52, 54, 64, 72), dict(ns_form=NS_GRAM)),   # 510 to 720, of which 520, 640 and 720 by XCD
    (640, 1000, 0.5, (1, 12, 17), dict(ns_form=NS_DIRECT)),      # s = 320: one-pass products at 252 and 357 blocks
    (450, 700, 1.0, (1, 8, 13), {}),                             # s = 450, DIRECT, 448 sides written of 512
    (960, 960, 0.25, (1, 26, 57), dict(ns_master=MASTER_FP32)),   # K = 960: the three-pass Gram splits from 1024
    (516, 1030, 0.25, (1, 86), dict(ns_chain=CHAIN_F16)),        # s = 129, l = 8 s: fp16 products
])
def test_tiles_bitwise_across_batches(hip_device, rows, cols, alpha, batches, kw):
    W, M, G = workloads.make_group(one_group_workload(rows, cols, name=f"tile{rows}x{cols}"), 0, hip_device)
    first = None
    for n in batches:
        Wn, Mn, Gn = (t.repeat(n, 1, 1) for t in (W, M, G))
        ws = nan_workspace(n, rows, cols, alpha, hip_device, **kw)
        launches = gram_launches(lambda: binding.dion2_step_ex(Wn, Mn, Gn, alpha, workspace=ws, **kw))
        assert launches == gram_products(n, rows, cols, alpha, **kw), f"batch {n}: K split"
        got = Wn.view(torch.int16)
        if first is None:
            first = got[0].clone()
        assert bool((got == first).all()), f"batch {n}"


@pytest.mark.parametrize("rows,cols,alpha,batch,kw,tol", [
    (260, 2050, 0.25, 1, {}, 2e-2),                              # K = 2080: three parts of unequal length
    (2112, 260, 0.25, 7, {}, 2e-2),                              # columns
    (128, 4100, 0.5, 2, {}, 2e-2),                               # s = 64: the one-launch chain after a split Gram
    (516, 4200, 0.25, 2, dict(ns_master=MASTER_FP32), 2e-3),     # three passes
    (640, 2100, 0.5, 1, dict(ns_form=NS_DIRECT), 2e-2),          # fp16 A from parts, every step
    (520, 2176, 0.25, 1, dict(ns_chain=CHAIN_F16), 2e-2),        # into the fp16 chain
    (2304, 392, 0.25, 1, dict(select_rule=SELECT_RANDOM), 2e-2),  # the unscaled columns left O before the parts came
    (128, 8192, 1.0, 90, {}, 2e-2),                              # 128 x 128 tiles, two parts
])
def test_split_k(hip_device, rows, cols, alpha, batch, kw, tol):
    W, M, G = workloads.make_group(one_group_workload(rows, cols, count=batch, name=f"split{rows}x{cols}"), 0, hip_device)
    run = dict(form=kw.get("ns_form", binding.NS_AUTO), chain=kw.get("ns_chain", binding.CHAIN_HILO),
               master=kw.get("ns_master", binding.MASTER_BF16))
    if "select_rule" in kw:
        run.update(rand=(0, 0, 0), norms=False)
    W2, M2 = W.clone(), M.clone()
    res = run_gpu(W, M, G, alpha, **run)
    for b in (0, batch - 1):
        check_matrix(res, b, alpha, ns_tol=tol, rand=run.get("rand"))
    ws = nan_workspace(batch, rows, cols, alpha, hip_device, **kw)
    launches = gram_launches(lambda: binding.dion2_step_ex(W2, M2, G, alpha, workspace=ws, **kw))
    assert launches == 2 * gram_products(batch, rows, cols, alpha, **kw), "K not split"
    assert torch.equal(W2.cpu().view(torch.int16), res["W"].view(torch.int16)) and torch.equal(M2.cpu(), res["M"])


@pytest.mark.parametrize("rows,cols,batch", [
    (8192, 132, 1),     # one narrow strip: 32-row blocks, shortest allowed
    (1000, 771, 2),     # scalar columns, a last block of 8 rows (waves without rows)
    (290, 2048, 1),     # columns by request on a wide matrix: a second block of 34 rows
    (4096, 1024, 64),   # wide blocks
    (4097, 1024, 65),   # wide blocks, a last block of one row
    (520, 772, 300),    # single streaming waves, a last strip of one vector; a column folded by one thread
    (1030, 1028, 52),   # the same just under their number; by four
    (1030, 1028, 60),   # and just over
])
@pytest.mark.parametrize("gdt", ["bf16", "f32"])
def test_column_norm_blocks(hip_device, rows, cols, batch, gdt):
    """Row blocking and waves of the column norms: exact l1 norms, selection
    and momentum in each, on the smallest compact matrix (the partials share
    its memory)."""
    wl = one_group_workload(rows, cols, axis=AXIS_COLS, name=f"cols{rows}x{cols}")
    W, M, G = workloads.make_group(wl, 0, hip_device)
    G = G.float() if gdt == "f32" else G
    Wn, Mn, Gn = (t.repeat(batch, 1, 1) for t in (W, M, G))
    res = run_gpu(Wn, Mn, Gn, 0.02, axis=AXIS_COLS, ns_steps=1)
    check_matrix(res, batch - 1, 0.02, ns_steps=1, axis=AXIS_COLS)
    assert bool((res["norms"] == res["norms"][0]).all())


def test_direct_rows_on_small_tiles(hip_device):
    """DIRECT's X-side products with X^T as rows: 128 x 128 tiles for one
    matrix, 256 x 256 for a batch, bitwise the same; and against the oracle."""
    W, M, G = workloads.make_group(one_group_workload(2048, 2304, name="rows2048"), 0, hip_device)
    W4, M4, G4 = (t.repeat(4, 1, 1) for t in (W, M, G))
    res = run_gpu(W, M, G, 1.0)
    check_matrix(res, 0, 1.0)
    binding.dion2_step_strided(W4, M4, G4, 1.0)
    torch.cuda.synchronize()
    want = res["W"][0].view(torch.int16)
    assert all(torch.equal(W4[i].cpu().view(torch.int16), want) for i in range(4))


@pytest.mark.parametrize("shapes,kw", [
    ([(520, 4096, 8)], {}),                       # s = 130: three 64-tiles a side of the four padded, 5 parts
    ([(520, 4096, 8), (1000, 1100, 1)], {}),      # beside a wider member (s = 250): zeros past its own side
    ([(540, 8192, 4), (800, 2700, 3)], {}),       # s = 135 and 200, both split, the second over 64-tile rows of its own
    ([(256, 4096, 40)], {}),                      # s = 64: into the one-launch chain, one tile of four
    ([(768, 3072, 12), (1000, 4096, 1)], dict(ns_chain=CHAIN_F16)),    # into the fp16 chain
    ([(640, 1040, 20), (1020, 1040, 1)], dict(ns_master=MASTER_FP32)),  # three passes, split from K = 1024
])
def test_split_k_in_grouped_calls(hip_device, shapes, kw):
    """A Gram product split over K is cut alike in a grouped call, whose shared
    chain may need A_0 further than the group's own side: bitwise the per-group
    calls. Every group here but the one 1100 long is split (two launches a Gram
    product)."""
    wl = workloads.Workload("gsplit", "test", tuple(workloads.Group(f"g{i}", *s) for i, s in enumerate(shapes)), (0.25,))
    stacks = [workloads.make_group(wl, i, hip_device) for i in range(len(shapes))]
    solo = [tuple(t.clone() for t in st) for st in stacks]

    for W, M, G in solo:
        want = 2 if W.shape[-1] != 1100 else 1
        assert gram_launches(lambda: binding.dion2_step_ex(W, M, G, 0.25, **kw)) == want
    binding.dion2_step_groups([(W, M, G, AXIS_AUTO) for W, M, G in stacks], 0.25, **kw)
    torch.cuda.synchronize()
    for i, ((W, M, _), (Ws, Ms, _)) in enumerate(zip(stacks, solo)):
        assert torch.equal(M, Ms), f"group {i}: momentum"
        assert torch.equal(W.view(torch.int16), Ws.view(torch.int16)), f"group {i}: weights"


@pytest.mark.parametrize("rows,cols,batches", [
    (64, 512, (1, 3)),        # short rows, through the caches
    (65, 516, (1, 3)),        # past them, not whole vectors a lane
    (33, 2052, (1, 2)),       # one vector behind a chunk
    (40, 4092, (1, 2)),       # a rest one vector short of a chunk
    (1024, 4092, (1, 70)),    # the launch's rests past 2^27 entries
    (512, 508, (1, 130)),     # short rows past 2^25 entries
])
def test_row_norm_rests(hip_device, rows, cols, batches):
    """The rest of a row past its whole chunks, by either loop of the row norms:
    exact norms, momentum and selection; bitwise the same whatever the batch."""
    W, M, G = workloads.make_group(one_group_workload(rows, cols, axis=AXIS_ROWS, name=f"rest{rows}x{cols}"), 0, hip_device)
    res = run_gpu(W.clone(), M.clone(), G, 0.05, axis=AXIS_ROWS, ns_steps=1)
    check_matrix(res, 0, 0.05, ns_steps=1, axis=AXIS_ROWS)
    for n in batches[1:]:
        Wn, Mn, Gn = (t.repeat(n, 1, 1) for t in (W, M, G))
        norms = torch.empty((n, rows), dtype=torch.float64, device=hip_device)
        binding.dion2_step_ex(Wn, Mn, Gn, 0.05, ns_steps=1, axis=AXIS_ROWS, dbg_norms=norms)
        torch.cuda.synchronize()
        assert bool((norms.cpu() == res["norms"][0]).all()) and bool((Mn == res["M"][0].to(hip_device)).all())


@pytest.mark.parametrize("rows,cols,batch", [
    (4097, 1000, 3),    # blocks down a strip, a last one of one row
    (4097, 997, 3),     # the same with columns past the last vector
    (8192, 1020, 2),    # as many blocks a matrix as that order takes
    (8200, 1020, 2),    # more: along the rows
    (8200, 2047, 1),
    (2048, 1024, 6),    # whole strips: along the rows
])
@pytest.mark.parametrize("rand", [None, (3, 1, 0)], ids=["l1", "random"])
def test_column_update_orders(hip_device, rows, cols, batch, rand):
    """The column update's two block orders: M, K, W given O, the norms of the
    single pass, and every matrix of a batch alike."""
    W, M, G = workloads.make_group(one_group_workload(rows, cols, axis=AXIS_COLS, name=f"upd{rows}x{cols}"), 0, hip_device)
    Wn, Mn, Gn = (t.repeat(batch, 1, 1) for t in (W, M, G))
    res = run_gpu(Wn, Mn, Gn, 0.02, axis=AXIS_COLS, ns_steps=1, rand=rand, norms=rand is None)
    for b in sorted({0, batch - 1}):
        check_matrix(res, b, 0.02, ns_steps=1, axis=AXIS_COLS, rand=rand)
    if rand is None:
        assert bool((res["M"] == res["M"][0]).all()) and bool((res["W"] == res["W"][0]).all())
