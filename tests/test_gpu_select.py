"""The selection kernel at the edges of its line counts, on keys that differ in
every bit position or in none: indices, ranks (through the column gather) and
ties against a plain sort."""
import numpy as np
import pytest
import torch

from paper_2512_16928_amd import binding
from paper_2512_16928_amd.binding import AXIS_COLS, AXIS_ROWS

pytestmark = pytest.mark.gpu


def norms_of(kind, n, rng):
    """Line norms, exactly representable as a sum of two fp32 values."""
    if kind == "equal":
        return np.ones(n), np.zeros(n)
    if kind == "last-bits":   # 1 + i 2^-52: only the lowest bits differ, every pass is needed
        return np.ones(n), rng.permutation(n).astype(np.float64) * 2.0 ** -52
    if kind == "ties":        # few distinct values, zeros among them
        return rng.integers(0, 4, n).astype(np.float64), np.zeros(n)
    # "wide": every exponent; 2^100 apart at most, so that the normalised entries
    # (2^-100 times 2^-13 at least) stay above fp32's smallest normal value,
    # 2^-126, and the relative bound below holds for them
    return np.exp2(rng.integers(-50, 50, n)).astype(np.float64), np.zeros(n)


@pytest.mark.parametrize("n", [1, 2, 63, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4097, 8192, 8193])
@pytest.mark.parametrize("kind", ["equal", "last-bits", "ties", "wide"])
@pytest.mark.parametrize("axis", [AXIS_ROWS, AXIS_COLS])
def test_selection_at_the_edges(hip_device, n, kind, axis):
    rng = np.random.default_rng(n)
    hi, lo = norms_of(kind, n, rng)
    lines = np.zeros((n, 4), dtype=np.float32)
    lines[:, 0], lines[:, 2] = hi, -lo
    M0 = lines if axis == AXIS_ROWS else lines.T.copy()
    want_order = np.lexsort((np.arange(n), -(hi + lo)))   # largest first, ties to the lower index
    for k in sorted({1, (n + 1) // 2, max(1, n - 1), n}):
        alpha = min(1.0, (k - 0.5) / n)
        M = torch.from_numpy(M0.copy()).to(hip_device)
        W = torch.zeros(M.shape, dtype=torch.float32, device=hip_device)
        G = torch.zeros_like(W)
        kk, _ = binding.dion2_plan_info(*M.shape, alpha, axis)
        assert kk == k
        sel = torch.full((1, k), -1, dtype=torch.int32, device=hip_device)
        binding.dion2_step_ex(W, M, G, alpha, 0.5, 1.0, 0, axis, dbg_sel_idx=sel)
        torch.cuda.synchronize()
        K = np.sort(want_order[:k])
        np.testing.assert_array_equal(sel[0].cpu().numpy(), K)
        # the momentum decayed on K alone (columns: placed by rank), and the
        # normalised lines subtracted from W there
        want = M0.copy()
        pick = (K, slice(None)) if axis == AXIS_ROWS else (slice(None), K)
        want[pick] *= np.float32(0.5)
        np.testing.assert_array_equal(M.cpu().numpy(), want)
        X = np.zeros(M0.shape)
        X[pick] = M0[pick]
        nx = np.linalg.norm(X)
        if nx > 0:
            rows, cols = M0.shape
            ref = -np.sqrt(rows / cols) * X / (nx + np.float64(np.float32(1e-7)))
            # two fp32 roundings (the scale, the scaled value) and W's own
            np.testing.assert_allclose(W.cpu().numpy(), ref, rtol=4 * 2.0 ** -23, atol=0)
