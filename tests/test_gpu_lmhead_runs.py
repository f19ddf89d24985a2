"""Workgroups of the projection's kernel that take several tiles one after the other: their loads run on into the next tile
and the stores of the last are still on their way.  Contractions of two slices (fewer than the loads run ahead, so the
cursors pass a whole tile between two of its barriers), of three and more; vocabularies whose last block is partial, alone in its
run or behind others; a last row block with rows that repeat the last one.

Reference and tolerances as in test_gpu_lmhead_tiles.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,d_model,V", [
    (429, 128, 70000),          # 2 slices, 548 tiles, 2 to 3 per workgroup
    (417, 128, 70001),          # ... the last vocabulary block holds 113 entries
    (429, 384, 98305),          # 6 slices; one entry
    (1040, 256, 33016),         # 4 slices, five full row blocks
    (641, 640, 40008),          # odd row tiles, the last row block nearly empty
    (240, 128, 140000),         # row tiles whose slices fill the LDS: a tile per workgroup
])
def test_lm_head_runs_of_tiles(rows, d_model, V):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    T = 1.1
    li = W.make_lm_head_inputs(rows, d_model, V, seed=rows + V)
    dev = runner.DeviceLmHead(li, temperature=T)
    h, w = dev.hidden.double(), dev.weight.double()
    exact = h @ w.t()
    tol = exact.abs() * 2.0 ** -8 + 1e-5 * (h.abs() @ w.abs().t())
    for _ in range(2):
        dev.logits.fill_(float("nan"))
        dev.run()
        got = dev.logits.double()
        assert bool(torch.isfinite(got).all())
        assert bool(((got - exact).abs() <= tol).all())
        m, z = dev.segment_stats()
        for s in range((V + 8191) // 8192):
            seg = got[:, s * 8192:(s + 1) * 8192].cpu().numpy()
            assert np.array_equal(m[:, s].astype(np.float64), seg.max(axis=1)), f"segment {s} maximum"
            zr = np.exp((seg - seg.max(axis=1, keepdims=True)) / T).sum(axis=1)
            assert np.max(np.abs(z[:, s] - zr) / zr) < 3e-6, f"segment {s} sum"
