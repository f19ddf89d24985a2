"""Every workgroup tile of the projection's kernel (lm_head_tile_kernel<vocabulary entries / 64, row tiles of 16>: 128
entries with 2 to 8 row tiles, 256 with 4 to 16; even and odd), with row counts just past a tile or block, vocabularies
that end inside a block (odd: scalar stores), two slices of the contraction (fewer than the loads run ahead) and more.

Reference: the product in fp64 (plain torch).  Tolerance as in test_gpu_lmhead.py: half a bf16 step of the exact value
plus 1e-5 sum_k |h_k w_k| for fp32 accumulation; statistics against fp64 sums over the kernel's own logits (exact
maximum; sums to 3e-6, the fp32 exponentials and partial sums)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,d_model,V,tile", [
    # 128 vocabulary entries per workgroup
    (145, 2048, 300, (2, 2)),           # 2 row tiles, several row blocks, 32 slices
    (16, 128, 130, (2, 2)),             # 2, one full row tile, a second vocabulary block of two entries
    (33, 384, 16411, (2, 3)),           # 3 (odd vocabulary)
    (64, 128, 16640, (2, 4)),           # 4
    (65, 640, 16648, (2, 5)),           # 5
    (81, 128, 16464, (2, 6)),           # 6
    (127, 1024, 16425, (2, 8)),         # 8
    # 256
    (129, 128, 13150, (4, 4)),          # 4
    (129, 384, 21888, (4, 6)),          # 6
    (193, 128, 21888, (4, 8)),          # 8
    (129, 128, 32939, (4, 10)),         # 10, odd vocabulary
    (161, 256, 32939, (4, 11)),         # 11: the two wave rows hold 6 and 5 row tiles
    (353, 128, 21888, (4, 12)),         # 12, three row blocks
    (193, 384, 32939, (4, 13)),         # 13
    (209, 128, 32939, (4, 14)),         # 14
    (225, 256, 32939, (4, 15)),         # 15
    (481, 128, 21888, (4, 16)),         # 16, two row blocks
])
def test_lm_head_tiles(rows, d_model, V, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import binding, runner
    plan = binding.spec_describe_lm_head_plan(rows, d_model, V)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:       # the rule counts compute units
        assert f"lm_head_tile_kernel<{tile[0]}, {tile[1]}>" in plan, plan
    T = 0.9
    li = W.make_lm_head_inputs(rows, d_model, V, seed=rows + V)
    dev = runner.DeviceLmHead(li, temperature=T)
    dev.logits.fill_(float("nan"))
    dev.run()
    got = dev.logits.double()
    h, w = dev.hidden.double(), dev.weight.double()
    exact = h @ w.t()
    tol = exact.abs() * 2.0 ** -8 + 1e-5 * (h.abs() @ w.abs().t())
    assert bool(torch.isfinite(got).all())
    assert bool(((got - exact).abs() <= tol).all())
    m, z = dev.segment_stats()
    for s in range((V + 8191) // 8192):
        seg = got[:, s * 8192:(s + 1) * 8192].cpu().numpy()
        assert np.array_equal(m[:, s].astype(np.float64), seg.max(axis=1)), f"segment {s} maximum"
        zr = np.exp((seg - seg.max(axis=1, keepdims=True)) / T).sum(axis=1)
        assert np.max(np.abs(z[:, s] - zr) / zr) < 3e-6, f"segment {s} sum"
