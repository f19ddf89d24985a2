"""Token-split attention body, fp32 result: the largest weight of a row carries no rounding error, also where a later tile
raises the row's maximum by little."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_10325_amd import binding as sv
from paper_2503_10325_amd import workloads as W

from gpu_util import oracle_attn
from test_gpu_attn_bodies import attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("nodes,requests", [(4, 3), (8, 3), (4, 140), (8, 140)])   # 32 and 64 rows; eight and four waves
def test_largest_weight_is_exact(head_dim, nodes, requests):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_10325_amd import runner
    a = attention([nodes] * requests, [300] * requests, head_dim, False)
    # scores in log2 units: token 0 has 0, token 256 (a later tile of the same wave) 5 to 7.9, every other one less than -80
    x = np.linspace(5.0, 7.9, a.q.shape[0] * a.q.shape[1]).reshape(a.q.shape[:2])
    a.q[:], a.k_pool[:] = 0, 0
    a.q[..., 0] = W.f32_to_bf16_bits((x * np.sqrt(head_dim) * np.log(2.0)).astype(np.float32))
    a.k_pool[..., 0] = W.f32_to_bf16_bits(np.array([-16.0], dtype=np.float32))[0]
    for b in range(requests):
        a.k_pool[a.block_table[b, 0], :, 0, 0] = 0
        a.k_pool[a.block_table[b, 16], :, 0, 0] = W.f32_to_bf16_bits(np.array([1.0], dtype=np.float32))[0]
    dev = runner.DeviceAttn(a, out_dtype=torch.float32)
    assert "attn_stream_kernel" in sv.spec_describe_attn_plan(dev.desc)
    dev.run()
    torch.cuda.synchronize()
    ref, _ = oracle_attn(a)
    # the smaller weight, at most 2^-5, is good to 2^-18 (two bf16 terms) and 2^-18 (2^x of a score near 8); product, sums and
    # quotient in fp32 add 4 x 2^-24.  A larger weight of two bf16 terms alone would be off by 2^-19 on average.
    err = np.linalg.norm(dev.out.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err < 2.0 ** -21, err
