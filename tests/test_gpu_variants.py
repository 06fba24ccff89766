"""GPU parity at the edges of the kernels' dispatch rules: sizes on both sides of every line at which
another build of a kernel takes over, with remainders in every tile dimension.  Oracle, checks and
tolerances are those of test_gpu_parity.py."""
import pytest
import torch

from test_gpu_parity import DEV, run_full_case
from workloads import WORKLOADS, make_qkv

pytestmark = pytest.mark.gpu


# fp32 attention: 16, 32 and 64 query rows per workgroup (up to 64, up to 768, more 64-row tiles in all)
@pytest.mark.parametrize("L,H,d,B,r,check", [
    (64 * 32, 2, 128, 64, 0.8, [0, 1]),           # 64 tiles: the last size with 16 rows
    (64 * 21 + 1, 3, 128, 64, 0.9, [0, 2]),       # 66 tiles, one row in the last: 32 rows
    (64 * 21 + 50, 3, 64, 128, 0.5, [1]),         # the same at head_dim 64, block 128
    (64 * 32, 24, 128, 128, 0.9, [0, 23]),        # 768 tiles: the last size with 32 rows
    (64 * 32 + 17, 24, 128, 64, 0.95, [0, 23]),   # 792 tiles: 64 rows
    (64 * 32 + 63, 24, 64, 64, 0.8, [7]),
])
def test_fp32_rows_per_workgroup(lib, L, H, d, B, r, check):
    w = WORKLOADS["tiny"].with_(name=f"fp32-rows-{L}-{H}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=r,
                                seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=check)


@pytest.mark.parametrize("L,H", [(64 * 21 + 1, 3), (64 * 32 + 17, 24)])
def test_fp32_all_blocks_selected_is_bitwise_dense(lib, L, H):
    w = WORKLOADS["tiny"].with_(heads=H, seq_len=L, head_dim=128, sparsity=0.0)
    q, k, v = (x.to(DEV) for x in make_qkv(w))
    res = lib.forward_in_steps(q, k, v, w.block, 0.0, want_lse=True)
    dense, lse = lib.dense_attention(q, k, v, w.block, want_lse=True)
    assert torch.equal(res["out"], dense) and torch.equal(res["lse"], lse)
