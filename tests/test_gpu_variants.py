"""GPU parity at the edges of the kernels' dispatch rules: sizes on both sides of every line at which
another build of a kernel takes over, with remainders in every tile dimension.  Oracle, checks and
tolerances are those of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import test_gpu_parity
from oracle import pisa_oracle as po
from parity_util import COS_MIN, TOL, head_np, row_errors, rows_of_blocks
from test_gpu_parity import DEV, run_full_case
from workloads import WORKLOADS, make_qkv

pytestmark = pytest.mark.gpu


# fp32 attention: calls of 64 to 792 64-row tiles
@pytest.mark.parametrize("L,H,d,B,r,check", [
    (64 * 32, 2, 128, 64, 0.8, [0, 1]),           # 64 tiles
    (64 * 21 + 1, 3, 128, 64, 0.9, [0, 2]),       # 66 tiles, one row in the last
    (64 * 21 + 50, 3, 64, 128, 0.5, [1]),         # the same at head_dim 64, block 128
    (64 * 32, 24, 128, 128, 0.9, [0, 23]),        # 768 tiles
    (64 * 32 + 17, 24, 128, 64, 0.95, [0, 23]),   # 792 tiles
    (64 * 32 + 63, 24, 64, 64, 0.8, [7]),
])
def test_fp32_rows_per_workgroup(lib, L, H, d, B, r, check):
    w = WORKLOADS["tiny"].with_(name=f"fp32-rows-{L}-{H}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=r,
                                seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=check)


# fp32 attention: the lines of the split, in groups of 32 rows per XCD (an eighth of all): eight waves up to 32, 16 rows
# to a workgroup up to 16, and to a workgroup of four waves where a row walks up to 32 pieces of 16 keys; above, the groups past
# a round of 32 CUs (at head_dim 128 also up to half a round of 64 workgroups) are halved
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("L,H,B,check", [
    (32 * 15 - 20, 9, 64, [0, 8]),      # 17: eight blocks, two of them exact: 9 pieces
    (32 * 51 - 7, 4, 64, [0, 3]),       # 26: 26 blocks, six exact: 26
    (32 * 63, 4, 64, [0, 3]),           # 32: 32 blocks, seven exact: 30
    (32 * 60, 4, 128, [0, 3]),          # 30: 15 blocks, three exact: 25
    (32 * 32, 6, 128, [0, 5]),          # 24: 8 blocks, two exact: 17
    (32 * 80, 3, 64, [0, 2]),           # 30: 40 blocks, eight exact: 35, eight waves
    (1024, 4, 64, [0, 3]),              # 16: all in halves
    (32 * 33 - 20, 4, 128, [0, 3]),     # 17: none, the last half of 12 rows
    (1024, 8, 64, [0, 7]),              # 32
    (32 * 33 - 16, 8, 64, [0, 7]),      # 33: one in halves, of which one has no row
    (32 * 49, 8, 128, [7]),             # 49: none
    (32 * 27 - 31, 24, 64, [0, 23]),    # 81: 17 in halves at head_dim 128, none at 64; one row in the last group
    (32 * 21 + 5, 37, 64, [0, 36]),     # 102, six in halves; fewer in the last XCD
])
def test_fp32_split(lib, L, H, B, check, d):
    w = WORKLOADS["tiny"].with_(name=f"fp32-split-{L}-{H}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=0.8,
                                seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=check)


@pytest.mark.parametrize("L,H", [(64 * 21 + 1, 3), (64 * 32 + 17, 24), (450, 10), (512, 14), (513, 14)])
def test_fp32_all_blocks_selected_is_bitwise_dense(lib, L, H):
    w = WORKLOADS["tiny"].with_(heads=H, seq_len=L, head_dim=128, sparsity=0.0)
    q, k, v = (x.to(DEV) for x in make_qkv(w))
    res = lib.forward_in_steps(q, k, v, w.block, 0.0, want_lse=True)
    dense, lse = lib.dense_attention(q, k, v, w.block, want_lse=True)
    assert torch.equal(res["out"], dense) and torch.equal(res["lse"], lse)


# Spectral norm of the block heterogeneity: blocks whose H_j has a low rank or clustered singular values.  (H_j - H_bar, which
# the norm is taken of, has full rank all the same; the tests with a dominant channel have matrices of rank one.)
@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (64, "bf16"), (128, "fp32"), (64, "fp32")])
@pytest.mark.parametrize("B", [64, 128])
def test_spectral_heterogeneity_of_special_blocks(lib, d, dtype, B):
    """Per key block j a centred H_j of known structure, H_bar included by the reference (numpy SVD in fp64): random
    rows, 1 or 2 or 5 distinct tokens (rank 0, 1, 4), pairs of tokens with equal weight in orthogonal channels (repeated
    singular values), a ragged last block of 3 tokens.  1e-9 of the largest norm is what the fp64 products and a Ritz
    value with a 1e-7 residual leave room for (its error is quadratic in the residual)."""
    g = torch.Generator().manual_seed(d + B)
    n, rows = 9, []
    for j in range(n):
        m = 3 if j == n - 1 else B
        k, v = torch.randn(m, d, generator=g), torch.randn(m, d, generator=g)
        if j in (1, 2, 3):                       # few distinct tokens
            pick = torch.arange(m) % (1, 2, 5)[j - 1]
            k, v = k[pick], v[pick]
        if j == 4:                               # +- unit vectors: every singular value of sum k^T v equal
            k = torch.eye(d)[torch.arange(m) // 2 % d] * (1.0 - 2.0 * (torch.arange(m) % 2))[:, None]
            v = k.clone()
        rows.append((k, v))
    k, v = (torch.cat([r[i] for r in rows])[None, None] for i in range(2))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    k, v = k.to(dt).to(DEV), v.to(dt).to(DEV)
    shape = lib.make_shape(k, B)
    st = lib.block_stats(k, k, v, B)
    for norm, ord_ in ((lib.PISA_NORM_SPECTRAL, 2), (lib.PISA_NORM_FROBENIUS, "fro")):
        log_m = lib.block_heterogeneity(shape, k, v, st["kbar64"], norm, 1e-6)[0, 0].cpu().numpy()
        K, V = k[0, 0].double().cpu().numpy(), v[0, 0].double().cpu().numpy()
        H = [(K[j * B:(j + 1) * B] - K[j * B:(j + 1) * B].mean(0)).T @ V[j * B:(j + 1) * B] for j in range(n)]
        bar = sum(H) / n
        M = np.array([np.linalg.norm(h - bar, ord_) for h in H])
        assert np.abs(np.exp(log_m) - 1e-6 - M).max() <= 1e-9 * M.max(), norm


# Up to 320 items of 128 rows nothing is paired: keep-or-drop without a workspace, which has no room for the tables, gives
# the same bits as with one.  Past the line it does not (which shows that the check can tell).
@pytest.mark.parametrize("L,H,d,paired", [
    (128 * 129, 2, 128, False),          # 33 items per XCD: 32 taken whole, one in halves
    (128 * 160, 2, 128, False),          # 40
    (128 * 320 - 50, 1, 128, False),
    (128 * 190, 2, 64, False),           # 48 at head_dim 64: all in halves
    (128 * 196 - 9, 2, 64, True),        # 49
    (128 * 161, 2, 128, True),           # 322 in all
])
def test_short_calls_pair_nothing(lib, L, H, d, paired):
    g = torch.Generator(device=DEV).manual_seed(L)
    q, k, v = (torch.randn(1, H, L, d, generator=g, device=DEV).bfloat16() for _ in range(3))
    n, k_top, shape = lib.num_blocks(L, 64), 20, lib.make_shape(q, 64)
    idx = torch.rand(1, H, n, n, generator=g, device=DEV).topk(k_top).indices.sort().values.int().contiguous()
    tiny = torch.empty(16, dtype=torch.uint8, device=DEV)
    with_ws, without = (lib.attention(shape, q, k, v, None, None, None, idx, k_top, workspace=w)[0] for w in (None, tiny))
    assert torch.equal(with_ws, without) == (not paired)


# Reduction of the partial H sums, one element a thread (few heads) and four, over chunk counts around the sixteen and the
# eight loads in flight; one call (reduction inside the selection's launch) and three calls (a launch of its own)
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("H,n", [(1, 1), (2, 15), (2, 16), (2, 17), (8, 32), (8, 33), (9, 128), (33, 128), (33, 40), (2, 129)])
def test_reduction_of_partial_sums(lib, H, n, d):
    """hsum against fp64: |error| <= 1e-4 of the head's largest element, as for the statistics everywhere; the two ways
    give the same bits."""
    w = WORKLOADS["flux"].with_(name="reduce", heads=H, seq_len=64 * n - 3, head_dim=d, sparsity=0.8, grid=None, seed=n)
    q, k, v = (x.to(DEV) for x in make_qkv(w, device="cpu"))
    res = lib.forward_in_steps(q, k, v, 64, w.sparsity)
    one, _ = lib.forward(lib.make_shape(q, 64), q, k, v, res["k_top"])
    assert torch.equal(one, res["out"])
    ref = _centred_products(k[0, H - 1].cpu(), v[0, H - 1].cpu(), 64).sum(0).numpy()
    got = res["stats"]["hsum"][0, H - 1].cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("d,B", [(128, 64), (128, 128), (64, 64), (64, 128)])
@pytest.mark.parametrize("H,L", [(2, 64 * 9 + 5), (40, 64 * 76 + 13), (40, 64 * 520 + 64)])
def test_fast_heterogeneity_over_many_blocks(lib, H, L, d, B):
    """Workgroups of the fast Frobenius kind with 1 to 44 blocks (the norms are finished eight at a time), against the exact
    kind: both take H_bar from the same fp32 hsum, and the fast one carries fp32 rounding (1e-7 measured)."""
    g = torch.Generator(device=DEV).manual_seed(L + d)
    k, v = (torch.randn(1, H, L, d, generator=g, device=DEV).bfloat16() for _ in range(2))
    shape = lib.make_shape(k, B)
    st = lib.block_stats(k, k, v, B)
    exact, fast = (lib.block_heterogeneity(shape, k, v, st["kbar64"], n, 1e-6, hsum=st["hsum"]).exp()
                   for n in (lib.PISA_NORM_FROBENIUS, lib.PISA_NORM_FROBENIUS_FAST))
    assert float(((fast - exact).abs().amax(-1) / exact.amax(-1)).max()) <= 1e-6


def test_spectral_heterogeneity_of_identical_blocks(lib):
    """All blocks alike: H_j - H_bar is rounding only, log(M + eps) is log(eps) to the last digits."""
    g = torch.Generator().manual_seed(5)
    k, v = (torch.randn(64, 128, generator=g).repeat(4, 1)[None, None].bfloat16().to(DEV) for _ in range(2))
    st = lib.block_stats(k, k, v, 64)
    log_m = lib.block_heterogeneity(lib.make_shape(k, 64), k, v, st["kbar64"], lib.PISA_NORM_SPECTRAL, 1e-6)
    # |H_j| is about 100; its fp64 rounding, times 128 channels, stays below 1e-11
    assert float((log_m.exp() - 1e-6).abs().max()) < 1e-11


def _centred_products(k, v, B):
    """[N, d, d] fp64: sum over the tokens of each block of (k_n - kbar_j)^T v_n (one head)."""
    k, v = k.double(), v.double()
    return torch.stack([(kb - kb.mean(0)).T @ vb for kb, vb in zip(k.split(B), v.split(B))])


# Partial sums over chunks of blocks: chunks of one and of three blocks with a short last one, more blocks in all
# than the rule for few blocks covers, and the eight-wave bf16 kernel (64 rows, ragged, block 128 ending in its first half)
@pytest.mark.parametrize("dtype,H,L,d,B", [
    (torch.float32, 8, 64 * 70 + 20, 128, 64), (torch.float32, 12, 64 * 64, 64, 64),
    (torch.float32, 65, 64 * 63 + 1, 64, 64), (torch.float32, 7, 128 * 31 + 70, 128, 128),
    (torch.bfloat16, 1, 64, 128, 64), (torch.bfloat16, 24, 64 * 22 + 9, 128, 64), (torch.bfloat16, 3, 128 * 11 + 5, 128, 128),
])
def test_sums_over_chunks(lib, dtype, H, L, d, B):
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn(1, H, L, d, generator=g).to(dtype).to(DEV) for _ in range(3))
    st = lib.block_stats(q, k, v, B)
    log_m = lib.block_heterogeneity(lib.make_shape(k, B), k, v, st["kbar64"], lib.PISA_NORM_FROBENIUS, 0.0)
    for h in sorted({0, H // 2, H - 1}):
        ref = _centred_products(k[0, h], v[0, h], B)
        # fp32 products and sums, or the bf16 hi + lo split of the centred keys (2^-17 of each product at most)
        assert float((st["hsum"][0, h] - ref.sum(0)).norm() / ref.sum(0).norm()) < 2.0 ** -17
        for name, x in (("qbar", q), ("kbar", k)):
            means = torch.stack([b.double().mean(0) for b in x[0, h].split(B)])
            assert float((st[name + "64"][0, h] - means).abs().max()) < 1e-12 and torch.equal(st[name][0, h], st[name + "64"][0, h].float())
        norms = (ref - ref.mean(0)).flatten(1).norm(dim=1)
        if ref.shape[0] > 1:
            assert float((log_m[0, h].exp() - norms).abs().max() / norms.max()) < 1e-9


# bf16 attention: calls of few items (most of them in halves of 64 rows altogether); ragged tiles of 1, 9, 33 and 63 rows,
# one and two centroid tiles, no full tile, no selected block
@pytest.mark.parametrize("L,H,d,B,r,check", [
    (40, 2, 128, 64, 0.0, [0, 1]), (65, 1, 64, 64, 0.5, [0]), (1000, 2, 128, 64, 0.8, [0, 1]),
    (64 * 3 + 33, 3, 128, 128, 0.5, [0, 2]), (64 * 5 + 63, 2, 64, 128, 1.0, [0, 1]), (64 * 9 + 9, 2, 128, 64, 1.0, [1]),
    (64 * 70 + 1, 2, 128, 64, 0.9, [0, 1]), (64 * 129, 1, 64, 64, 0.95, [0]),
    (1400, 16, 128, 128, 0.7, [0, 15]), (1409, 16, 128, 128, 0.7, [0, 15]),
    (2048, 20, 128, 64, 0.85, [0, 19]), (2049, 20, 128, 64, 0.85, [0, 19]),
    (2048, 16, 128, 64, 0.1, [0, 15]), (2049, 16, 128, 64, 0.1, [0, 15]),
    (1024, 16, 128, 64, 1.0, [0, 15]), (1025, 16, 128, 64, 1.0, [0, 15]),
    (1024, 16, 64, 128, 0.9, [0, 15]), (1025, 16, 64, 128, 0.9, [0, 15]),
])
def test_bf16_short_calls(lib, L, H, d, B, r, check):
    w = WORKLOADS["flux"].with_(name=f"short-{L}-{H}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=r, grid=None,
                                seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({x for x in (0, 1, n // 2, n - 2, n - 1) if 0 <= x < n}), heads=check)


# bf16 attention: which items of 128 rows are taken in halves, in items per XCD (an eighth of all)
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("L,H,B,r,check", [
    (128 * 16, 8, 128, 0.95, [0, 7]),             # 16, one block of 128 tokens: all
    (128 * 17, 8, 128, 0.95, [0, 7]),             # 17: none
    (128 * 25 - 70, 8, 128, 0.8, [0, 7]),         # 25, one row to an item: none at head_dim 128, all at 64 (the last has one half)
    (128 * 33 - 3, 8, 128, 0.8, [7]),             # 33: one
    (128 * 32, 8, 64, 0.2, [7]),                  # 32, more than three quarters of the blocks: all
    (128 * 49, 8, 64, 0.2, [7]),                  # 49: none
    (128 * 48 - 64, 8, 64, 0.85, [0, 7]),         # 48, two rows to an item: 16, at head_dim 64 all; an odd number of blocks
    (128 * 27 + 9, 14, 64, 0.8, [0, 13]),         # 49: none, at head_dim 64 17
    (128 * 27 + 9, 24, 64, 0.9, [0, 23]),         # 84: 20
])
def test_bf16_halved_items(lib, L, H, B, r, check, d):
    w = WORKLOADS["flux"].with_(name=f"halved-{L}-{H}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=r, grid=None,
                                seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=check)


# bf16 attention at head_dim 64 and block 64: four workgroups on a CU where a call has 97 to 128 of them per XCD (items past the
# last round in halves: two) or 128 items and more, an item walks two lists and there is a selected block
@pytest.mark.parametrize("L,H,r,first_order,approximate", [
    (128 * 16, 40, 0.8, True, True),              # 80 items, 96 workgroups: three
    (128 * 27 - 9, 24, 0.8, True, True),          # 81, 98: four
    (128 * 16 - 64, 48, 0.95, True, True),        # 96, 128: four; an odd number of blocks, two selected
    (128 * 12 + 63, 59, 0.8, True, True),         # 96 (95.9), 128; the last half of 63 rows, no row for the other
    (128 * 97, 8, 0.9, True, True),               # 97, 130: three
    (128 * 15 + 1, 64, 0.5, True, True),          # 128; one row in the last item
    (128 * 15 + 1, 64, 0.25, True, True),         # 128, just over three quarters selected: three
    (128 * 16, 65, 0.25, True, True),             # 130, three quarters: four
    (128 * 16, 64, 1.0, True, True),              # 128, none selected: three
    (1409, 55, 0.7, True, False), (1409, 55, 0.7, False, True),
])
def test_bf16_four_workgroups(lib, L, H, r, first_order, approximate):
    w = WORKLOADS["flux"].with_(name=f"four-{L}-{H}", heads=H, seq_len=L, head_dim=64, block=64, sparsity=r, grid=None,
                                seed=L + H)
    n = -(-L // 64)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=[0, H - 1], first_order=first_order,
                  approximate=approximate)


def test_bf16_halved_items_with_all_xcds_on_a_head(lib):
    """A head too long for an XCD of its own: its 547 items are dealt in groups of 8, the last 35 (from row 65 536 on)
    in halves, with paired query blocks."""
    w = WORKLOADS["flux"].with_(name="halved-long", heads=1, seq_len=70000, head_dim=128, sparsity=0.95, grid=None, seed=3)
    run_full_case(lib, w, blocks_per_head=[0, 1000, 1023, 1024, 1025, 1060, 1092, 1093], heads=[0])


@pytest.mark.parametrize("L,H,B", [(1000, 2, 64), (1400, 16, 64), (1400, 16, 128), (1500, 16, 64), (2048, 20, 64), (63, 1, 128),
                                   (128 * 33, 8, 64), (128 * 24, 8, 64), (128 * 25, 8, 64), (128 * 43 - 3, 8, 128)])
@pytest.mark.parametrize("d", [64, 128])
def test_bf16_all_blocks_selected_is_bitwise_dense(lib, L, H, B, d):
    """Where items are taken whole the number of blocks is even: a 128-row workgroup walks the last of an odd number
    on its own, in half tiles, whose row sums add up in another order."""
    w = WORKLOADS["flux"].with_(heads=H, seq_len=L, head_dim=d, block=B, sparsity=0.0, grid=None)
    q, k, v = (x.to(DEV) for x in make_qkv(w))
    res = lib.forward_in_steps(q, k, v, B, 0.0, want_lse=True)
    dense, lse = lib.dense_attention(q, k, v, B, want_lse=True)
    assert torch.equal(res["out"], dense) and torch.equal(res["lse"], lse)


# the pairing decides which blocks make an item: the same checks at sizes where items are taken whole as well as in halves
# (43 and 41 items per XCD)
@pytest.mark.parametrize("L,approximate", [(64 * 340 - 21, True), (64 * 322, True), (64 * 340 - 21, False)])
def test_query_blocks_paired_in_long_calls(lib, L, approximate):
    test_gpu_parity.test_query_blocks_paired_by_row_similarity(lib, L, approximate)


# the same at head_dim 64, where the build with four workgroups on a CU makes its rows again from the pairs after the walk; items
# per XCD in brackets
@pytest.mark.parametrize("L,H,sparsity", [
    (64 * 256 + 33, 8, 0.85),        # 129: four; an odd number of blocks, the last of 33 rows
    (64 * 264 - 20, 5, 0.85),        # 83, the last 19 in halves, 102 workgroups: four
    (64 * 260 - 40, 6, 0.85),        # 98, the last 34 in halves, 132 workgroups: three
    (64 * 257 + 5, 4, 0.81),         # 65, one in halves: three
    (64 * 2558, 1, 0.98),            # 160, all XCDs on the head: the longest trip list that leaves room for four
    (64 * 2558 + 1, 1, 0.98),        # one block more: three; its last has one row
])
def test_query_blocks_paired_at_64_channels(lib, L, H, sparsity):
    w = WORKLOADS["wan"].with_(name=f"pairing64-{L}", heads=H, seq_len=L, head_dim=64, grid=None, block_offset_std=0.5,
                               sparsity=sparsity, seed=L)
    scale, n = lib.resolved_scale(64), -(-L // 64)
    q, k, v = make_qkv(w, device="cpu")
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    k_top = lib.topk_count(n, sparsity)
    assert 5 * k_top <= n and H * -(-L // 128) > 384
    st = lib.block_stats(qd, kd, vd, 64)
    shape = lib.make_shape(qd, 64)
    idx, _ = lib.select(shape, st["qbar64"], st["kbar64"], k_top, want_gap=False)
    out = torch.full_like(qd, float("nan"))
    lse = torch.full(qd.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    lib.attention(shape, qd, kd, vd, st["kbar"], st["vsum"], st["hsum"], idx, k_top, out=out, lse=lse)
    assert not out.isnan().any() and not lse.isnan().any(), "a query block was left out of the pairing"
    rng = np.random.default_rng(L)
    blocks = sorted({0, 1, n - 2, n - 1} | set(rng.choice(n, 12, replace=False).tolist()))
    rows = rows_of_blocks(blocks, 64, L)
    for h in {0, H - 1}:
        Q, K, V = (head_np(x, 0, h) for x in (q, k, v))
        ref, ref_lse = po.attention_head(Q, K, V, 64, idx[0, h].cpu().numpy(), scale, "hybrid", blocks=blocks,
                                         stats=po.block_stats(Q, K, V, 64))
        rel, cos = row_errors(out[0, h].float().cpu().numpy()[rows], ref)
        assert rel <= TOL[torch.bfloat16] and cos >= COS_MIN, (h, rel, cos)
        assert np.abs(lse[0, h].cpu().numpy()[rows] - ref_lse).max() <= 2e-2


def _heterogeneity_against_svd(lib, k, v, B):
    """Spectral M_j of one head, each within 1e-9 of its own value (numpy SVD in fp64): the fp64 products and a Ritz value
    with a 1e-7 residual (its error is quadratic in the residual) leave room for that."""
    st = lib.block_stats(k, k, v, B)
    log_m = lib.block_heterogeneity(lib.make_shape(k, B), k, v, st["kbar64"], lib.PISA_NORM_SPECTRAL, 0.0)
    H = _centred_products(k[0, 0].cpu(), v[0, 0].cpu(), B).numpy()
    M = np.array([np.linalg.norm(h - H.mean(0), 2) for h in H])
    got = np.exp(log_m[0, 0].cpu().numpy())
    assert np.all(np.abs(got - M) <= 1e-9 * M), np.abs(got / M - 1.0).max()


# one singular value of H_j - H_bar far above the others: the Krylov space ends after one or two steps
@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (64, "bf16"), (128, "fp32"), (64, "fp32")])
@pytest.mark.parametrize("B", [64, 128])
@pytest.mark.parametrize("factor", [float("inf"), 1e4, 3e3])     # the value channel over the others
def test_spectral_heterogeneity_with_a_dominant_channel(lib, d, dtype, B, factor):
    g = torch.Generator().manual_seed(d + B)
    k, v = (torch.randn(1, 1, 24 * B, d, generator=g) for _ in range(2))
    v[..., 5] *= min(factor, 1e4)
    if factor == float("inf"):
        v[..., :5] = 0.0
        v[..., 6:] = 0.0                         # every H_j - H_bar has rank one
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    _heterogeneity_against_svd(lib, k.to(dt).to(DEV), v.to(dt).to(DEV), B)


@pytest.mark.parametrize("B,d", [(64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("c", [1.0, 0.25, 8.0])
def test_spectral_heterogeneity_of_multiples_of_the_identity(lib, B, d, dtype, c):
    """D_0 = c I = -D_1: A = D^T D maps the start vector to a multiple of itself without rounding, so that the first
    off-diagonal of the Lanczos matrix can be exactly zero."""
    k, v = torch.zeros(2, B, d), torch.zeros(2, B, d)
    n = torch.arange(B)
    for j in range(2):                           # tokens +-e_i: sum over the block of k^T v = +-2 on half of the channels
        ch, used = (n // 2 + j * (d // 2)) % d, n < d
        k[j, n[used], ch[used]] = 1.0 - 2.0 * (n[used] % 2)
        v[j] = k[j] * (c if j == 0 else -c)
    _heterogeneity_against_svd(lib, k.view(1, 1, -1, d).to(dtype).to(DEV), v.view(1, 1, -1, d).to(dtype).to(DEV), B)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("entry", [2 ** 30, 2 ** 31 - 1, -2 ** 31, -1, 5])
def test_index_entries_far_out_of_range(lib, dtype, entry):
    """Ignored whatever their size (64 times 2^30 does not fit an int)."""
    g = torch.Generator(device=DEV).manual_seed(3)
    q, k, v = (torch.randn(1, 2, 300, 64, generator=g, device=DEV).to(dtype) for _ in range(3))
    shape = lib.make_shape(q, 64)
    idx = torch.tensor([0, 2, 3], dtype=torch.int32, device=DEV).repeat(1, 2, 5, 1).contiguous()
    want = lib.attention(shape, q, k, v, None, None, None, idx, 3, want_lse=True)
    got = lib.attention(shape, q, k, v, None, None, None, torch.cat([idx, torch.full_like(idx[..., :1], entry)], -1).contiguous(), 4,
                        want_lse=True)
    for a, b in zip(got, want):
        assert float((a.float() - b.float()).abs().max()) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_that_attend_nothing(lib, dtype, d):
    """Keep-or-drop with every index entry out of range: log of an empty sum, and 0 / 0."""
    q, k, v = (torch.randn(1, 2, 300, d, device=DEV).to(dtype) for _ in range(3))
    shape = lib.make_shape(q, 64)
    idx = torch.full((1, 2, 5, 2), 9, dtype=torch.int32, device=DEV)
    idx[:, :, 1] = torch.tensor([0, 3], dtype=torch.int32, device=DEV)
    out, lse = lib.attention(shape, q, k, v, None, None, None, idx, 2, want_lse=True)
    empty = torch.ones(300, dtype=torch.bool, device=DEV)
    empty[64:128] = False
    assert bool((lse[:, :, empty] == -float("inf")).all()) and bool(out[:, :, empty].isnan().all())
    assert bool(lse[:, :, ~empty].isfinite().all()) and bool(out[:, :, ~empty].isfinite().all())


# a mask in a channel of its own: q = 1, k = a huge negative number or -inf, as finite as the type's lowest value
@pytest.mark.parametrize("low", [-float("inf"), -3e38, -1e12])
@pytest.mark.parametrize("masked", [(0, 32), (0, 16), (32, 64), (16, 48), (130, 470), (460, 520)])
@pytest.mark.parametrize("d,scale", [(64, None), (128, None), (128, 1.0), (64, 0.3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_keys_masked_by_a_channel(lib, dtype, d, scale, masked, low):
    """Keys whose logits are lowest or -inf get no weight, wherever they fall among the pieces that a wave takes; the same
    keys by a plain softmax over the others in fp64.  Tolerances: those of the oracle comparisons."""
    g = torch.Generator().manual_seed(d)
    L, H = 520, 2
    q, k, v = (torch.randn(1, H, L, d, generator=g).to(dtype) for _ in range(3))
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:, :, masked[0]:masked[1], 0] = low
    out, lse = lib.dense_attention(q.to(DEV), k.to(DEV), v.to(DEV), 64, scale=scale, want_lse=True)
    idx = torch.arange(9, dtype=torch.int32, device=DEV).repeat(1, H, 9, 1)[..., :8].contiguous()
    part, _ = lib.attention(lib.make_shape(q, 64, scale), q.to(DEV), k.to(DEV), v.to(DEV), None, None, None, idx, 8)
    keep = torch.ones(L, dtype=torch.bool)
    keep[masked[0]:masked[1]] = False
    s = lib.resolved_scale(d, scale)
    for got, n in ((out, L), (part, 512)):
        on = keep[:n].nonzero()[:, 0]
        z = (q.double() @ k[:, :, on].double().transpose(-1, -2)) * s
        ref = z.softmax(-1) @ v[:, :, on].double()
        err = (got.double().cpu() - ref).abs().amax(-1) / ref.abs().amax(-1)
        assert float(err.max()) <= TOL[dtype], n       # (NaN fails)
        if n == L:
            assert float((lse.double().cpu() - z.logsumexp(-1)).abs().max()) <= (1e-4 if dtype == torch.float32 else 2e-2)


# the same masks in calls whose items are taken whole (128 rows a workgroup, mostly; the last ones in halves): one list to an
# item (dense, block 128, nearly every block selected), two lists (tile 0 is in one of them only, so that it is walked in
# split trips of 32 keys), four workgroups on a CU at head_dim 64; items per XCD in brackets
@pytest.mark.parametrize("low", [-float("inf"), -3e38, -1e12])
@pytest.mark.parametrize("masked", [(0, 32), (0, 64), (0, 200)])
@pytest.mark.parametrize("d,H,L,B,k_top", [
    (128, 10, 4096, 64, 32),         # 40
    (128, 10, 4096 - 21, 64, 60),    # 40, just under all blocks
    (64, 10, 4096, 64, 56),          # 40, more than three quarters of the blocks
    (64, 25, 2048 - 9, 64, 16),      # 50: three workgroups on a CU
    (64, 64, 2048, 64, 16),          # 128: four
    (128, 10, 4096, 128, 8), (64, 10, 4096 - 70, 128, 8),
])
def test_keys_masked_by_a_channel_in_long_calls(lib, d, H, L, B, k_top, masked, low):
    g = torch.Generator(device=DEV).manual_seed(L + H)
    q, k, v = (torch.randn(1, H, L, d, generator=g, device=DEV).bfloat16() for _ in range(3))
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:, :, masked[0]:masked[1], 0] = low
    n, s = lib.num_blocks(L, B), lib.resolved_scale(d)
    dense, dense_lse = lib.dense_attention(q, k, v, B, want_lse=True)
    rows = torch.arange(1, k_top + 1, dtype=torch.int32).repeat(n, 1)         # blocks 1 .. k_top or 0, 2 .. k_top
    rows[::2, 0] = 0
    idx = rows.repeat(1, H, 1, 1).contiguous().to(DEV)
    part, part_lse = lib.attention(lib.make_shape(q, B), q, k, v, None, None, None, idx, k_top, want_lse=True)
    token = torch.arange(L, device=DEV)
    keep = ~((token >= masked[0]) & (token < masked[1]))
    chosen = torch.zeros(n, n, dtype=torch.bool, device=DEV).scatter_(1, idx[0, 0].long(), True)
    attends = chosen[token // B][:, token // B]
    for h in (0, H // 2, H - 1):
        z = (q[0, h].double() @ k[0, h].double().T.contiguous()) * s
        for got, lse, on in ((dense, dense_lse, keep[None].expand(L, L)), (part, part_lse, attends & keep)):
            w = z.masked_fill(~on, -float("inf"))
            ref = w.softmax(-1) @ v[0, h].double()
            err = (got[0, h].double() - ref).abs().amax(-1) / ref.abs().amax(-1)
            assert float(err.max()) <= TOL[torch.bfloat16], h       # (NaN fails)
            assert float((lse[0, h].double() - w.logsumexp(-1)).abs().max()) <= 2e-2
    assert bool(dense.isfinite().all()) and bool(part.isfinite().all())


@pytest.mark.parametrize("low", [-float("inf"), -3e38, -1e12])
@pytest.mark.parametrize("d,H,L,B", [(128, 2, 520, 64), (128, 10, 4096 + 30, 64), (64, 64, 2048 + 63, 64), (128, 30, 4096 + 9, 128)])
def test_masked_ragged_tile_before_the_centroids(lib, d, H, L, B, low):
    """The last block is the only exact one and masked throughout: what is left are the centroids of the others."""
    g = torch.Generator(device=DEV).manual_seed(L)
    q, k, v = (torch.randn(1, H, L, d, generator=g, device=DEV).bfloat16() for _ in range(3))
    n, s = lib.num_blocks(L, B), lib.resolved_scale(d)
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:, :, (n - 1) * B:, 0] = low
    st = lib.block_stats(q, k, v, B)
    idx = torch.full((1, H, n, 1), n - 1, dtype=torch.int32, device=DEV)
    out, _ = lib.attention(lib.make_shape(q, B), q, k, v, st["kbar"], st["vsum"], None, idx, 1)
    for h in (0, H // 2, H - 1):
        z = (q[0, h].double() @ st["kbar"][0, h, :-1].double().T.contiguous()) * s
        ref = z.softmax(-1) @ (st["vsum"][0, h, :-1].double() / B)
        err = (out[0, h].double() - ref).abs().amax(-1) / ref.abs().amax(-1)
        assert float(err.max()) <= TOL[torch.bfloat16], h
    assert bool(out.isfinite().all())


@pytest.mark.parametrize("d,L,H", [(64, 70, 1), (128, 1000, 2), (128, 64 * 22 + 9, 10), (64, 64 * 40 + 17, 20)])
def test_fp32_infinite_value_in_the_last_row(lib, d, L, H):
    """The rows a ragged tile lacks must add nothing: with an infinite value in the last row that is there, its channel is
    infinite and the others stay what they were; the same for the last block's value sum among the centroids."""
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn(1, H, L, d, generator=g).to(DEV) for _ in range(3))
    w = v.clone()
    w[:, :, -1, 3] = float("inf")
    others = [c for c in range(d) if c != 3]
    a, b = lib.dense_attention(q, k, v)[0], lib.dense_attention(q, k, w)[0]
    assert bool((b[..., 3] == float("inf")).all()) and torch.equal(a[..., others], b[..., others])
    n, shape = lib.num_blocks(L, 64), lib.make_shape(q, 64)
    idx = torch.zeros(1, H, n, 1, dtype=torch.int32, device=DEV)       # block 0 exactly, the rest by their centroids
    a, b = ((lib.attention(shape, q, k, x, st["kbar"], st["vsum"], None, idx, 1)[0])
            for x in (v, w) for st in (lib.block_stats(q, k, x, 64),))
    assert bool((b[..., 3] == float("inf")).all()) and torch.equal(a[..., others], b[..., others])


# bf16 items taken whole (12 items a head at 1 409 and 1 500 tokens; at head_dim 64 and block 64 from 49 per XCD on): what most
# of the small shapes of test_gpu_parity.py do not reach
@pytest.mark.parametrize("L,H,d,B,r,mode", [
    (1409, 29, 64, 64, 1.0, "hybrid"),           # no selected block
    (1409, 12, 64, 128, 1.0, "hybrid"),
    (1409, 29, 128, 64, 0.8, "pisa0"), (1409, 29, 64, 128, 0.8, "pisa0"),
    (1409, 29, 64, 64, 0.7, "sparse"), (1409, 29, 128, 64, 0.7, "sparse"),      # 23 blocks: the last workgroup holds one
    (1409, 29, 128, 128, 0.7, "sparse"),
    (64 * 17 + 1, 40, 128, 64, 0.5, "hybrid"),
    (1409, 37, 64, 64, 1.0, "hybrid"), (1409, 37, 64, 64, 0.7, "sparse"), (64 * 17 + 1, 46, 64, 64, 0.5, "hybrid"),
])
def test_bf16_long_calls(lib, L, H, d, B, r, mode):
    w = WORKLOADS["flux"].with_(name=f"long-{L}-{H}-{mode}", heads=H, seq_len=L, head_dim=d, block=B, sparsity=r, grid=None,
                                block_offset_std=0.5, seed=L + H)
    n = -(-L // B)
    run_full_case(lib, w, blocks_per_head=sorted({0, 1, n // 2, n - 2, n - 1}), heads=[0, H - 1],
                  first_order=mode == "hybrid", approximate=mode != "sparse")


def _check_heads(lib, q, k, v, B, idx, out, heads, blocks, scale, mode="hybrid", what=""):
    """Rows of the listed blocks and heads against the oracle; idx[h]: the head's index rows."""
    rows = rows_of_blocks(blocks, B, q.shape[2])
    for h in heads:
        Q, K, V = head_np(q, 0, h), head_np(k, 0, h), head_np(v, 0, h)
        st = po.block_stats(Q, K, V, B)
        ref, _ = po.attention_head(Q, K, V, B, None if idx is None else idx[h], scale, mode, blocks=blocks, stats=st)
        rel, cos = row_errors(out[0, h].float().cpu().numpy()[rows], ref)
        assert rel <= TOL[q.dtype] and cos >= COS_MIN, (what, h, rel, cos)


@pytest.mark.parametrize("direction", ["rising", "falling", "spike"])
@pytest.mark.parametrize("d,H", [(64, 18), (128, 18), (64, 22), (64, 37)])
def test_runaway_maximum_in_long_calls(lib, direction, d, H):
    """test_runaway_maximum with items taken whole (18 a head; 64 channels, sparse: at 22 heads, four workgroups on a CU
    at 37), where the maximum is refreshed only when a tile sum nears overflow."""
    L, B = 2304, 64
    w = WORKLOADS["flux"].with_(name=f"runaway-{direction}", heads=H, seq_len=L, head_dim=d, grid=None, sparsity=0.5)
    q, k, v = make_qkv(w, device="cpu")
    u = torch.zeros(d)
    u[:8] = 1.0
    pos = torch.arange(L, dtype=torch.float32) / L
    ramp = {"rising": pos - 0.5, "falling": 0.5 - pos, "spike": torch.zeros(L)}[direction]
    if direction == "spike":
        ramp[L // 2 + 5] = 1.0
    q = (q.float() * 0.25 + 24.0 * u).to(torch.bfloat16)
    k = (k.float() * 0.25 + (35.0 * ramp)[:, None] * u).to(torch.bfloat16)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    scale = lib.resolved_scale(d)
    dense, _ = lib.dense_attention(qd, kd, vd, B)
    res = lib.forward_in_steps(qd, kd, vd, B, w.sparsity)
    blocks = [0, 1, 17, 35]
    _check_heads(lib, q, k, v, B, None, dense, [0, H - 1], blocks, scale, "dense", direction)
    _check_heads(lib, q, k, v, B, res["idx"][0].cpu().numpy(), res["out"], [0, H - 1], blocks, scale, "hybrid", direction)


@pytest.mark.parametrize("d,H", [(64, 28), (128, 28), (64, 37), (64, 55)])
def test_out_of_range_index_entries_in_long_calls(lib, d, H):
    """Entries outside [0, N) at different places of the two rows of a 128-row workgroup: their lists differ in length, so
    that some tiles of either are left without a partner."""
    L, B = 1500, 64
    w = WORKLOADS["flux"].with_(name="badidx", heads=H, seq_len=L, head_dim=d, grid=None, sparsity=0.6)
    q, k, v = make_qkv(w, device="cpu")
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    shape, scale = lib.make_shape(qd, B), lib.resolved_scale(d)
    ws = lib.alloc_workspace(shape, DEV)
    st = lib.block_stats(qd, kd, vd, B, ws)
    n, k_top = lib.num_blocks(L, B), lib.topk_count(lib.num_blocks(L, B), w.sparsity)
    idx, _ = lib.select(shape, st["qbar64"], st["kbar64"], k_top, ws)
    bad = idx.clone()
    for i in range(n):                                        # neighbours lose 0 to 4 entries, at the front or at the back
        lost = (0, 3, 4, 1, 0, 2)[i % 6]
        for t in range(lost):
            bad[:, :, i, t if i % 2 else -1 - t] = (n + 7, -3, 2 ** 31 - 1, -2 ** 31)[t]
    out, _ = lib.attention(shape, qd, kd, vd, st["kbar"], st["vsum"], st["hsum"], bad, k_top, workspace=ws)
    kept = [[r[(r >= 0) & (r < n)] for r in bad[0, h].cpu().numpy()] for h in range(H)]
    _check_heads(lib, q, k, v, B, kept, out, [0, H - 1], list(range(n)), scale)


@pytest.mark.parametrize("d,scale,H", [(128, 0.2, 29), (64, 0.01, 29), (64, 0.01, 37), (64, 0.01, 55)])
def test_custom_softmax_scale_in_long_calls(lib, d, scale, H):
    L, B = 1409, 64
    w = WORKLOADS["flux"].with_(name=f"scale-{scale}", heads=H, seq_len=L, head_dim=d, grid=None, sparsity=0.75)
    q, k, v = make_qkv(w, device="cpu")
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    s32 = lib.resolved_scale(d, scale)
    res = lib.forward_in_steps(qd, kd, vd, B, w.sparsity, scale=scale)
    dense, _ = lib.dense_attention(qd, kd, vd, B, scale=scale)
    blocks = [0, 1, 11, 21, 22]
    _check_heads(lib, q, k, v, B, res["idx"][0].cpu().numpy(), res["out"], [0, H - 1], blocks, s32)
    _check_heads(lib, q, k, v, B, None, dense, [0, H - 1], blocks, s32, "dense")


def test_static_scratch_in_long_calls(lib):
    """pisa_attention_static with the pairing tables in the built-in scratch (340 items, 340 blocks): the bits of the call
    with a workspace."""
    w = WORKLOADS["flux"].with_(heads=2, seq_len=64 * 340 - 21, grid=None, sparsity=0.85)
    q, k, v = (x.to(DEV) for x in make_qkv(w, device="cpu"))
    res = lib.forward_in_steps(q, k, v, w.block, w.sparsity, want_lse=True)
    st, out, lse = res["stats"], torch.full_like(q, float("nan")), torch.full_like(res["lse"], float("nan"))
    lib.attention_static(lib.make_shape(q, w.block), q, k, v, st["kbar"], st["vsum"], st["hsum"], res["idx"], res["k_top"],
                         out=out, lse=lse)
    assert torch.equal(out, res["out"]) and torch.equal(lse, res["lse"])
