"""GPU parity: the HIP path (through the C ABI) against the fp64 CPU oracle, element by element,
on the same seeded inputs.  Sizes span several tiles and ragged tails."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from _util import assert_close, attn_layout, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2604_12219_amd as P
    assert torch.cuda.is_available(), "these tests need the MI355X"
    P.load_library()
    return P


def _inputs(grid, heads, d, seed=0, batch=1):
    return workloads.make_qkv(grid, heads, d, seed=seed, device="cuda", batch=batch)


# ------------------------------------------------------------------------------------------------
# dense reference kernel (Eq.1)
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("grid,heads,d", [((4, 16, 16), 2, 64), ((3, 11, 13), 2, 128), ((1, 5, 7), 1, 128),
                                          ((2, 16, 16), 3, 128)])
def test_dense_matches_oracle(P, grid, heads, d):
    q, k, v = _inputs(grid, heads, d)
    shape = P.Shape.of(q)
    out, lse = P.attn_dense_ref(q, k, v, shape, want_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v), return_lse=True)
    assert_close(to_f64(out), ref, what=f"dense {grid} d={d}")
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=2e-2)


@pytest.mark.parametrize("n,heads,d", [(449, 1, 64), (575, 2, 64), (1345, 2, 64), (705, 1, 128), (768, 3, 128), (833, 2, 128), (959, 1, 128)])
def test_dense_of_small_grids_in_two_teams_matches_oracle(P, n, heads, d):
    """at most one query tile per compute unit: the keys are halved between two teams of waves.  Odd and even numbers of key tiles
    from the smallest on, a last tile of 1, 63 and 64 keys in the second half"""
    q, k, v = _inputs((1, 1, n), heads, d, seed=n)
    out, lse = P.attn_dense_ref(q, k, v, P.Shape.of(q), want_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v), return_lse=True)
    assert_close(to_f64(out), ref, what=f"dense n={n} d={d}")
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=2e-2)


@pytest.mark.parametrize("n,d", [(449, 64), (1000, 64), (705, 128), (1024, 128)])
def test_dense_in_two_teams_against_one_walk_per_query_tile(P, n, d):
    """the same heads in a grid of 32 workgroups per XCD (two teams of waves) and of 33 (one): equal up to the rounding of P and of
    the output to bf16, tolerances as for key-range slicing below"""
    q, k, v = (torch.cat([t] * 17, dim=1)[:, :33].contiguous() for t in _inputs((1, 1, n), 2, d, seed=n))
    assert P.attn_variant(P.Shape.of(q[:, :32])) == ("short_teams" if n < 961 and d == 64 else "teams")
    assert P.attn_variant(P.Shape.of(q)) in ("short", "whole", "wide")
    two, two_lse = P.attn_dense_ref(q[:, :32], k[:, :32], v[:, :32], P.Shape.of(q[:, :32]), want_lse=True)
    one, one_lse = P.attn_dense_ref(q, k, v, P.Shape.of(q), want_lse=True)
    torch.cuda.synchronize()
    assert not torch.equal(two, one[:, :32])  # (so both paths did run)
    a, b = two.float(), one[:, :32].float()
    assert (a - b).abs().max().item() <= 2e-2 * b.abs().max().item()
    assert (a - b).abs().mean().item() <= 1e-3 * b.abs().mean().item()
    np.testing.assert_allclose(two_lse.cpu().numpy(), one_lse[:32].cpu().numpy(), atol=1e-3)


@pytest.mark.parametrize("n,d", [(1025, 128), (1089, 64), (1280, 128), (1281, 64), (1537, 128), (2047, 128), (2048, 64)])
def test_dense_in_wide_workgroups(P, n, d):
    """32 heads take workgroups of 256 query rows, 33 those of 128 (one wide workgroup more than an XCD has compute units): a row meets its
    keys in the same order in both.  Last wide tiles of 1, 65, 128, 255 and 256 rows, last key tiles of 1, 63 and 64 keys, odd and even numbers of them"""
    q2, k2, v2 = _inputs((1, 1, n), 2, d, seed=n)
    q, k, v = (torch.cat([t] * 17, dim=1)[:, :33].contiguous() for t in (q2, k2, v2))
    assert P.attn_variant(P.Shape.of(q[:, :32])) == "wide" and P.attn_variant(P.Shape.of(q)) == "whole"
    wide, wide_lse = P.attn_dense_ref(q[:, :32], k[:, :32], v[:, :32], P.Shape.of(q[:, :32]), want_lse=True)
    narrow, narrow_lse = P.attn_dense_ref(q, k, v, P.Shape.of(q), want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(wide, narrow[:, :32]) and torch.equal(wide_lse, narrow_lse[:32])
    ref, ref_lse = oracle.dense_attention(to_f64(q2), to_f64(k2), to_f64(v2), return_lse=True)
    assert_close(to_f64(wide[:, 30:]), ref, what=f"wide dense n={n} d={d}")
    np.testing.assert_allclose(wide_lse[30:32].cpu().numpy(), ref_lse, atol=2e-2)


def test_dense_respects_strides_and_scale(P):
    q, k, v = _inputs((2, 9, 10), 2, 128)
    B, H, n, d = q.shape
    big = torch.zeros((3, B, n, H, d + 8), dtype=torch.bfloat16, device="cuda")  # [which, B, n, H, d+pad]
    for i, t in enumerate((q, k, v)):
        big[i, :, :, :, :d] = t.permute(0, 2, 1, 3)
    qs, ks, vs = (big[i, :, :, :, :d].permute(0, 2, 1, 3) for i in range(3))  # [B,H,n,d] views, n-stride H*(d+8)
    shape = P.Shape.of(qs, scale=0.11)
    out = torch.zeros_like(big[0])[:, :, :, :d].permute(0, 2, 1, 3)
    P.attn_dense_ref(qs, ks, vs, shape, out=out)
    torch.cuda.synchronize()
    ref = oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v), scale=0.11)
    assert_close(to_f64(out), ref, what="strided dense")


# ------------------------------------------------------------------------------------------------
# stage 1: scores
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("grid,d,block", [((4, 16, 16), 64, 64), ((3, 21, 13), 128, 64), ((3, 21, 13), 128, 128)])
def test_block_scores_match_oracle(P, grid, d, block):
    q, k, _ = _inputs(grid, 2, d)
    shape = P.Shape.of(q, block=block)
    nb = P.num_blocks(shape)
    bias = torch.randn((2, nb), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    s0 = P.block_score(q, k, shape)
    s1 = P.block_score(q, k, shape, key_bias=bias)
    torch.cuda.synchronize()
    ref = oracle.block_scores(to_f64(q), to_f64(k), block)
    tol = 1e-3 * np.abs(ref).max()
    np.testing.assert_allclose(s0.cpu().numpy(), ref, atol=tol, rtol=0)
    np.testing.assert_allclose(s1.cpu().numpy(), ref + bias.cpu().numpy()[:, None, :], atol=tol, rtol=0)


@pytest.mark.parametrize("grid,d,block,group", [((4, 16, 16), 64, 64, 32), ((3, 21, 13), 128, 64, 32), ((3, 21, 13), 128, 128, 8),
                                                ((9, 20, 23), 128, 64, 64), ((9, 20, 23), 64, 64, 1000), ((1, 5, 7), 128, 64, 32)])
def test_block_scores_from_the_statistics_workspace(P, grid, d, block, group):
    """pasa_block_score_with_stats: the block-mean keys come from pasa_kv_stats' workspace, K is not read again"""
    q, k, v = _inputs(grid, 2, d, seed=3)
    shape = P.Shape.of(q, block=block, group=group)
    nb = P.num_blocks(shape)
    bias = torch.randn((2, nb), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    ws = P.kv_stats(k, v, shape)
    s0 = P.block_score(q, None, shape, stats_ws=ws)
    s1 = P.block_score(q, None, shape, key_bias=bias, stats_ws=ws)
    plain = P.block_score(q, k, shape)
    torch.cuda.synchronize()
    ref = oracle.block_scores(to_f64(q), to_f64(k), block)
    tol = 1e-3 * np.abs(ref).max()
    np.testing.assert_allclose(s0.cpu().numpy(), ref, atol=tol, rtol=0)
    np.testing.assert_allclose(s1.cpu().numpy(), ref + bias.cpu().numpy()[:, None, :], atol=tol, rtol=0)
    # the two routes to the scores differ only by the summation order of the key means
    np.testing.assert_allclose(s0.cpu().numpy(), plain.cpu().numpy(), atol=2e-5 * np.abs(ref).max(), rtol=0)
    # the statistics workspace still serves the attention kernel afterwards
    k_sel = P.topk_count(nb, 0.3)
    idx, mask = P.route(s0, k_sel, 5, 0.1)
    out = P.sparse_attn_fwd(q, k, v, shape, idx, mask, ws=ws, prepared=True)
    torch.cuda.synchronize()
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group)
    assert_close(to_f64(out), res, what="attention after scoring from the statistics")
    with pytest.raises(P.PasaError):  # approximation off: the statistics call leaves no key means
        P.block_score(q, None, P.Shape.of(q, block=block, group=0), stats_ws=ws)


@pytest.mark.parametrize("grid,d,block,group", [((4, 16, 16), 64, 64, 32), ((5, 21, 13), 128, 64, 8),
                                                ((9, 20, 23), 128, 64, 32), ((9, 20, 23), 128, 64, 64),
                                                ((9, 20, 23), 128, 64, 1000), ((9, 20, 23), 128, 128, 32),
                                                ((9, 20, 23), 64, 64, 1)])
def test_key_prior_matches_oracle_and_feeds_the_scores(P, grid, d, block, group):
    """covariance-aware routing prior (Eq.8): beta against the oracle, then scores with it as key bias"""
    q, k, v = _inputs(grid, 2, d, seed=5)
    shape = P.Shape.of(q, block=block, group=group)
    ws = P.kv_stats(k, v, shape)
    beta = P.key_prior(k, v, shape, ws, eps=1e-6)
    torch.cuda.synchronize()
    ref = oracle.key_prior(to_f64(k), to_f64(v), block, group, eps=1e-6)
    if group == 1:  # every block is its own group: the norm is rounding noise, only "tiny" can be compared
        assert np.all(beta.cpu().numpy() < np.log(1e-2)) and np.all(ref < np.log(1e-5))
    else:
        np.testing.assert_allclose(beta.cpu().numpy(), ref, atol=2e-3, rtol=0)
    s = P.block_score(q, k, shape, key_bias=beta)
    torch.cuda.synchronize()
    want = oracle.block_scores(to_f64(q), to_f64(k), block) + beta.cpu().numpy().astype(np.float64)[:, None, :]
    np.testing.assert_allclose(s.cpu().numpy(), want, atol=1e-3 * np.abs(want).max(), rtol=0)


@pytest.mark.parametrize("n,heads,d,block,group", [
    (64 * 129 - 3, 1, 128, 64, 64),   # units of 1 block: 64 + 64 + 1 units in the three groups
    (64 * 90, 3, 64, 64, 32),         # units of 2 blocks: 16 + 16 + 13 units
    (64 * 21 + 1, 1, 128, 64, 1000),  # one group of 22 blocks, units of 1: remainder of 6 after 2 rounds of 8
    (128 * 5, 2, 64, 128, 4),         # a group of one block behind a whole one
])
def test_statistics_of_small_problems(P, n, heads, d, block, group):
    """few blocks: the units of the statistics shrink and the groups are put together from many of them.  Tolerances as in
    the tests of the prior and of the attention above and below (fp32 sums in another order move neither)"""
    q, k, v = _inputs((1, 1, n), heads, d, seed=n)
    shape = P.Shape.of(q, block=block, group=group)
    ws = P.kv_stats(k, v, shape, ws=torch.full((P.attn_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda"))
    beta = P.key_prior(k, v, shape, ws)
    idx, mask = P.route(P.block_score(q, k, shape), 1, 3, 0.2)
    out = P.sparse_attn_fwd(q, k, v, shape, idx, mask, ws=ws, prepared=True)
    torch.cuda.synchronize()
    want, got = oracle.key_prior(to_f64(k), to_f64(v), block, group, eps=1e-6), beta.cpu().numpy()
    alone = want < np.log(1e-5)  # a block that is its own group: the norm is rounding noise
    np.testing.assert_allclose(got[~alone], want[~alone], atol=2e-3, rtol=0)
    assert np.all(got[alone] < np.log(1e-2))
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group)
    assert_close(to_f64(out), res, what="attention with the statistics of a small problem")


@pytest.mark.parametrize("n,heads,d,block,group", [(64 * 129 - 3, 1, 128, 64, 64), (64 * 90, 3, 64, 64, 32), (64 * 21 + 1, 1, 128, 64, 1000),
                                                   (64 * 100, 2, 128, 64, 96), (128 * 5, 2, 64, 128, 4)])
def test_statistics_without_room_for_small_units(P, n, heads, d, block, group):
    """the smallest workspace that is accepted: the statistics take the units that it has room for, nothing behind it is touched, and
    statistics made with the room are read by calls that are told of the smaller size (and the other way round)"""
    q, k, v = _inputs((1, 1, n), heads, d, seed=n)
    shape = P.Shape.of(q, block=block, group=group)
    full, least = P.attn_workspace_bytes(shape), attn_layout(shape)[0]
    whole = [torch.full((full + 4096,), 0xFF, dtype=torch.uint8, device="cuda") for _ in range(2)]
    idx, mask = P.route(P.block_score(q, k, shape), 1, 3, 0.2)
    P.kv_stats(k, v, shape, ws=whole[0][:least])
    assert bool((whole[0][least:] == 0xFF).all())
    P.kv_stats(k, v, shape, ws=whole[1][:full])
    want = oracle.key_prior(to_f64(k), to_f64(v), block, group, eps=1e-6)
    alone = want < np.log(1e-5)  # a block that is its own group: the norm is rounding noise
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group)
    for w, size in ((whole[0], full), (whole[0], least), (whole[1], full), (whole[1], least)):
        beta = P.key_prior(k, v, shape, w[:size]).cpu().numpy()
        np.testing.assert_allclose(beta[~alone], want[~alone], atol=2e-3, rtol=0)
        assert_close(to_f64(P.sparse_attn_fwd(q, k, v, shape, idx, mask, ws=w[:size], prepared=True)), res, what=f"{size} bytes")


@pytest.mark.parametrize("n,heads,d,block,group,unit", [(64 * 110 - 39, 60, 64, 64, 32, 16),  # (the prior's kernel takes 8 blocks in all of these)
                                                        (64 * 110, 40, 128, 64, 64, 16),      # the same, four units to a group
                                                        (128 * 52 + 5, 116, 64, 128, 1000, 16),  # one group of 53 blocks
                                                        (64 * 110, 40, 64, 64, 16, 16)])       # a unit is a group, the prior's half of one
def test_statistics_in_larger_units_than_the_prior_takes(P, n, heads, d, block, group, unit):
    """more units of 8 than run at a time: the statistics take larger ones, the prior's kernel its own.  First and last head against
    the oracle, tolerances as above"""
    gen = torch.Generator(device="cuda").manual_seed(n)  # (a smooth field along one axis of this length is slow to make)
    q, k, v = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=block, group=group)
    ws = P.kv_stats(k, v, shape, ws=torch.full((P.attn_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda"))
    _, at, slots = attn_layout(shape)  # one slot for every unit of 8 blocks: those of larger units stay as they were
    sums = ws[at:at + heads * slots * d * d * 4].view(torch.int32).view(heads, slots, d * d)
    assert slots == -(-P.num_blocks(shape) // 8) and int((sums != -1).any(-1).sum()) == heads * -(-P.num_blocks(shape) // unit)
    beta = P.key_prior(k, v, shape, ws)
    idx, mask = P.route(P.block_score(q, k, shape), 1, 3, 0.2)
    out = P.sparse_attn_fwd(q, k, v, shape, idx, mask, ws=ws, prepared=True)
    torch.cuda.synchronize()
    for h in (0, heads - 1):
        qh, kh, vh = (to_f64(t[:, h:h + 1]) for t in (q, k, v))
        np.testing.assert_allclose(beta[h:h + 1].cpu().numpy(), oracle.key_prior(kh, vh, block, group, eps=1e-6), atol=2e-3, rtol=0)
        res = oracle.pasa_attention(qh, kh, vh, idx[h:h + 1].cpu().numpy(), block, group=group)
        assert_close(to_f64(out[:, h:h + 1]), res, what=f"head {h}")


# ------------------------------------------------------------------------------------------------
# stage 2: routing is bit-exact against the oracle fed the GPU's scores
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("nb,k_sel,amp", [(16, 4, 0.0), (16, 4, 0.5), (67, 9, 1.0), (130, 130, 0.3), (515, 77, 2.0),
                                          (1182, 177, 0.7), (64, 1, 0.1), (1000, 150, 0.3), (1500, 1500, 0.1),
                                          (2000, 3, 0.2), (4096, 300, 0.5)])
def test_routing_bit_exact(P, nb, k_sel, amp):
    g = torch.Generator("cuda").manual_seed(nb)
    scores = torch.randn((3, nb, nb), device="cuda", generator=g)
    scores[0, 0, : nb // 2] = 0.25  # ties
    scores[1, 1, :] = -1.5          # a fully tied row
    scores[2, 0, 0] = -0.0
    seed = 0x1234_5678_9ABC_DEF0 + nb
    idx, mask = P.route(scores, k_sel, seed, amp)
    torch.cuda.synchronize()
    want = oracle.route(scores.cpu().numpy(), k_sel, seed, amp)
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    words = mask.cpu().numpy().view(np.uint32)
    bits = np.zeros((3, nb, words.shape[-1] * 32), bool)
    for h in range(3):
        for i in range(nb):
            bits[h, i, want[h, i]] = True
    packed = np.packbits(bits.reshape(3, nb, -1, 32), axis=-1, bitorder="little").view(np.uint32)[..., 0]
    np.testing.assert_array_equal(words, packed)


@pytest.mark.parametrize("nb,k_sel,tau", [(16, 4, 0.0), (67, 9, 1.0), (515, 77, 0.3), (1182, 177, 0.125)])
def test_gumbel_routing_matches_oracle_up_to_the_rounding_of_the_logarithms(P, nb, k_sel, tau):
    """Relaxed parity: the oracle takes the two logarithms in fp64, the kernel in binary32, so a block may differ
    only if its perturbed logit lies within rounding distance of the k-th largest of its row."""
    g = torch.Generator("cuda").manual_seed(nb)
    scores = torch.randn((3, nb, nb), device="cuda", generator=g)
    seed = 0x0FED_CBA9_8765_4321 + nb
    idx, mask = P.route(scores, k_sel, seed, tau, noise="gumbel")
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    want, r = oracle.route_gumbel(scores.cpu().numpy(), k_sel, seed, tau, return_noisy=True)
    assert (np.diff(got, axis=-1) > 0).all() and got.min() >= 0 and got.max() < nb  # k distinct blocks, ascending
    bits = (mask.cpu().numpy().view(np.uint32)[..., None] >> np.arange(32, dtype=np.uint32)) & 1
    sel = np.zeros((3, nb, nb), bool)
    np.put_along_axis(sel, got.astype(np.int64), True, axis=-1)
    np.testing.assert_array_equal(bits.reshape(3, nb, -1)[..., :nb].astype(bool), sel)
    # |g| <= 17 for this grid of u; binary32 logarithms and the fused multiply-add: a few ulp of the largest term
    delta = 64 * 2.0**-24 * (np.abs(r).max() + 17 * tau)
    kth = np.sort(r, axis=-1)[..., nb - k_sel][..., None]
    want_sel = np.zeros_like(sel)
    np.put_along_axis(want_sel, want.astype(np.int64), True, axis=-1)
    differ = sel != want_sel
    assert (np.abs(r - kth)[differ] <= delta).all()
    assert differ.mean() < 1e-3
    if tau == 0.0:
        assert not differ.any()



def test_routing_on_real_scores_and_determinism(P):
    q, k, _ = _inputs((4, 16, 16), 2, 64)
    shape = P.Shape.of(q)
    scores = P.block_score(q, k, shape)
    idx, mask = P.route(scores, 4, 99, 0.4)
    idx2, mask2 = P.route(scores, 4, 99, 0.4)
    idx3, _ = P.route(scores, 4, 100, 0.4)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2) and torch.equal(mask, mask2)
    assert not torch.equal(idx, idx3)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.route(scores.cpu().numpy(), 4, 99, 0.4))


# ------------------------------------------------------------------------------------------------
# stages 3+4: piecewise attention
# ------------------------------------------------------------------------------------------------
def _run_sparse(P, q, k, v, block, group, keep, seed=3, amp=0.3, kv_slices=0):
    shape = P.Shape.of(q, block=block, group=group, kv_slices=kv_slices)
    nb = P.num_blocks(shape)
    k_sel = P.topk_count(nb, keep)
    scores = P.block_score(q, k, shape)
    idx, mask = P.route(scores, k_sel, seed, amp)
    out, lse = P.sparse_attn_fwd(q, k, v, shape, idx, mask, want_lse=True)
    torch.cuda.synchronize()
    return out, lse, idx


CASES = [
    # grid, heads, d, block, group, keep
    ((4, 16, 16), 2, 64, 64, 32, 0.25),     # the tiny workload
    ((4, 16, 16), 2, 128, 64, 32, 0.25),
    ((5, 21, 13), 2, 128, 64, 32, 0.2),     # n=1365: 22 blocks, tail of 21 tokens
    ((9, 20, 23), 1, 128, 64, 32, 0.15),    # n=4140: 65 blocks (3 chunks, last group 1 block), tail 44
    ((9, 20, 23), 1, 128, 128, 32, 0.1),    # block 128: 33 blocks, tail 44 (< 64: second half-tile empty)
    ((9, 20, 23), 1, 128, 64, 0, 0.15),     # approximation off
    ((9, 20, 23), 1, 128, 64, 1000, 0.15),  # one global matrix (Eq.6/Eq.7)
    ((9, 20, 23), 1, 128, 64, 64, 0.15),    # 64 blocks per group
    ((9, 20, 23), 1, 128, 64, 8, 0.15),     # small groups
    ((9, 20, 23), 1, 128, 64, 1, 0.05),     # per-block first-order term (Eq.13)
    ((9, 20, 23), 1, 64, 128, 32, 0.1),
    ((1, 5, 7), 1, 128, 64, 32, 1.0),       # n=35: shorter than one tile
    ((1, 9, 11), 2, 64, 64, 32, 0.5),       # n=99: two blocks, the second one ragged; one block each selected
    ((2, 16, 16), 1, 128, 64, 32, 0.3),     # n=512: no ragged tile at all
    ((1, 9, 11), 1, 128, 128, 32, 1.0),     # n=99 with 128-token blocks: a single block, its second tile ragged
    ((12, 30, 33), 1, 128, 64, 32, 0.1),    # n=11880: 186 blocks = 6 chunks (5 of them whole), tail of 40 tokens
    ((12, 30, 32), 1, 64, 64, 64, 0.1),     # n=11520: 180 blocks, groups of two chunks, head dimension 64
    ((12, 30, 32), 1, 128, 128, 32, 0.1),   # 90 blocks of 128 tokens: 3 chunks
]


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257, 320])
def test_sequence_lengths_around_tile_and_block_boundaries(P, n, block):
    """every length around a multiple of 64 and of 128, dense and sparse (one of two, or two of three blocks kept)"""
    q, k, v = _inputs((1, 1, n), 1, 128, seed=n)
    shape = P.Shape.of(q, block=block, group=32)
    out = P.attn_dense_ref(q, k, v, shape)
    torch.cuda.synchronize()
    assert_close(to_f64(out), oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v)), what=f"dense n={n}")
    out, lse, idx = _run_sparse(P, q, k, v, block, 32, 0.6)
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=32, return_all=True)
    assert_close(to_f64(out), res["o"], what=f"sparse n={n} b={block}")
    np.testing.assert_allclose(lse.cpu().numpy(), res["lse"], atol=2e-2)


def test_sparse_path_respects_strides_batch_and_scale(P):
    """Q, K, V and O as views of token-major storage [B, n, H, d + pad] (what a transformer block hands over),
    batch 2, a non-default logit scale: every stage reads through the strides of the shape"""
    q, k, v = _inputs((5, 21, 13), 3, 128, seed=13, batch=2)
    B, H, n, d = q.shape
    big = torch.zeros((4, B, n, H, d + 8), dtype=torch.bfloat16, device="cuda")
    for i, t in enumerate((q, k, v)):
        big[i, :, :, :, :d] = t.permute(0, 2, 1, 3)
    qs, ks, vs, out = (big[i, :, :, :, :d].permute(0, 2, 1, 3) for i in range(4))
    scale = 0.07
    shape = P.Shape.of(qs, block=64, group=32, scale=scale)
    nb = P.num_blocks(shape)
    k_sel = P.topk_count(nb, 0.2)
    scores = P.block_score(qs, ks, shape)
    idx, mask = P.route(scores, k_sel, 77, 0.2)
    P.sparse_attn_fwd(qs, ks, vs, shape, idx, mask, out=out)
    torch.cuda.synchronize()
    ref_scores = oracle.block_scores(to_f64(q), to_f64(k), 64, scale=scale)
    np.testing.assert_allclose(scores.cpu().numpy(), ref_scores, atol=1e-3 * np.abs(ref_scores).max(), rtol=0)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.route(scores.cpu().numpy(), k_sel, 77, 0.2))
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), 64, group=32, scale=scale)
    assert_close(to_f64(out), res, what="strided sparse path")
    assert torch.all(big[3, :, :, :, d:] == 0)  # the padding between rows was not written


@pytest.mark.parametrize("grid,heads,d,block,group,keep", CASES)
def test_sparse_matches_oracle(P, grid, heads, d, block, group, keep):
    q, k, v = _inputs(grid, heads, d, seed=7)
    out, lse, idx = _run_sparse(P, q, k, v, block, group, keep)
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group,
                                return_all=True)
    assert_close(to_f64(out), res["o"], what=f"sparse {grid} d={d} b={block} G={group}")
    np.testing.assert_allclose(lse.cpu().numpy(), res["lse"], atol=2e-2)


SLICED_CASES = [
    # grid, d, block, group, keep, kv_slices   (needs at least kv_slices chunks of 32 key blocks)
    ((8, 45, 46), 128, 64, 32, 0.15, 8),    # n=16,560: 259 blocks (tail 48), 9 chunks over 8 slices
    ((8, 45, 46), 128, 64, 0, 0.02, 8),     # approximation off, very sparse: some slices hold no selected block
    ((12, 40, 46), 64, 64, 32, 0.1, 8),     # d = 64
    ((16, 40, 52), 128, 64, 32, 0.05, 16),  # n=33,280: 520 blocks, 17 chunks over 16 slices (two rounds per XCD)
    ((16, 40, 52), 128, 128, 32, 0.1, 8),   # block 128: 260 blocks, 9 chunks
]


@pytest.mark.parametrize("grid,d,block,group,keep,kv_slices", SLICED_CASES)
def test_key_range_slicing_matches_oracle_and_unsliced_kernel(P, grid, d, block, group, keep, kv_slices):
    q, k, v = _inputs(grid, 1, d, seed=13)
    out, lse, idx = _run_sparse(P, q, k, v, block, group, keep, kv_slices=kv_slices)
    out1, lse1, idx1 = _run_sparse(P, q, k, v, block, group, keep, kv_slices=1)
    assert torch.equal(idx, idx1)
    # same arithmetic up to summation order and one bf16 rounding
    a, b = out.float(), out1.float()
    assert (a - b).abs().max().item() <= 2e-2 * b.abs().max().item()
    assert (a - b).abs().mean().item() <= 1e-3 * b.abs().mean().item()
    np.testing.assert_allclose(lse.cpu().numpy(), lse1.cpu().numpy(), atol=1e-3)
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group,
                                return_all=True)
    assert_close(to_f64(out), res["o"], what=f"sliced {grid} d={d} b={block} G={group} S={kv_slices}")
    np.testing.assert_allclose(lse.cpu().numpy(), res["lse"], atol=2e-2)


def _lists(rng, nb, k_sel, keep_own):
    """index lists [1, nb, k_sel]: every row selects (keep_own: both, first, none) of the blocks 2 (i // 2), 2 (i // 2) + 1, the
    ones its workgroup visits first if they are in both rows of the pair, and random others"""
    idx = np.empty((1, nb, k_sel), np.int32)
    for i in range(nb):
        pair = [j for j in (i - i % 2, i - i % 2 + 1) if j < nb]
        own = {"both": pair, "first": pair[:1], "none": []}[keep_own]
        rest = rng.permutation([j for j in range(nb) if j not in pair])[:k_sel - len(own)]
        idx[0, i] = np.sort(np.concatenate([own, rest]).astype(np.int32))
    return idx


@pytest.mark.parametrize("n,d,block,kv_slices", [(1283, 128, 64, 0), (1345, 64, 64, 0), (1408, 128, 128, 0), (1409, 64, 128, 0),
                                                 (16460, 64, 64, 8)])
@pytest.mark.parametrize("keep_own", ["both", "first", "none"])
def test_blocks_visited_first_are_visited_once(P, n, d, block, kv_slices, keep_own):
    """whole, ragged and missing partners of the last pair, 128-token blocks, walks that start in the middle of the bitmap"""
    rng = np.random.default_rng(n)
    q, k, v = _inputs((1, 1, n), 1, d, seed=n)
    shape = P.Shape.of(q, block=block, group=32, kv_slices=kv_slices)
    nb = P.num_blocks(shape)
    idx = _lists(rng, nb, 7, keep_own)
    out, lse = P.sparse_attn_fwd(q, k, v, shape, torch.from_numpy(idx).cuda(), None, want_lse=True)
    torch.cuda.synchronize()
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx, block, group=32, return_all=True)
    assert_close(to_f64(out), res["o"], what=f"{n} d={d} b={block} own={keep_own}")
    np.testing.assert_allclose(lse.cpu().numpy(), res["lse"], atol=2e-2)


def _bitmap(chosen):
    """[BH, nb, nb] booleans -> [BH, nb, words] int32"""
    bh, nb, _ = chosen.shape
    bits = torch.nn.functional.pad(chosen, (0, -nb % 32)).view(bh, nb, -1, 32).long() << torch.arange(32, device=chosen.device)
    word = bits.sum(-1)
    return torch.where(word >= 2 ** 31, word - 2 ** 32, word).to(torch.int32)


def _quad_heads(P, n, group, d=128, batch=1):
    """the fewest heads that take workgroups of four query blocks (keys and values have to exceed the caches)"""
    of = lambda h: P.Shape(batch, h, n, d, 64, group, h * n * d, n * d, d)
    return next(h for h in range(1, 41) if P.attn_variant(of(h), 353) == "quad")


@pytest.mark.parametrize("n,group,kind", [
    (75712, 32, "routed"), (75713, 64, "routed"), (75775, 2000, "routed"), (75840, 0, "routed"), (75904, 32, "routed"),
    (75712, 32, "uneven"), (75841, 0, "uneven"), (75967, 32, "uneven"), (76800, 32, "same"), (76801, 32, "apart"),
    (76480, 64, "one"), (76481, 32, "empty"), (262144, 32, "few"), (262145, 0, "few")])
def test_workgroups_of_four_query_blocks_against_two(P, n, group, kind):
    """The number of selected blocks that the caller declares decides between workgroups of four and of two query blocks; the kernels read
    the bitmap, so the same bitmap is given to both.  Numbers of query blocks with 0 to 3 left over, ragged last blocks of 1 and 63 tokens; equal numbers
    of selected blocks (routed), very different ones in neighbouring rows, none and all of them (uneven), four rows alike, four rows without a common
    block, one block, no whole block at all in some rows (empty), as many key blocks as can be planned and a ragged one more"""
    _compare_routes(P, n, _quad_heads(P, n, group), 128, group, kind, 353, "quad")


@pytest.mark.parametrize("n,heads,d,group,kind", [
    (4096, 4, 128, 64, "routed"), (4097, 3, 128, 32, "routed"), (4159, 2, 64, 16, "routed"), (8191, 2, 128, 0, "uneven"), (4161, 4, 64, 32, "uneven"),
    (5000, 2, 64, 1000, "same"), (5120, 1, 128, 8, "apart"), (4224, 3, 128, 32, "one"), (4225, 2, 64, 32, "empty")])
def test_ring_of_eight_tiles_against_four(P, n, heads, d, group, kind):
    """The same for small grids, where the declared number decides between rings of eight and of four tiles: odd and even numbers of
    shared and of private blocks, one query block running out of them before the other, ragged last blocks of 1, 8, 33 and 63 tokens"""
    _compare_routes(P, n, heads, d, group, kind, 8, "deep")


@pytest.mark.parametrize("n,heads,d,group,kind", [
    (1500, 3, 128, 32, "routed"), (1409, 2, 128, 8, "uneven"), (1536, 2, 128, 0, "one"), (4140, 2, 64, 32, "routed"), (4097, 2, 64, 16, "uneven"),
    (4160, 1, 64, 0, "one")])
def test_blocks_of_128_in_short_walks_against_pipelined_steps(P, n, heads, d, group, kind):
    """The declared number of blocks decides between steps of one tile and pipelined ones; a tile's keys are met in the same order and the same halves in
    both, so the results have the same bits.  Ragged last blocks of 1, 44, 64, 92 tokens and none; rows of one block, of none but the ragged one, of all"""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=128, group=group)
    nb, few = P.num_blocks(shape), 5 if d == 128 else 31
    assert P.attn_variant(shape, few) == "short" and P.attn_variant(shape, few + 1) == "whole"
    if kind == "routed":
        _, mask = P.route(P.block_score(q, k, shape), nb // 3, 5, 0.5)
    else:
        chosen = torch.rand((heads, nb, nb), generator=g, device="cuda") < torch.linspace(-0.3, 1.3, nb, device="cuda")[:, None]
        if kind == "one":
            chosen = (torch.arange(nb, device="cuda")[:, None] == torch.arange(nb, device="cuda").flip(0)).expand(heads, -1, -1).clone()
        chosen[:, :, nb - 1] |= ~chosen.any(-1)
        mask = _bitmap(chosen)
    ws = P.kv_stats(k, v, shape, ws=torch.empty(P.attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda"))
    short, short_lse = P.sparse_attn_fwd(q, k, v, shape, None, mask, ws=ws, want_lse=True, prepared=True, k_sel=few)
    whole, whole_lse = P.sparse_attn_fwd(q, k, v, shape, None, mask, ws=ws, want_lse=True, prepared=True, k_sel=few + 1)
    torch.cuda.synchronize()
    assert torch.isfinite(whole.float()).all()
    assert torch.equal(short, whole) and torch.equal(short_lse, whole_lse)


def _compare_routes(P, n, heads, d, group, kind, declared, variant):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + heads)
    q, k, v = (torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=64, group=group)
    assert P.attn_variant(shape, declared) == variant and P.attn_variant(shape, 1) == "whole"
    nb = P.num_blocks(shape)
    u = torch.rand((heads, nb, nb), generator=g, device="cuda")
    rows = torch.arange(nb, device="cuda")[:, None]
    if kind == "routed":
        idx, mask = P.route(P.block_score(q, k, shape), min(60, nb // 6), 7, 0.5)
    else:
        density = {"same": 0.2, "apart": 0.2, "few": 40 / nb}.get(kind, 0.1)
        if kind == "uneven":
            density = torch.tensor([0.0, 0.004, 0.02, 0.3, 1.1], device="cuda")[torch.randint(0, 5, (nb, 1), generator=g, device="cuda")]
        if kind == "same":
            u = u[:, :1].expand(-1, nb, -1)
        chosen = u < density
        if kind == "apart":
            chosen = chosen & (torch.arange(nb, device="cuda")[None, :] % 4 == rows % 4)
        if kind == "one":
            chosen = (rows * 7 + 3) % nb == torch.arange(nb, device="cuda")[None, :]
            chosen = chosen.expand(heads, -1, -1).clone()
        if kind == "empty":  # nothing but the ragged last block
            chosen = chosen & (rows % 3 == 0)
        if kind in ("uneven", "empty"):
            chosen = chosen.clone()
            chosen[:, :, nb - 1] |= ~chosen.any(-1)
        mask = _bitmap(chosen)
    ws = torch.empty(P.attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    P.kv_stats(k, v, shape, ws=ws)
    out4, lse4 = P.sparse_attn_fwd(q, k, v, shape, None, mask, ws=ws, want_lse=True, prepared=True, k_sel=declared)
    again = P.sparse_attn_fwd(q, k, v, shape, None, mask, ws=ws, prepared=True, k_sel=declared)
    out2, lse2 = P.sparse_attn_fwd(q, k, v, shape, None, mask, ws=ws, want_lse=True, prepared=True, k_sel=1)
    torch.cuda.synchronize()
    assert torch.equal(out4, again)
    if declared > 100 and kind not in ("one", "empty", "same"):
        assert not torch.equal(out4, out2)  # (so both did run; rows that are all alike meet their blocks in the same order in both)
    # P is rounded to bf16 relative to the maximum so far, so differently in the two orders.  The values are white noise, whose weighted mean is as small
    # as the error that the rounding makes of it: 2^-9 / sqrt(3) of the result for each, 1.6e-3 for both, and 2^-9 / sqrt(12) twice for the
    # output's own rounding: 1.8e-3 in the 2-norm, which bounds the mean of the absolute values
    a, b = out4.float(), out2.float()
    assert torch.isfinite(a).all()
    for h in range(heads):
        assert (a[0, h] - b[0, h]).abs().max().item() <= 2e-2 * b[0, h].abs().max().item()
        assert (a[0, h] - b[0, h]).abs().mean().item() <= 2e-3 * b[0, h].abs().mean().item()
    np.testing.assert_allclose(lse4.cpu().numpy(), lse2.cpu().numpy(), atol=1e-3)


@pytest.mark.parametrize("variant,n,d,block,declared", [
    ("quad", 75841, 128, 64, 353), ("quad", 75810, 128, 64, 353), ("deep", 4161, 128, 64, 8), ("deep", 4131, 64, 64, 8), ("whole", 1345, 128, 64, 4),
    ("whole", 1500, 128, 128, 6), ("short", 1409, 64, 128, 3), ("wide", 1089, 128, 64, 0), ("wide", 1281, 64, 64, 0), ("teams", 1345, 128, 64, 0),
    ("short_teams", 575, 64, 64, 0), ("short", 300, 128, 64, 0)])
def test_forms_of_the_kernel_respect_strides_batch_and_scale(P, variant, n, d, block, declared):
    """Every form of the attention kernel (declared = 0: dense) on views of token-major storage [B, n, H, d + pad], batch 2, a scale of the caller's and a
    ragged last block: the bits of the contiguous run, nothing written beside the output (the inputs' padding holds NaN), and the oracle's values"""
    B, scale, group = 2, 0.07, 32
    of = lambda h: P.Shape(B, h, n, d, block, group, h * n * d, n * d, d, scale)
    heads = next(h for h in range(1, 41) if P.attn_variant(of(h), declared) == variant)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn((B, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    big = torch.full((4, B, n, heads, d + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
    big[3] = 7.0
    for i, t in enumerate((q, k, v)):
        big[i, :, :, :, :d] = t.permute(0, 2, 1, 3)
    qs, ks, vs, out_s = (big[i, :, :, :, :d].permute(0, 2, 1, 3) for i in range(4))
    shape, strided = of(heads), P.Shape.of(qs, block=block, group=group, scale=scale)
    assert P.attn_variant(strided, declared) == variant
    if declared:
        nb = P.num_blocks(shape)
        idx, mask = P.route(P.block_score(q, k, shape), min(declared, 60), 9, 0.5)
        out, lse = P.sparse_attn_fwd(q, k, v, shape, None, mask, want_lse=True, k_sel=declared)
        _, lse_s = P.sparse_attn_fwd(qs, ks, vs, strided, None, mask, out=out_s, want_lse=True, k_sel=declared)
    else:
        out, lse = P.attn_dense_ref(q, k, v, shape, want_lse=True)
        _, lse_s = P.attn_dense_ref(qs, ks, vs, strided, out=out_s, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out_s, out) and torch.equal(lse_s, lse)
    assert (big[3, :, :, :, d:] == 7.0).all()
    last = tuple(to_f64(t[-1:, -1:]) for t in (q, k, v))
    got, got_lse = to_f64(out[-1:, -1:]), lse[-1].cpu().numpy()
    if declared:
        blocks = sorted({0, nb // 2, nb - 3, nb - 2, nb - 1})
        res = oracle.pasa_attention(*last, idx[-1:].cpu().numpy(), block, group=group, scale=scale, q_blocks=blocks, return_all=True)
        rows = np.concatenate([np.arange(j * block, min((j + 1) * block, n)) for j in blocks])
        ref, ref_lse = res["o"][:, rows], res["lse"][0, rows]
    else:
        rows = np.unique(np.concatenate([np.arange(0, n, 7), np.arange(n - 70, n)]))
        ref, ref_lse = oracle.dense_attention(*last, scale=scale, q_rows=rows, return_lse=True)
        ref_lse = ref_lse[0]
    assert_close(got[:, rows], ref, what=f"{variant} n={n} d={d}")
    np.testing.assert_allclose(got_lse[rows], ref_lse, atol=2e-2)


@pytest.mark.parametrize("variant,n,d,block,group,step,declared", [
    ("whole", 133 * 64 - 9, 128, 64, 96, 2.0, 1), ("whole", 133 * 64 - 9, 64, 64, 96, 2.0, 1), ("whole", 133 * 128 - 70, 128, 128, 128, 1.5, 8),
    ("short", 133 * 128 - 70, 128, 128, 128, 1.5, 1), ("deep", 133 * 64 - 9, 128, 64, 1000, 1.5, 8), ("deep", 133 * 64 - 9, 64, 64, 96, 2.0, 8),
    ("quad", 75610, 128, 64, 320, 0.5, 353)])
def test_weights_of_a_group_follow_a_maximum_that_grows_within_it(P, variant, n, d, block, group, step, declared):
    """A group's first-order term takes the summed weights of its chunks of 32 blocks, each relative to the maximum at its time.  Here every row selects the
    last block, whose logits are low, and the mean-key logits rise by `step` from chunk to chunk: sums that stayed relative to an older maximum would
    count e^step times too much a chunk.  The first component of the keys carries the logit and a deviation of +-1/2 that the values follow, so the
    first-order term is half as large as the zeroth one; both are exact in bf16"""
    of = lambda h: P.Shape(1, h, n, d, block, group, h * n * d, n * d, d)
    heads = next(h for h in range(1, 41) if P.attn_variant(of(h), declared) == variant)
    shape = of(heads)
    nb = P.num_blocks(shape)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    rnd = lambda *size: torch.randn(size, generator=g, device="cuda")
    token = torch.arange(n, device="cuda")
    chunk = token // (32 * block)
    side = (token % 2).float() * 2 - 1
    q, k, v = rnd(n, d), 0.1 * rnd(n, d), 1.0 + 0.3 * rnd(n, d) + side[:, None]
    q[:, 0] = d ** 0.5
    k[:, 0] = torch.where(chunk == chunk[-1], torch.full_like(side, -4.0), step * chunk) + side / 2
    q, k, v = (t.to(torch.bfloat16).expand(1, heads, n, d).contiguous() for t in (q, k, v))
    idx = torch.full((heads, nb, 1), nb - 1, dtype=torch.int32, device="cuda")
    out, lse = P.sparse_attn_fwd(q, k, v, shape, None, _bitmap(torch.arange(nb, device="cuda").expand(heads, nb, nb) == nb - 1), want_lse=True, k_sel=declared)
    torch.cuda.synchronize()
    blocks = sorted({0, 1, 2, 3, nb // 2, nb - 2, nb - 1})
    first = tuple(to_f64(t[:, :1]) for t in (q, k, v))
    res = oracle.pasa_attention(*first, idx[:1].cpu().numpy(), block, group=group, q_blocks=blocks, return_all=True)
    rows = np.concatenate([np.arange(j * block, min((j + 1) * block, n)) for j in blocks])
    part = np.abs(res["parts"][0, rows])
    assert part[:, 2].mean() > 0.3 * part[:, 1].mean()  # the term is there
    for h in {0, heads - 1}:
        assert_close(to_f64(out[:, h:h + 1])[:, rows], res["o"][:, rows], what=f"{variant} head {h}")
        np.testing.assert_allclose(lse[h].cpu().numpy()[rows], res["lse"][0, rows], atol=2e-2)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_values_of_a_ragged_block_that_a_neighbour_selected_stay_out(P, bad):
    """workgroups of four query blocks fetch the ragged last key block for whichever of them selected it; without the approximation a query
    block that did not select it must not see its values, also where they are not finite"""
    n, declared = 75610, 353
    heads = _quad_heads(P, n, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    q, k, v = (torch.randn((1, heads, n, 128), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=64, group=0)
    assert P.attn_variant(shape, declared) == "quad"
    nb = P.num_blocks(shape)
    chosen = torch.rand((1, nb, nb), generator=g, device="cuda") < 0.02
    chosen[:, :, 0] = True
    chosen[:, :, nb - 1] = torch.arange(nb, device="cuda") % 4 == 1
    mask = _bitmap(chosen).expand(heads, -1, -1).contiguous()
    clean = P.sparse_attn_fwd(q, k, v, shape, None, mask, k_sel=declared)
    v[:, :, 64 * (nb - 1):] = bad
    out = P.sparse_attn_fwd(q, k, v, shape, None, mask, k_sel=declared)
    torch.cuda.synchronize()
    selected = (torch.arange(n, device="cuda") // 64) % 4 == 1
    assert torch.equal(out[:, :, ~selected], clean[:, :, ~selected])
    assert not torch.isfinite(out[:, :, selected].float()).any()


@pytest.mark.parametrize("n,heads,d,block", [(65536, 9, 128, 64), (65537, 7, 128, 64), (65537, 8, 128, 64), (131072, 1, 64, 64),
                                              (128 * 2049 + 77, 1, 64, 128)])
def test_blocks_visited_first_at_the_ends_of_the_rule(P, n, heads, d, block):
    """keys and values of 32 MB a head and just above, of 256 MB in all and just above; own blocks in the last word of the walk's
    first 64 words and beyond it.  First and last head"""
    gen = torch.Generator(device="cuda").manual_seed(n)  # (a smooth field along one axis of this length is slow to make)
    q, k, v = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=block, group=32)
    nb = P.num_blocks(shape)
    rng = np.random.default_rng(n)
    idx = np.empty((heads, nb, 7), np.int32)
    for i in range(nb):  # the workgroup's own pair (or the block alone at an odd end) and random others, the same in every head
        own = {i - i % 2, min(i - i % 2 + 1, nb - 1)}
        others = [j for j in rng.choice(nb, 9, replace=False) if j not in own]
        idx[:, i] = np.sort(np.array(sorted(own) + others[:7 - len(own)], np.int32))
    out, lse = P.sparse_attn_fwd(q, k, v, shape, torch.from_numpy(idx).cuda(), None, want_lse=True)
    torch.cuda.synchronize()
    blocks = sorted({0, 1, nb // 2, nb // 2 + 1, nb - 3, nb - 2, nb - 1})
    rows = np.concatenate([np.arange(j * block, min((j + 1) * block, n)) for j in blocks])
    for h in {0, heads - 1}:
        qh, kh, vh = (to_f64(t[:, h:h + 1]) for t in (q, k, v))
        res = oracle.pasa_attention(qh, kh, vh, idx[h:h + 1], block, group=32, q_blocks=blocks, return_all=True)
        assert_close(to_f64(out[:, h:h + 1]), res["o"], rows=rows, what=f"{n} d={d} b={block} head {h}")
        np.testing.assert_allclose(lse[h].cpu().numpy()[rows], res["lse"][0, rows], atol=2e-2)


@pytest.mark.parametrize("n,heads,batch,d,block,group", [(63, 1, 1, 64, 64, 32), (1345, 3, 1, 128, 64, 32), (1345, 2, 2, 64, 64, 1),
                                                         (2113, 2, 1, 64, 128, 64), (1345, 2, 1, 128, 64, 0)])
def test_bitmap_built_with_the_statistics_equals_the_callers(P, n, heads, batch, d, block, group):
    """index lists alone (the bitmap is built in the statistics launch, without the approximation in one of its own) against the
    routing's own bitmap: the same bits, whatever the workspace held"""
    q, k, v = _inputs((1, 1, n), heads, d, seed=n, batch=batch)
    shape = P.Shape.of(q, block=block, group=group)
    idx, mask = P.route(P.block_score(q, k, shape), P.topk_count(P.num_blocks(shape), 0.2), 3, 0.2)
    ws = torch.full((P.attn_workspace_bytes(shape),), 0xFF, dtype=torch.uint8, device="cuda")
    lists, lists_lse = P.sparse_attn_fwd(q, k, v, shape, idx, None, ws=ws, want_lse=True)
    both, both_lse = P.sparse_attn_fwd(q, k, v, shape, idx, mask, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(lists, both) and torch.equal(lists_lse, both_lse)


def test_keep_everything_equals_dense_kernel_and_oracle(P):
    q, k, v = _inputs((5, 21, 13), 2, 128, seed=2)
    out, _, idx = _run_sparse(P, q, k, v, 64, 32, 1.0)
    assert idx.shape[-1] == 22
    ref = oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v))
    assert_close(to_f64(out), ref, what="keep=1")
    dense = P.attn_dense_ref(q, k, v, P.Shape.of(q))
    torch.cuda.synchronize()
    assert_close(to_f64(out), to_f64(dense).astype(np.float64), what="keep=1 vs dense kernel")


def test_batch_and_heads_are_independent_and_results_are_deterministic(P):
    q, k, v = _inputs((3, 16, 16), 3, 128, seed=11, batch=2)
    out, _, idx = _run_sparse(P, q, k, v, 64, 32, 0.25)
    out2, _, idx2 = _run_sparse(P, q, k, v, 64, 32, 0.25)
    assert torch.equal(out, out2) and torch.equal(idx, idx2)  # bitwise run-to-run
    # batch 1, head 2 alone (routing noise is keyed by bh, so feed the same routing rows)
    shape1 = P.Shape.of(q[1:2, 2:3], block=64, group=32)
    bh = 1 * 3 + 2
    nb = idx.shape[1]
    mask = torch.zeros((1, nb, (nb + 31) // 32), dtype=torch.int32, device="cuda")
    words = np.zeros((nb, (nb + 31) // 32), np.uint32)
    for i, row in enumerate(idx[bh].cpu().numpy()):
        for j in row:
            words[i, j >> 5] |= np.uint32(1) << np.uint32(j & 31)
    mask[0] = torch.from_numpy(words.view(np.int32)).cuda()
    single = P.sparse_attn_fwd(q[1:2, 2:3], k[1:2, 2:3], v[1:2, 2:3], shape1, idx[bh:bh + 1].contiguous(), mask)
    torch.cuda.synchronize()
    assert torch.equal(single[0, 0], out[1, 2])
    ref = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), 64, group=32)
    assert_close(to_f64(out), ref, what="batch=2")


@pytest.mark.parametrize("grid,d,block,group,keep", [((4, 16, 16), 64, 64, 32, 0.25), ((9, 20, 23), 128, 64, 32, 0.15),
                                                     ((9, 20, 23), 128, 128, 8, 0.3), ((5, 21, 13), 128, 64, 0, 0.2)])
def test_single_call_forward_equals_the_stage_calls(P, grid, d, block, group, keep):
    """pasa_forward against the four stage entry points (bit for bit: the same kernels in the same order) and the oracle"""
    q, k, v = _inputs(grid, 2, d, seed=31)
    shape = P.Shape.of(q, block=block, group=group)
    nb = P.num_blocks(shape)
    k_sel = P.topk_count(nb, keep)
    out, lse = P.forward_single_call(q, k, v, shape, keep, 123, 0.2, want_lse=True)
    ws = P.kv_stats(k, v, shape)
    scores = P.block_score(q, None, shape, stats_ws=ws) if group > 0 else P.block_score(q, k, shape)
    idx, mask = P.route(scores, k_sel, 123, 0.2)
    want, want_lse = P.sparse_attn_fwd(q, k, v, shape, idx, mask, ws=ws, prepared=True, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and torch.equal(lse, want_lse)
    ref = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), block, group=group)
    assert_close(to_f64(out), ref, what="pasa_forward")


def test_forward_convenience_wrapper(P):
    q, k, v = _inputs((4, 16, 16), 2, 64)
    out, idx = P.forward(q, k, v, keep_ratio=0.25, seed=5, noise_amp=0.2)
    torch.cuda.synchronize()
    ref = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), 64, group=32)
    assert_close(to_f64(out), ref, what="forward()")


def test_forward_buffers_are_not_shared_between_layouts(P):
    """one buffers dict, the same shape head-major and token-major"""
    q, k, v = _inputs((4, 16, 16), 2, 64)
    want, want_idx = P.forward(q, k, v, keep_ratio=0.25, seed=5, noise_amp=0.2)
    want = want.clone()
    buffers = {}
    for layout in ("heads", "tokens", "heads"):
        x = (q, k, v) if layout == "heads" else tuple(t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v))
        out, idx = P.forward(*x, keep_ratio=0.25, seed=5, noise_amp=0.2, buffers=buffers)
        torch.cuda.synchronize()
        assert out.stride() == x[0].stride()
        assert torch.equal(out, want) and torch.equal(idx, want_idx), layout


# ------------------------------------------------------------------------------------------------
# calibration signal of the curvature-aware budget: mean L1 distance of two tensors
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n,dtype", [(1, torch.float32), (7, torch.bfloat16), (4096, torch.bfloat16), (1000003, torch.float32),
                                     (16 * 21 * 45 * 80 + 5, torch.bfloat16), (64 * 1024 * 1024, torch.bfloat16)])
def test_l1_distance_matches_oracle_and_is_deterministic(P, n, dtype):
    g = torch.Generator("cuda").manual_seed(n % 1000)
    a = torch.randn(n, device="cuda", generator=g).to(dtype)
    b = (a.float() + 0.3 * torch.randn(n, device="cuda", generator=g)).to(dtype)
    got = P.l1_distance(a, b)
    again = P.l1_distance(a, b)
    torch.cuda.synchronize()
    want = oracle.l1_distance(a.float().cpu().numpy(), b.float().cpu().numpy())
    assert abs(got.item() - want) <= 2e-6 * want + 1e-12
    assert got.item() == again.item()
    assert P.l1_distance(a, a).item() == 0.0


# ------------------------------------------------------------------------------------------------
# the whole path on a side stream and inside a HIP graph (launch-bound serving loops capture it)
# ------------------------------------------------------------------------------------------------
def test_forward_on_a_side_stream_and_in_a_graph_replays_identically(P):
    q, k, v = _inputs((9, 20, 23), 2, 128, seed=21)
    shape = P.Shape.of(q, block=64, group=32)
    nb = P.num_blocks(shape)
    k_sel = P.topk_count(nb, 0.15)
    scores = torch.empty((2, nb, nb), dtype=torch.float32, device="cuda")
    idx = torch.empty((2, nb, k_sel), dtype=torch.int32, device="cuda")
    mask = torch.empty((2, nb, P.mask_words(nb)), dtype=torch.int32, device="cuda")
    ws_s = torch.empty(P.score_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ws_a = torch.empty(P.attn_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)

    def run():
        P.block_score(q, k, shape, scores=scores, ws=ws_s)
        P.route(scores, k_sel, 99, 0.125, idx=idx, mask=mask)
        P.sparse_attn_fwd(q, k, v, shape, idx, mask, out=out, ws=ws_a)

    run()
    torch.cuda.synchronize()
    eager = out.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        out.zero_()
        run()
    side.synchronize()
    assert torch.equal(out, eager)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        (out.float().sum()).item()  # eager work between the replays


# ------------------------------------------------------------------------------------------------
# the method-variant tables (group sizes, routing noise, selection-count histogram) on the tiny workload
# ------------------------------------------------------------------------------------------------
def _table_rows(text):
    rows = [[c.strip() for c in line.strip().strip("|").split("|")] for line in text.splitlines() if line.startswith("|")]
    return [r for r in rows if not set("".join(r)) <= set("-")]  # without the separator rows


def test_sweep_tables_on_the_tiny_workload(P, capsys):
    import paper_2604_12219_amd.sweeps as sweeps
    sweeps.selection_histogram("tiny", 6, 1.0)  # a bias as large as the logit spread of this small workload
    rows = _table_rows(capsys.readouterr().out)
    assert [r[0] for r in rows[1:]] == ["deterministic", "stochastic, uniform bias", "stochastic, Gumbel bias"]
    pct = lambda s: float(s.rstrip("%"))
    for r in rows[1:]:
        assert abs(pct(r[1]) + pct(r[2]) + pct(r[3]) + pct(r[4]) - 100.0) < 0.5   # the four classes partition the pairs
        assert abs(pct(r[1]) + pct(r[5]) - 100.0) < 0.2                           # never + ever = all
    det, sto = rows[1], rows[2]
    assert pct(sto[5]) > pct(det[5])          # the seeded bias spreads the exact computation over more pairs ...
    assert float(sto[6]) < float(det[6])      # ... each of which is selected in fewer steps
    sweeps.sweep_noise("tiny")
    rows = _table_rows(capsys.readouterr().out)
    changed = [pct(r[1]) for r in rows[1:]]
    assert changed[0] == 0.0 and all(a <= b + 1e-9 for a, b in zip(changed, changed[1:])) and changed[-1] > 5.0
    sweeps.sweep_groups("tiny", 0.125, 1.0)
    rows = _table_rows(capsys.readouterr().out)
    assert [r[0] for r in rows[1:]] == ["0 (drop)", "1 (per block)", "16 (global)"] or rows[1][0] == "0 (drop)"
    errs = {r[0]: float(r[5]) for r in rows[1:]}
    assert errs["0 (drop)"] > errs["1 (per block)"]  # the approximation of the unselected blocks pays


# ------------------------------------------------------------------------------------------------
# seeded random configurations: shapes, strides, block and group sizes, keep ratios drawn at random
# ------------------------------------------------------------------------------------------------
def _random_config(rng):
    d = int(rng.choice([64, 128]))
    block = int(rng.choice([64, 128]))
    n = int(rng.integers(1, 2600))
    nb = (n + block - 1) // block
    group = int(rng.choice([0, 1, 2, 4, 8, 16, 32, 64, 10_000]))
    keep = float(rng.choice([0.02, 0.1, 0.25, 0.5, 0.9, 1.0]))
    heads, batch = int(rng.integers(1, 4)), int(rng.integers(1, 3))
    token_major = bool(rng.integers(0, 2))
    scale = float(rng.choice([0.0, 0.05, 0.2]))
    return dict(d=d, block=block, n=n, nb=nb, group=group, keep=keep, heads=heads, batch=batch, token_major=token_major, scale=scale)


@pytest.mark.parametrize("case", range(24))
def test_random_configurations_against_oracle(P, case):
    rng = np.random.default_rng(1000 + case)
    c = _random_config(rng)
    q, k, v = workloads.make_qkv((1, 1, c["n"]), c["heads"], c["d"], seed=case, device="cuda", batch=c["batch"])
    if c["token_major"]:
        q, k, v = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v))
    shape = P.Shape.of(q, block=c["block"], group=c["group"], scale=c["scale"])
    k_sel = P.topk_count(c["nb"], c["keep"])
    scale = c["scale"] if c["scale"] > 0 else None
    ws = P.kv_stats(k, v, shape)
    scores = P.block_score(q, None, shape, stats_ws=ws) if c["group"] > 0 else P.block_score(q, k, shape)
    idx, mask = P.route(scores, k_sel, 7 * case + 1, 0.3)
    out, lse = P.sparse_attn_fwd(q, k, v, shape, idx, mask, want_lse=True)
    dense = P.attn_dense_ref(q, k, v, shape)
    torch.cuda.synchronize()
    what = f"case {case}: {c}"
    assert P.check_selection(idx, mask, c["nb"], k_sel).item() == 0, what
    ref_scores = oracle.block_scores(to_f64(q), to_f64(k), c["block"], scale=scale)
    np.testing.assert_allclose(scores.cpu().numpy(), ref_scores, atol=1e-3 * max(np.abs(ref_scores).max(), 1e-3), rtol=0, err_msg=what)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.route(scores.cpu().numpy(), k_sel, 7 * case + 1, 0.3), err_msg=what)
    res = oracle.pasa_attention(to_f64(q), to_f64(k), to_f64(v), idx.cpu().numpy(), c["block"], group=c["group"], scale=scale,
                                return_all=True)
    assert_close(to_f64(out), res["o"], what=what)
    np.testing.assert_allclose(lse.cpu().numpy(), res["lse"], atol=2e-2, err_msg=what)
    assert_close(to_f64(dense), oracle.dense_attention(to_f64(q), to_f64(k), to_f64(v), scale=scale), what="dense, " + what)


@pytest.mark.parametrize("n,heads,d,block,group,batch", [
    (100, 1, 128, 64, 32, 1), (1023, 3, 64, 64, 32, 1), (4140, 4, 128, 64, 64, 1), (4097, 9, 64, 128, 16, 2), (3000, 2, 128, 64, 0, 1),
    (2113, 1, 128, 64, 1000, 2), (40960, 4, 128, 64, 32, 1), (40961, 4, 128, 64, 32, 1), (130, 511, 128, 64, 32, 1), (130, 256, 128, 64, 32, 2)])
def test_forward_leaves_what_its_stages_leave(P, n, heads, d, block, group, batch):
    """Statistics and scoring share launches in a whole forward up to 20 Mi elements (40,960 and 40,961 tokens are the line) and below 512 units of the
    statistics (511 and 512 heads): the same bits as the stages one by one, for both origins of the block-mean keys, with and without a second launch over the units of a group, heads dealt by XCD or not"""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn((batch, heads, n, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    shape = P.Shape.of(q, block=block, group=group)
    k_sel = P.topk_count(P.num_blocks(shape), 0.2)
    buffers = {}
    out, idx = P.forward(q, k, v, 0.2, 11, 0.125, block=block, group=group, buffers=buffers)
    scores = P.block_score(q, k, shape)
    want_idx, want_mask = P.route(scores, k_sel, 11, 0.125)
    assert torch.equal(buffers["scores"], scores) and torch.equal(idx, want_idx) and torch.equal(buffers["mask"], want_mask)
    assert torch.equal(out, P.sparse_attn_fwd(q, k, v, shape, want_idx, want_mask))
    single, lse = P.forward_single_call(q, k, v, shape, 0.2, 11, 0.125, want_lse=True)
    ws = P.kv_stats(k, v, shape)
    want_idx, want_mask = P.route(P.block_score(q, k, shape, stats_ws=ws if group else None), k_sel, 11, 0.125)
    want, want_lse = P.sparse_attn_fwd(q, k, v, shape, want_idx, want_mask, ws=ws, want_lse=True, prepared=True)
    assert torch.equal(single, want) and torch.equal(lse, want_lse)
