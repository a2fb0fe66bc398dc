"""The one-chunk-per-workgroup scoring kernels and the finishing launch at the edges of their variants, against the
oracle (needs an MI355X)."""
import pytest
import torch

import oracle
from parity_util import RTOL, check_index_row, check_scores, split_packed

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F32, BF16 = torch.float32, torch.bfloat16

# (dtype, n, Hq, Hkv, d, L, W, pool, pool_mode, budget): head sizes with half and missing pieces, one row tile and
# several of them side by side (few chunks), chunk ends, prefixes and kept rows around the most that are finished in
# one launch, pooling wider than it does, all and no keys ranked
CASES = [
    (F32, 1, 8, 1, 64, 1536, 16, 7, "max", 1536), (F32, 1, 8, 1, 64, 1537, 16, 7, "avg", 200), (F32, 2, 4, 4, 8, 257, 3, 5, "max", 64),
    (F32, 1, 6, 2, 200, 511, 9, 9, "avg", 77), (F32, 1, 2, 1, 256, 300, 40, 11, "max", 100), (F32, 1, 8, 8, 128, 8449, 4, 7, "max", 128),
    (BF16, 1, 8, 1, 64, 700, 32, 7, "max", 32), (BF16, 1, 16, 2, 72, 1025, 16, 3, "max", 65), (BF16, 2, 8, 2, 96, 640, 24, 9, "max", 64),
    (BF16, 1, 8, 2, 256, 769, 20, 7, "avg", 300), (BF16, 1, 8, 8, 128, 4096, 8, 7, "max", 128), (BF16, 1, 28, 4, 128, 1000, 32, 13, "max", 70),
    (BF16, 1, 2, 1, 128, 16384 + 8, 8, 7, "max", 300), (BF16, 1, 2, 1, 128, 16385 + 8, 8, 7, "max", 300), (BF16, 1, 4, 1, 24, 9000, 70, 1, "max", 128),
    (BF16, 1, 2, 1, 128, 8192 + 8, 8, 7, "max", 128), (BF16, 1, 2, 1, 128, 8192 + 8, 8, 5, "avg", 129), (BF16, 1, 2, 1, 128, 8193 + 8, 8, 7, "max", 128),
    (BF16, 1, 2, 1, 128, 8189 + 8, 8, 9, "avg", 128), (BF16, 1, 2, 1, 128, 8190 + 8, 8, 7, "max", 128), (F32, 2, 2, 1, 128, 2048 + 8, 8, 7, "max", 67),
    (BF16, 1, 2, 1, 128, 4096 + 8, 8, 7, "max", 384), (BF16, 1, 2, 1, 128, 4096 + 8, 8, 5, "avg", 385), (BF16, 1, 2, 1, 128, 4094 + 8, 8, 7, "max", 384),
    # many score rows around 128 and 256 chunks
    (BF16, 1, 64, 8, 64, 4096, 32, 7, "max", 200), (BF16, 1, 64, 8, 64, 4100, 32, 7, "max", 200),
    (BF16, 1, 64, 8, 64, 8192, 20, 5, "avg", 96), (BF16, 1, 64, 8, 64, 8193, 20, 7, "max", 96),
    # around four row tiles, the most that the kernels of larger calls stage together, and 64 chunks
    (BF16, 1, 32, 8, 128, 4097, 32, 7, "max", 100), (BF16, 1, 32, 8, 128, 8193, 32, 7, "max", 100), (BF16, 1, 32, 8, 128, 4200, 24, 7, "avg", 100),
    (BF16, 1, 64, 8, 128, 4097, 36, 7, "max", 100), (BF16, 1, 64, 8, 128, 4097, 40, 7, "max", 100),
    (BF16, 1, 32, 8, 64, 2048, 32, 7, "max", 100), (BF16, 1, 32, 8, 64, 2049, 32, 7, "avg", 100), (BF16, 1, 32, 8, 64, 8200, 24, 7, "max", 100),
    # the last call of these kernels and the first of those that walk a segment: one row tile, 32 chunks a head and 512 in all; heads of
    # more than 128 elements, two row tiles and 512 chunks, three and 64; fp32 and 128 chunks
    (BF16, 1, 32, 8, 128, 8192, 8, 7, "max", 100), (BF16, 1, 32, 8, 128, 8193, 8, 7, "max", 100), (BF16, 8, 8, 8, 64, 2048, 8, 7, "max", 100),
    (BF16, 9, 8, 8, 64, 2048, 8, 7, "avg", 100), (BF16, 8, 8, 8, 136, 2048, 33, 7, "max", 100), (BF16, 8, 8, 8, 136, 2049, 33, 7, "max", 100),
    (BF16, 1, 8, 8, 256, 2048, 70, 7, "max", 100), (BF16, 1, 8, 8, 256, 2049, 70, 7, "max", 100), (F32, 1, 8, 8, 128, 4096, 4, 7, "max", 100),
    (F32, 1, 8, 8, 128, 4097, 4, 7, "max", 100),
    # long heads, so few that a workgroup per chunk is one round of them; more than eight row tiles of 256 elements
    (F32, 1, 1, 1, 128, 49152, 4, 7, "max", 100), (F32, 1, 1, 1, 128, 49153, 4, 7, "avg", 100), (F32, 1, 1, 1, 128, 65536, 4, 7, "max", 100),
    (F32, 1, 1, 1, 128, 65537, 4, 7, "max", 100), (BF16, 1, 1, 1, 256, 131072, 65, 7, "max", 100), (BF16, 1, 1, 1, 256, 131073, 65, 7, "max", 100),
    (BF16, 1, 8, 8, 256, 2049, 256, 7, "max", 260), (BF16, 1, 8, 8, 256, 2049, 257, 7, "max", 260), (BF16, 9, 24, 8, 256, 127, 87, 7, "max", 120),
]


@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,L,W,pool,mode,budget", CASES)
def test_small_and_fp32_evictions(dtype, n, Hq, Hkv, d, L, W, pool, mode, budget):
    import paper_2505_20334_amd as laq
    print("case:", dtype, n, Hq, Hkv, d, L, W, pool, mode, budget, flush=True)
    g = torch.Generator().manual_seed(L + d)
    q = (1.5 * torch.randn(n, Hq, W, d, generator=g)).to(dtype)
    k, v = (torch.randn(n, Hkv, L, d, generator=g).to(dtype) for _ in range(2))
    b = [budget - 3 * i for i in range(n)]
    # one window of mixed positions (long ones travel in the workspace) and the trailing one
    for pos, keep in ((None, None), ([(37 * w) % L if w % 3 else L + w for w in range(W)], min(5, budget))):
        scores, idx, ko, vo = laq.laq_evict(q.to(DEV), k.to(DEV), v.to(DEV), b, pool, q_pos=pos, keep=keep, pool_mode=mode)
        torch.cuda.synchronize()
        parts, kp, vp = (split_packed(x.cpu(), b, Hkv, L) for x in (idx, ko, vo))
        for i in range(n):
            pooled, _, _, _ = oracle.evict(q[i], k[i], v[i], b[i], pool, q_pos=pos, keep=keep, pool_mode=mode)
            check_scores(scores[i].cpu(), pooled, dtype, "scores")
            kept = W if keep is None else keep
            want = oracle.select(scores[i].cpu(), kept, b[i])
            assert torch.equal(parts[i], want)
            for h in range(Hkv):
                check_index_row(parts[i][h].numpy(), pooled[h].float().numpy(), kept, b[i], RTOL[dtype], "list")
            assert torch.equal(kp[i], oracle.compact(k[i], want)) and torch.equal(vp[i], oracle.compact(v[i], want))


# a workgroup per head; the finishing launch; pooling in the selecting launch, and the gather in one of its own
@pytest.mark.parametrize("budget,choose", [(64, "auto"), (64, "two-pass"), (200, "two-pass")])
@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("pool", [1, 5, 7, 9])
def test_a_nan_shows_in_the_scores_of_one_launch_as_in_those_of_several(pool, mode, budget, choose):
    """A key of NaNs makes the scores of its head NaN; whatever launch pools them, it does as laq_score."""
    import paper_2505_20334_amd as laq
    g = torch.Generator().manual_seed(pool)
    q, k, v = (torch.randn(1, h, r, 64, generator=g).to(DEV) for h, r in ((4, 8), (2, 601), (2, 601)))
    k[0, 1, 77] = float("nan")
    scores = laq.laq_evict(q, k, v, [budget], pool, pool_mode=mode, choose=choose)[0]
    want = laq.laq_score(q, k, pool, pool_mode=mode, choose=choose)
    torch.cuda.synchronize()
    half = pool // 2                        # (windows over either end of the prefix hold zeros, which a maximum takes over a NaN)
    assert torch.isnan(want[0, 1, half:601 - 8 - half]).all() and not torch.isnan(want[0, 0]).any()
    assert torch.equal(torch.isnan(scores), torch.isnan(want)) and torch.equal(scores[0, 0], want[0, 0])


# (dtype, n, Hq, Hkv, d, W, choose), 480 to 700 keys; score rows that do not fill a tile of 32, and that do.  The first five take a
# workgroup per head or (fp32, d = 128 beyond 512 keys) per chunk, the next four one per chunk, and the others the kernels that walk
# a segment: d = 64 and 128 on request, the others with more than 128 chunks (fp32), 512 (d = 104 and 200) or two row
# tiles (d = 96); with 160 score rows, a second group of them
ROWS = [(F32, 1, 2, 2, 64, 8, "auto"), (F32, 1, 28, 4, 128, 4, "auto"), (BF16, 1, 8, 2, 96, 7, "auto"), (BF16, 1, 8, 2, 128, 2, "auto"), (F32, 1, 4, 1, 64, 8, "auto"),
        (F32, 1, 2, 2, 64, 8, "two-pass"), (F32, 1, 4, 1, 200, 20, "two-pass"), (BF16, 1, 8, 2, 96, 7, "two-pass"), (BF16, 1, 8, 2, 200, 5, "two-pass"),
        (BF16, 1, 8, 2, 64, 7, "two-pass"), (BF16, 2, 8, 2, 128, 40, "two-pass"), (BF16, 1, 8, 2, 96, 10, "two-pass"), (BF16, 86, 8, 2, 200, 25, "two-pass"),
        (F32, 33, 4, 2, 64, 8, "two-pass"), (F32, 86, 4, 2, 104, 5, "two-pass"), (F32, 33, 8, 2, 128, 40, "two-pass"), (F32, 33, 8, 2, 96, 10, "two-pass")]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,W,choose", ROWS)
def test_keys_behind_every_query_do_not_matter(dtype, n, Hq, Hkv, d, W, choose, bad):
    """Rows of a buffer that no query sees (not yet written, say) have the score 0, whatever they hold."""
    import paper_2505_20334_amd as laq
    L, seen = 700, 590
    g = torch.Generator().manual_seed(d)
    q, k = (torch.randn(n, h, r, d, generator=g).to(dtype) for h, r in ((Hq, W), (Hkv, L)))
    k[:, :, seen:] = 0.0
    pos = [seen - 1 - 3 * w for w in range(W)]
    pooled = [oracle.evict(q[i], k[i], k[i], 64, 1, q_pos=pos, keep=0)[0] for i in (0, n - 1)]
    k[:, :, seen:] = bad
    scores, idx, _, _ = laq.laq_evict(q.to(DEV), k.to(DEV), k.to(DEV), [64] * n, 1, q_pos=pos, keep=0, choose=choose)
    torch.cuda.synchronize()
    assert (scores[:, :, seen:] == 0).all() and int(idx.max()) < seen
    for i, want in zip((0, n - 1), pooled):
        check_scores(scores[i].cpu(), want, dtype, "scores")
        assert torch.equal(idx.cpu().reshape(n, Hkv, 64)[i], oracle.select(scores[i].cpu(), 0, 64))


@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,W,choose", ROWS)
def test_a_key_whose_logits_are_all_minus_infinity(dtype, n, Hq, Hkv, d, W, choose):
    import paper_2505_20334_amd as laq
    L = 600
    g = torch.Generator().manual_seed(d)
    q, k = (torch.randn(n, h, r, d, generator=g).to(dtype) for h, r in ((Hq, W), (Hkv, L)))
    q[..., 5] = -q[..., 5].abs() - 0.125
    pos = [L + w for w in range(W)]
    without = k.clone()
    k[:, :, 100, 5] = float("inf")
    without[:, :, 100, 5] = 1.0e4                          # a logit far enough below the others: probability 0 too
    scores = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=0, choose=choose)
    torch.cuda.synchronize()
    assert (scores[:, :, 100] == 0).all()
    for i in (0, n - 1):
        pooled, _, _, _ = oracle.evict(q[i], without[i], without[i], 64, 1, q_pos=pos, keep=0)
        check_scores(scores[i].cpu(), pooled, dtype, "scores")


# the first four: a workgroup per head, or (fp32, d > 64, few heads) per chunk; then, with Hq = n * 4, Hkv = n * 2 heads: per chunk, and the
# kernels that walk a segment, with one group of score rows and two
@pytest.mark.parametrize("dtype,d,W,n,choose", [
    (F32, 64, 5, 1, "auto"), (F32, 128, 20, 1, "auto"), (F32, 200, 16, 1, "auto"), (BF16, 96, 20, 1, "auto"), (F32, 64, 5, 1, "two-pass"), (BF16, 96, 7, 1, "two-pass"),
    (BF16, 64, 5, 1, "two-pass"), (BF16, 128, 20, 1, "two-pass"), (BF16, 128, 80, 1, "two-pass"), (BF16, 96, 20, 1, "two-pass"), (BF16, 200, 50, 130, "two-pass"),
    (F32, 64, 5, 33, "two-pass"), (F32, 104, 20, 33, "two-pass"), (F32, 128, 80, 33, "two-pass")])
def test_probabilities_below_the_smallest_normal_number_stay_apart(dtype, d, W, n, choose):
    """Logits 0, -1/4, -1/2, ... -119.75 (exact in either type): a list that ends among the denormal scores."""
    import paper_2505_20334_amd as laq
    Hq, Hkv, L, budget = 4, 2, 480, 400              # 2^-126 lies at key 349, 2^-149 at 413
    g = torch.Generator().manual_seed(d)
    rank = torch.randperm(L, generator=g)
    q, k = torch.zeros(n, Hq, W, d), torch.zeros(n, Hkv, L, d)
    q[..., :2] = 1.0
    k[..., 0], k[..., 1] = -8.0 * (rank // 32), -0.25 * (rank % 32)
    q, k = q.to(dtype), k.to(dtype)
    pos = [L + w for w in range(W)]
    scores, idx, _, _ = laq.laq_evict(q.to(DEV), k.to(DEV), None, [budget] * n, 1, scale=1.0, q_pos=pos, keep=0, choose=choose)
    torch.cuda.synchronize()
    assert torch.equal(idx.cpu().reshape(n * Hkv, budget), torch.nonzero(rank < budget).flatten().int().expand(n * Hkv, budget))
    want = oracle.raw_scores(q[0], k[0], 1.0, q_pos=pos)
    # an exponent of up to 173 is rounded twice (by half of 2^-16, and the factor log2 e by 2^-25 of it): relative error
    # ln 2 * (2^-17 + 173 * 2^-25) = 9e-6, and the instruction's own 1e-7; every term and sum to half of 2^-149
    rows = Hq // Hkv * W
    assert ((scores.cpu().double() - want).abs() <= 1.2e-5 * want + rows * 2.0 ** -149).all()


# (heads, KV rows kept in KiB, keys): with a workgroup for most compute units the finishing launch takes longer prefixes and more rows
MANY = [(128, 96, 8192), (128, 97, 8192), (159, 128, 8193), (160, 128, 16384), (160, 129, 16384), (160, 128, 16381), (160, 128, 16382), (256, 128, 9001)]


@pytest.mark.parametrize("mode", ["max", "avg"])
@pytest.mark.parametrize("heads,kib,keys", MANY)
def test_one_launch_for_many_heads_gives_the_bits_of_several(heads, kib, keys, mode):
    import paper_2505_20334_amd as laq
    print("case:", heads, kib, keys, mode, flush=True)
    d, W = 32, 2
    n, Hkv = (heads // 8, 8) if heads % 8 == 0 else (heads, 1)
    budgets = [kib * 1024 // (2 * d)] * n
    g = torch.Generator(device=DEV).manual_seed(heads + keys)
    q, k, v = (torch.randn(n, Hkv, r, d, generator=g, device=DEV).to(BF16) for r in (W, keys + W, keys + W))
    got = laq.laq_evict(q, k, v, budgets, 7, pool_mode=mode)
    scores = laq.laq_score(q, k, 7, pool_mode=mode)
    idx = laq.laq_select(scores, budgets, 1, W)
    rows = laq.laq_compact(k, v, idx, budgets, W)
    torch.cuda.synchronize()
    for x, y in zip(got, (scores, idx) + tuple(rows)):
        assert torch.equal(x, y)
    for i, h in ((0, 0), (n - 1, Hkv - 1)):
        assert torch.equal(split_packed(idx.cpu(), budgets, Hkv, keys + W)[i][h], oracle.select(scores[i, h:h + 1].cpu(), W, budgets[0])[0])
