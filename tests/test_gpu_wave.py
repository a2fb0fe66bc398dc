"""The scoring kernels that walk a segment of keys without a barrier, and the pooling in the selection kernel, at the
edges of their variants, against the oracle and the separate launches (needs an MI355X)."""
import pytest
import torch

import oracle
from parity_util import check_scores

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F32, BF16 = torch.float32, torch.bfloat16

# (dtype, n, Hq, Hkv, d, L, W): tiles of 32 keys and blocks of 128 with remainders, waves without a tile, segments of one and
# several blocks (their statistics folded by the second kernel, or by a launch in between: more than 32), row tiles up to
# the four that are staged together and beyond, head sizes with half and missing pieces.  fp32 and the head sizes other than 64
# and 128 take these kernels from 129 and 65 chunks of 256 keys on.
CASES = [
    (BF16, 1, 2, 1, 128, 31, 3), (BF16, 1, 2, 1, 128, 33, 16), (BF16, 2, 4, 2, 64, 127, 17), (BF16, 1, 8, 2, 128, 129, 32),
    (BF16, 1, 8, 1, 64, 1025, 33), (BF16, 1, 8, 1, 128, 8200, 16), (BF16, 1, 2, 1, 128, 20011, 8), (BF16, 130, 2, 1, 64, 160, 16),
    (BF16, 17, 12, 4, 96, 257, 33), (BF16, 17, 12, 4, 256, 300, 33), (BF16, 17, 8, 4, 40, 127, 50), (BF16, 65, 8, 4, 200, 511, 50),
    (F32, 65, 4, 2, 64, 65, 8), (F32, 33, 8, 4, 96, 130, 33), (F32, 33, 8, 4, 128, 97, 24), (F32, 43, 3, 3, 8, 100, 70),
    (F32, 33, 8, 4, 104, 129, 20), (F32, 1, 2, 1, 128, 33000, 20), (F32, 1, 3, 1, 128, 33100, 70),
    # several groups of row tiles: as many segments as the second kernel, which takes one group after the other, has use for
    (F32, 100, 4, 2, 64, 600, 65), (F32, 65, 4, 2, 128, 400, 100), (BF16, 200, 4, 2, 64, 400, 65),
    # head sizes without a variant of their own, either side of the lines up to which a workgroup takes a chunk instead: short heads of three row tiles;
    # fp32 from 33 elements and two row tiles on; one row tile and 64 elements, and bf16 of more than 128, from 513 chunks; five row tiles
    (BF16, 17, 4, 4, 72, 128, 65), (BF16, 17, 4, 4, 72, 129, 65), (BF16, 17, 4, 4, 200, 128, 65), (F32, 33, 4, 4, 16, 128, 65), (F32, 33, 4, 4, 16, 129, 65),
    (F32, 17, 8, 8, 32, 200, 65), (F32, 17, 8, 8, 40, 200, 65), (F32, 1, 7, 7, 72, 5000, 33), (F32, 1, 8, 8, 72, 4800, 33), (F32, 171, 1, 1, 72, 600, 5),
    (F32, 170, 1, 1, 72, 600, 5), (BF16, 171, 1, 1, 136, 600, 70), (BF16, 170, 1, 1, 136, 600, 70), (BF16, 513, 1, 1, 136, 250, 70), (BF16, 171, 1, 1, 136, 600, 140),
    (BF16, 80, 8, 2, 256, 1000, 40), (BF16, 81, 8, 2, 256, 1000, 40),
]


@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,L,W", CASES)
def test_scores_against_the_oracle(dtype, n, Hq, Hkv, d, L, W):
    import paper_2505_20334_amd as laq
    print("case:", dtype, n, Hq, Hkv, d, L, W, flush=True)
    g = torch.Generator().manual_seed(L + d)
    q = (1.5 * torch.randn(n, Hq, W, d, generator=g)).to(dtype)
    k = torch.randn(n, Hkv, L, d, generator=g).to(dtype)
    for pos, keep in ((None, None), ([(37 * w) % L if w % 3 else L + w for w in range(W)], 0)):
        if pos is None and W > L:
            continue
        got = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=keep, choose="two-pass").cpu()
        # rows of a wider cache: the same bits
        wide = torch.zeros(n, Hkv, L, d + 16, dtype=dtype, device=DEV)
        wide[..., :d] = k.to(DEV)
        again = laq.laq_score(q.to(DEV), wide[..., :d], 1, q_pos=pos, keep=keep, choose="two-pass").cpu()
        assert torch.equal(got, again)
        for i in sorted({0, n // 2, n - 1}):
            want, _, _, _ = oracle.evict(q[i], k[i], k[i], max(1, W if keep is None else keep), 1, q_pos=pos, keep=keep)
            check_scores(got[i], want, dtype, "instance %d" % i)


@pytest.mark.parametrize("shape", ["rising", "falling", "spike", "steps-of-the-headroom"])
@pytest.mark.parametrize("dtype,d", [(BF16, 64), (BF16, 128), (BF16, 256), (F32, 64), (F32, 128)])
def test_logits_that_outgrow_the_reference(dtype, d, shape):
    """The first pass keeps the reference of a wave's exponents until the sum of a tile reaches 128 of it.  Logits that rise over a
    segment by less than that a tile, by just about that, all at once, and not at all; exponents of 40 at most, rounded by 2^-19."""
    import paper_2505_20334_amd as laq
    n, L, W = 9, 4100, 5
    g = torch.Generator().manual_seed(d)
    t = torch.arange(L) / L
    ramp = {"rising": 24 * t, "falling": 24 - 24 * t, "spike": 20.0 * (torch.arange(L) % 1500 == 700),
            "steps-of-the-headroom": (torch.arange(L) // 128) * 7.0 * 0.6931 % 24}[shape]
    q = 0.3 * torch.randn(n, 2, W, d, generator=g)
    q[..., 0] = 8.0
    k = torch.randn(n, 1, L, d, generator=g)
    k[..., 0] = ramp * d ** 0.5 / 8.0
    q, k = q.to(dtype), k.to(dtype)
    got = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=[L + w for w in range(W)], keep=0, choose="two-pass").cpu()
    for i in (0, n - 1):
        want, _, _, _ = oracle.evict(q[i], k[i], k[i], 64, 1, q_pos=[L + w for w in range(W)], keep=0)
        check_scores(got[i], want, dtype, "instance %d" % i)


@pytest.mark.parametrize("rising", ["first half", "second half", "in turn"])
@pytest.mark.parametrize("dtype,d", [(BF16, 64), (BF16, 96), (BF16, 128), (BF16, 256), (BF16, 200), (F32, 64), (F32, 96), (F32, 128), (F32, 104)])
def test_each_row_of_a_tile_has_a_reference_of_its_own(dtype, d, rising):
    """A lane works on rows r and 16 + r of a tile and keeps the reference of one of them.  Rows whose logits outgrow it, several times over a
    wave's keys, next to rows whose logits never do: 16 score rows of one kind and 16, 32 of the other, or every second one; exponents of 40 at most."""
    import paper_2505_20334_amd as laq
    n, L, W = 80, 2100, 16
    print("case:", dtype, d, rising, flush=True)
    g = torch.Generator().manual_seed(d)
    q = 0.3 * torch.randn(n, 3, W, d, generator=g)
    q[..., 0] = 0.0
    q[..., 1] = 1.0
    rows = q.view(n, 3 * W, d)
    which = {"first half": slice(0, 16), "second half": slice(16, 32), "in turn": slice(1, None, 2)}[rising]
    rows[:, which, 0] = 8.0
    k = torch.randn(n, 1, L, d, generator=g)
    k[..., 0] = 24.0 * torch.arange(L) / L * d ** 0.5 / 8.0
    k[..., 1] = 0.0
    q, k = q.to(dtype), k.to(dtype)
    pos = [L + w for w in range(W)]
    got = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=0, choose="two-pass").cpu()
    for i in (0, n - 1):
        want, _, _, _ = oracle.evict(q[i], k[i], k[i], 64, 1, q_pos=pos, keep=0)
        check_scores(got[i], want, dtype, "instance %d" % i)


@pytest.mark.parametrize("d", [64, 104, 128])
def test_fp32_infinities_and_nans_are_those_of_whole_products(d):
    """A float is taken apart into three for the products; an infinity leaves NaNs, and the tile is scored from whole
    floats instead.  A key whose logits are all -inf gets the score 0 and leaves the others alone; one whose logits are +inf, or
    that holds a NaN, makes the scores of its head NaN, and only those."""
    import paper_2505_20334_amd as laq
    L, W = (262400 if d == 104 else 33200), 4      # 1025, 130 chunks
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(1, 2, W, d, generator=g).abs(), torch.randn(1, 1, L, d, generator=g)
    pos = [L + w for w in range(W)]
    k[0, 0, 777, 3] = -float("inf")
    got = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=0).cpu()
    k[0, 0, 777] = k[0, 0, 778]
    other = torch.cat([k[:, :, :777], k[:, :, 778:]], 2)
    want, _, _, _ = oracle.evict(q[0], other[0], other[0], 64, 1, q_pos=[p - 1 for p in pos], keep=0)
    assert got[0, 0, 777] == 0
    check_scores(torch.cat([got[0, :, :777], got[0, :, 778:]], 1), want, F32, "scores")
    for bad in (float("inf"), float("nan")):
        two = torch.cat([k, torch.randn(1, 1, L, d, generator=g)])
        two[0, 0, L - 1, 0] = bad
        got = laq.laq_score(torch.cat([q, q]).to(DEV), two.to(DEV), 1, q_pos=pos, keep=0).cpu()
        assert got[0].isnan().all() and not got[1].isnan().any()


@pytest.mark.parametrize("n,L,d", [(130, 250, 128), (65, 600, 128), (65, 1100, 64)])
def test_fp32_products_of_parts_are_no_further_from_64_bits(n, L, d):
    """Logits of a standard deviation of 4, 2-norm of the error of the scores, 64 score rows; a workgroup per head, and the kernels
    that walk a segment: an fp32 sum of 128 products q k rounded to 2^-24 of the running sum at every one is off by about 2^-24 * sqrt(128 / 3) of a
    logit's deviation, 1.6e-6 of an exponent, and the fp32 instruction measured 7 to 13e-7; the left-out products are 2^-24 of
    the whole ones.  A product of parts more left out (2^-16) would show as 6e-5."""
    import paper_2505_20334_amd as laq
    g = torch.Generator().manual_seed(5)
    W = 16
    q, k = 4.0 * torch.randn(n, 4, W, d, generator=g), torch.randn(n, 1, L, d, generator=g)
    got = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=[L + w for w in range(W)], keep=0).cpu().double()
    s = q.double().reshape(n, 4 * W, d) @ k[:, 0].double().transpose(1, 2) / d ** 0.5
    want = torch.softmax(s, -1).sum(1).unsqueeze(1)
    assert ((got - want).norm() / want.norm()).item() < 7e-7


# (heads, keys, d): fp32 calls that a workgroup per head takes, and calls of the kernels that walk a segment
F32_SHORT = [(24, 500, 64), (300, 300, 64), (80, 1000, 64), (80, 300, 128)]
F32_LONG = [(65, 1100, 64), (65, 600, 96), (172, 600, 104), (65, 600, 128)]


def _logit_errors(q, k):
    """One query row per head and logits near 1024: errors of the logits over 1024, from the scores.  A constant of the head is lost
    in the softmax: it is taken so that the median over the keys `k[:, 0, ::2]` is 0."""
    import paper_2505_20334_amd as laq
    got = laq.laq_score(q.to(DEV), k.to(DEV), 1, scale=1.0, q_pos=[k.shape[2]], keep=0).cpu().double()[:, 0]
    s = (q.double()[:, 0] @ k.double()[:, 0].transpose(1, 2))[:, 0]
    assert (s - 1024).abs().max() < 32         # (exponents of up to 92, rounded by 2^-18)
    e = torch.log(got) - torch.log_softmax(s, -1)
    return (e - e[:, ::2].median(-1, keepdim=True)[0]) / 1024


def _low_bits(x, bits):
    return ((x.view(torch.int32) & ~0xffff) | bits).view(torch.float32)


@pytest.mark.parametrize("n,L,d", F32_SHORT + F32_LONG)
def test_fp32_single_products(n, L, d):
    """Rows of one element that is not 0, so that a logit is one product.  Left out of it are the products of second and third
    parts: 2 * 2^-8 * 2^-17 = 2^-24 at most of a logit (below 1056).  The sum of the small products and the large one is rounded
    once, 2^-24 more; where a workgroup takes a head the matrix instruction adds them, which may cut off a whole unit, 2^-23.
    Every second key has 8 bits of mantissa, of which nothing is left out: their errors are the rounding alone, and their median
    is 0 but for the sampling (1.25 * 2^-24 / sqrt(3 * L / 2), four times that).  The exponents are rounded by 2^-18."""
    g = torch.Generator().manual_seed(d)
    for bits in (0xffff, 0x7fff, 0x8000, 0x8080, 0x7f7f, 0x0180, None):
        q, k = torch.zeros(n, 1, 1, d), torch.zeros(n, 1, L, d)
        a = 1 + 2.0 ** -7 * torch.randint(0, 128, (n,), generator=g)
        b = (1021 + 6 * torch.rand(n, L, generator=g)) / a[:, None]
        if bits is not None:
            a, b = _low_bits(a, bits), _low_bits(b, bits)
        else:
            a = a + 2.0 ** -7 * torch.rand(n, generator=g)
        b[:, ::2] = _low_bits(b[:, ::2].contiguous(), 0)
        q[:, 0, 0, d // 3], k[:, 0, :, d // 3] = a, b
        rounding = 2.0 ** (-23 if (n, L, d) in F32_SHORT else -24)
        bound = (2.0 ** -24 + rounding) * 1056 / 1024 + 4 * 1.25 * 2.0 ** -24 / (1.5 * L) ** 0.5 + 2.0 ** -28
        worst = _logit_errors(q, k).abs().max().item()
        assert worst <= bound, "low bits %s: %.3g of %.3g" % (bits if bits is None else hex(bits), worst, bound)


@pytest.mark.parametrize("n,L,d", F32_SHORT + F32_LONG)
def test_fp32_products_are_not_off_to_one_side(n, L, d):
    """Rows of positive elements whose mantissas end in ones, or in zeros (8 bits: nothing is left out): the roundings of the sums
    go to both sides in both, and on the average over all keys of all heads there is no difference: less than half a unit of
    a logit, 2^-24 (left-out parts that follow the sign of the product are 1 to 2.5e-7)."""
    g = torch.Generator().manual_seed(d)
    for signs in (False, True):
        q, k = 1 + torch.rand(n, 1, 1, d, generator=g), 1 + torch.rand(n, 1, L, d, generator=g)
        k = k * (1022 + 4 * torch.rand(n, 1, L, 1, generator=g)) / (q * k).sum(-1, keepdim=True)
        q, ones, zeros = _low_bits(q, 0xffff), _low_bits(k, 0xffff), _low_bits(k, 0)
        ones[:, :, ::2] = zeros[:, :, ::2]
        # (the shortened keys' logits are up to 2^-7 smaller: brought back by an element of a bf16 value)
        s = (q.double() * ones.double()).sum(-1, keepdim=True)
        fix = ((1024 - s) / q[..., :1].double()).float().bfloat16().float()
        ones[..., :1] = _low_bits((ones[..., :1] + fix).contiguous(), 0)
        if signs:
            sg = 1 - 2.0 * torch.randint(0, 2, (n, 1, 1, d), generator=g)
            q, ones = q * sg, ones * sg
        e = _logit_errors(q, ones)
        off = (e[:, 1::2].mean() - e[:, ::2].mean()).abs().item()
        assert off <= 2.0 ** -24, off


@pytest.mark.parametrize("n,L,d", F32_SHORT + F32_LONG)
def test_fp32_keys_and_queries_of_any_magnitude(n, L, d):
    """Queries times a power of two and keys divided by it, also by way of the scale: parts of small numbers that bf16 does not hold
    are not lost from the logits."""
    import paper_2505_20334_amd as laq
    g = torch.Generator().manual_seed(L)
    q, k = 1.5 * torch.randn(n, 2, 5, d, generator=g), torch.randn(n, 1, L, d, generator=g)
    q[:, 0, 0] = 0.0                          # (a row of zeros is one of ordinary numbers)
    pos = [L - 3 * w for w in range(5)]
    for eq, ek, es in ((110, -110, 0), (122, -122, 0), (-110, 110, 0), (-122, 122, 0), (60, -120, 60), (-120, 60, 60), (100, 20, -120)):
        scaled, kk, scale = q * 2.0 ** eq, k * 2.0 ** ek, d ** -0.5 * 2.0 ** es
        got = laq.laq_score(scaled.to(DEV), kk.to(DEV), 1, scale=scale, q_pos=pos, keep=0).cpu()
        for i in (0, n - 1):
            check_scores(got[i], oracle.raw_scores(scaled[i], kk[i], scale, q_pos=pos), F32, "2^%d 2^%d 2^%d" % (eq, ek, es))


# (n, Hkv, L, keep): prefixes around the sizes at which a variant of the selection kernel ends, rows of any alignment
@pytest.mark.parametrize("n,Hkv,L,keep", [(1, 3, 300, 5), (3, 3, 4093, 0), (2, 3, 8193, 3), (2, 3, 16385, 8), (1, 3, 32767, 2), (1, 2, 32768, 0),
                                          (1, 2, 32777, 1), (400, 2, 2046, 4), (400, 2, 2501, 9), (400, 2, 8199, 4)])
def test_pooling_and_selection_in_one_launch_are_those_of_two(n, Hkv, L, keep):
    """laq_evict pools raw scores where it selects; laq_score pools them in a launch of its own, laq_select takes those: the
    same bits, for every width and both kinds."""
    import paper_2505_20334_amd as laq
    g = torch.Generator(device=DEV).manual_seed(L)
    q = torch.randn(n, 2 * Hkv, 5, 64, generator=g, device=DEV).bfloat16()
    k, v = (torch.randn(n, Hkv, L, 64, generator=g, device=DEV).bfloat16() for _ in range(2))
    pos = [L + w for w in range(5)]
    budgets = [min(L, 40 + keep + 300 * (i % 3)) for i in range(n)]
    for pool, mode in ((3, "max"), (5, "avg"), (7, "max"), (9, "avg"), (11, "max"), (13, "avg"), (15, "max"), (17, "avg"), (17, "max"), (19, "max")):
        raw = laq.laq_score(q, k, 1, q_pos=pos, keep=keep)
        pooled = laq.laq_score(q, k, pool, q_pos=pos, keep=keep, pool_mode=mode)
        scores, idx, ko, vo = laq.laq_evict(q, k, v, budgets, pool, q_pos=pos, keep=keep, pool_mode=mode)
        assert torch.equal(scores, pooled)
        P, half = L - keep, pool // 2
        win = torch.nn.functional.pad(raw[..., :P].cpu(), (half, half)).unfold(-1, pool, 1)
        if mode == "max":
            want = win.amax(-1)
        else:
            want = torch.zeros_like(win[..., 0])
            for o in range(pool):
                want = want + win[..., o]
            want = want / torch.full((1,), float(pool))    # (a tensor: by a number torch may multiply with the reciprocal)
        assert torch.equal(pooled[..., :P].cpu(), want) and torch.equal(pooled[..., P:], raw[..., P:])
        assert torch.equal(idx, laq.laq_select(pooled, budgets, 1, keep))
        for a, b in zip((ko, vo), laq.laq_compact(k, v, idx, budgets, keep)):
            assert torch.equal(a, b)


# the last list that the finishing launch takes after the single-read kernel, and the first that it leaves: heads * 1280 bytes of
# K rows, from 128 heads on 160 KiB; one more layer, shorter heads, the two budgets in one call
@pytest.mark.parametrize("n,L,budgets", [(8, 8300, [320]), (8, 8300, [321]), (8, 8300, [17, 320]), (17, 3900, [640]), (17, 3900, [641])])
def test_gather_after_the_single_read_kernel_is_that_of_the_stages(n, L, budgets):
    import paper_2505_20334_amd as laq
    g = torch.Generator(device=DEV).manual_seed(L)
    q = torch.randn(n, 16, 8, 128, generator=g, device=DEV).bfloat16()
    k, v = (torch.randn(n, 8, L, 128, generator=g, device=DEV).bfloat16() for _ in range(2))
    assert laq.laq_score_kernel(n, 16, 8, 128, L, 8, BF16) == "single-read"
    b = [budgets[i % len(budgets)] for i in range(n)]
    scores, idx, ko, vo = laq.laq_evict(q, k, v, b, 7)
    assert torch.equal(scores, laq.laq_score(q, k, 7))
    assert torch.equal(idx, laq.laq_select(scores, b, 1, 8))
    for x, y in zip((ko, vo), laq.laq_compact(k, v, idx, b, 8)):
        assert torch.equal(x, y)


# (dtype, n, Hq, Hkv, d, L, W, rows of a block): either side of 256 MiB of keys, from which on the second kernel takes the heads in the other order: a last
# tile of score rows that is half empty, a paged cache, several groups of row tiles, a head size without a variant of its own
LARGE = [(F32, 137, 6, 2, 128, 1900, 16, 0), (F32, 150, 6, 2, 128, 1900, 16, 0), (F32, 90, 9, 3, 104, 2600, 16, 0), (BF16, 45, 28, 4, 128, 6300, 16, 256),
         (BF16, 41, 28, 4, 128, 6300, 16, 512), (BF16, 31, 40, 8, 64, 9200, 32, 0)]


@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,L,W,block", LARGE)
def test_heads_in_either_order(dtype, n, Hq, Hkv, d, L, W, block):
    import paper_2505_20334_amd as laq
    print("case:", dtype, n, Hq, Hkv, d, L, W, block, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    q = torch.randn(n, Hq, W, d, generator=g, device=DEV).to(dtype)
    table, kw = None, {}
    if block:
        per = -(-L // block)
        table = torch.randperm(n * per, generator=g, device=DEV).reshape(n, per).int()
        k = torch.randn(n * per, Hkv, block, d, generator=g, device=DEV).to(dtype)
        k[table[:, -1].long(), :, L - (per - 1) * block:] = float("nan")
        kw = dict(block_table=table, L=L)
    else:
        k = torch.randn(n, Hkv, L, d, generator=g, device=DEV).to(dtype)
    pos = [L + w for w in range(W)]
    assert laq.laq_score_kernel(n, Hq, Hkv, d, L, W, dtype, q_pos=pos, keep=0, whole_heads=True) != "single-read"
    got = laq.laq_score(q, k, 1, q_pos=pos, keep=0, **kw).cpu()
    for i in (0, 1, n // 2, n - 1):
        ki = k[i].cpu() if table is None else oracle.gather_paged(k[table[i].long()].cpu(), torch.arange(per)[None].int(), L)[0]
        want, _, _, _ = oracle.evict(q[i].cpu(), ki, ki, 64, 1, q_pos=pos, keep=0)
        check_scores(got[i], want, dtype, "instance %d" % i)


@pytest.mark.parametrize("n,d,L,W", [(449, 168, 128, 32), (450, 168, 128, 32), (449, 176, 100, 21), (450, 176, 100, 21), (450, 200, 60, 32), (450, 160, 97, 32)])
def test_short_heads_of_more_than_256_rows(n, d, L, W):
    """14 query heads each: groups of three row tiles where four leave room for two workgroups on a compute unit, and of four; head sizes next to these."""
    test_scores_against_the_oracle(BF16, n, 14, 1, d, L, W)
