"""The kernel that takes a whole short head in one workgroup, at the edges of its variants, against the oracle (needs an
MI355X)."""
import pytest
import torch

import oracle
from parity_util import RTOL, check_index_row, check_scores, split_packed

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F32, BF16 = torch.float32, torch.bfloat16

# (dtype, n, Hq, Hkv, d, L, W, pool, pool_mode, budgets): the longest head of each variant and one key more (which takes other kernels),
# heads shorter than a tile, one workgroup per head by the hundreds (two per compute unit), row tiles beyond the four that
# are staged together and the 256 rows it takes, head sizes with half and missing pieces, all, none and one key ranked, more instances than
# a launch's table holds
CASES = [
    (BF16, 2, 4, 2, 64, 512, 8, 7, "max", [100, 512]), (BF16, 2, 4, 2, 64, 513, 8, 7, "avg", [100, 9]), (BF16, 1, 8, 2, 128, 511, 32, 5, "max", [300]),
    (BF16, 9, 8, 8, 128, 1024, 5, 13, "max", [90 + 20 * i for i in range(9)]), (BF16, 9, 8, 8, 128, 1025, 5, 7, "max", [90] * 9), (BF16, 9, 16, 8, 64, 1023, 20, 9, "avg", [64] * 9),
    (BF16, 33, 16, 8, 96, 512, 7, 7, "max", [64 + i for i in range(33)]), (BF16, 33, 16, 8, 128, 500, 16, 3, "avg", [500] * 33), (BF16, 33, 8, 8, 64, 481, 3, 17, "max", [70] * 33),
    (BF16, 2, 3, 1, 256, 512, 12, 7, "max", [65, 64]), (BF16, 2, 3, 1, 200, 300, 50, 11, "max", [60, 51]), (BF16, 1, 2, 1, 40, 31, 4, 7, "max", [5]),
    (BF16, 1, 2, 1, 8, 1, 1, 1, "max", [1]), (BF16, 300, 2, 1, 64, 70, 4, 7, "max", [8 + i % 40 for i in range(300)]), (BF16, 270, 2, 1, 64, 33, 4, 5, "avg", [9] * 270),
    (BF16, 1, 8, 1, 128, 400, 32, 7, "max", [77]), (BF16, 1, 8, 1, 128, 400, 33, 7, "max", [77]), (BF16, 1, 6, 1, 128, 450, 25, 7, "max", [450]),
    (F32, 1, 4, 2, 64, 512, 8, 7, "max", [64]), (F32, 10, 8, 8, 64, 1000, 6, 7, "avg", [64, 1000] * 5), (F32, 35, 8, 8, 64, 512, 9, 5, "max", [64] * 35),
    # few heads of many rows: the gather is another launch's
    (BF16, 1, 8, 2, 128, 900, 8, 7, "max", [700]), (F32, 2, 4, 2, 64, 700, 8, 5, "avg", [690, 20]), (BF16, 2, 4, 4, 128, 1024, 6, 7, "max", [1024, 600]),
    (F32, 3, 14, 7, 128, 512, 20, 7, "max", [200, 21, 512]), (F32, 3, 7, 7, 104, 130, 9, 13, "max", [40] * 3), (F32, 3, 7, 7, 24, 97, 9, 1, "max", [40] * 3),
]


@pytest.mark.parametrize("dtype,n,Hq,Hkv,d,L,W,pool,mode,budgets", CASES)
def test_short_heads(dtype, n, Hq, Hkv, d, L, W, pool, mode, budgets):
    import paper_2505_20334_amd as laq
    print("case:", dtype, n, Hq, Hkv, d, L, W, pool, mode, flush=True)
    g = torch.Generator().manual_seed(L + d)
    q = (1.5 * torch.randn(n, Hq, W, d, generator=g)).to(dtype)
    k, v = (torch.randn(n, Hkv, L, d, generator=g).to(dtype) for _ in range(2))
    for pos, keep in ((None, None), ([(37 * w) % L if w % 3 else L + w for w in range(W)], min(5, min(budgets)))):
        kept = W if keep is None else keep
        b = [max(x, kept, 1) for x in budgets]
        scores, idx, ko, vo = laq.laq_evict(q.to(DEV), k.to(DEV), v.to(DEV), b, pool, q_pos=pos, keep=keep, pool_mode=mode)
        # scores alone, raw and pooled: the same bits; and from a strided cache
        alone = laq.laq_score(q.to(DEV), k.to(DEV), pool, q_pos=pos, keep=keep, pool_mode=mode)
        rows = torch.zeros(n, L, Hkv, d + 8 if dtype == BF16 else d + 4, dtype=dtype, device=DEV)[..., :d].permute(0, 2, 1, 3)
        rows.copy_(k)
        strided = laq.laq_evict(q.to(DEV), rows, None, b, pool, q_pos=pos, keep=keep, pool_mode=mode)
        raw = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=keep)
        torch.cuda.synchronize()
        assert torch.equal(scores, alone) and torch.equal(scores, strided[0]) and torch.equal(idx, strided[1]) and torch.equal(ko, strided[2])
        assert torch.equal(idx, laq.laq_select(raw, b, pool, kept, pool_mode=mode))
        parts, kp, vp = (split_packed(x.cpu(), b, Hkv, L) for x in (idx, ko, vo))
        for i in sorted({0, n // 2, n - 1}):
            pooled, _, _, _ = oracle.evict(q[i], k[i], v[i], b[i], pool, q_pos=pos, keep=keep, pool_mode=mode)
            check_scores(scores[i].cpu(), pooled, dtype, "scores")
            want = oracle.select(scores[i].cpu(), kept, b[i])
            assert torch.equal(parts[i], want)
            for h in range(Hkv):
                check_index_row(parts[i][h].numpy(), pooled[h].float().numpy(), kept, b[i], RTOL[dtype], "list")
            assert torch.equal(kp[i], oracle.compact(k[i], want)) and torch.equal(vp[i], oracle.compact(v[i], want))


# score rows either side of a half tile, a tile and what the registers keep, by variant: (dtype, d, heads, L)
VARIANTS = [(F32, 64, 3, 500), (F32, 64, 80, 600), (F32, 128, 20, 333), (F32, 72, 20, 129), (BF16, 64, 3, 500), (BF16, 64, 80, 600), (BF16, 128, 3, 500),
            (BF16, 128, 80, 600), (BF16, 128, 300, 70), (BF16, 96, 3, 97), (BF16, 256, 3, 300), (BF16, 200, 3, 65)]


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("dtype,d,heads,L", VARIANTS)
def test_rows_kept_and_made_again(dtype, d, heads, L, rows):
    """One query per window position and head: `rows` score rows.  Ordinary logits, scores below 2^-90 and an infinite key."""
    import paper_2505_20334_amd as laq
    print("case:", dtype, d, heads, L, rows, flush=True)
    if laq.laq_score_kernel(1, heads, heads, d, L, rows, dtype, q_pos=[L] * rows, keep=0, whole_heads=True) != "whole-head":
        pytest.skip("other kernels")
    g = torch.Generator().manual_seed(rows + L)
    q, k = torch.randn(1, heads, rows, d, generator=g), torch.randn(1, heads, L, d, generator=g)
    pos = [L if w % 2 else (7 * w) % L for w in range(rows)]
    for kind in ("ordinary", "small"):
        if kind == "small":
            q[..., 0] = 8.0 * d ** 0.5
            k[..., ::5, 0] = -12.0
        qq, kk = q.to(dtype), k.to(dtype)
        got = laq.laq_score(qq.to(DEV), kk.to(DEV), 1, q_pos=pos, keep=0).cpu()
        want, _, _, _ = oracle.evict(qq[0], kk[0], kk[0], 1, 1, q_pos=pos, keep=0)
        if kind == "ordinary" or dtype == BF16:
            check_scores(got[0], want, dtype, kind)
        else:
            # exponents up to 145 (log2 units), rounded at that size by each of the products that follow the large one (six a step of 32
            # elements), by the scaling and by the subtraction
            slack = 145 * (6 * -(-d // 32) + 2) * 2.0 ** -24 * 0.6931
            err = (got[0].double() - want.double()).abs()
            assert (err <= (RTOL[dtype] + slack) * want.double().abs() + 1e-30).all(), (err / want.double().abs()).max()
    q, k = torch.randn(1, heads, rows, d, generator=g), torch.randn(1, heads, L, d, generator=g)
    k[0, 0, 3] = float("inf")
    q[0, 0] = -q[0, 0].abs() - 0.5            # the infinite key's logits are -inf: its scores are zero
    got = laq.laq_score(q.to(dtype).to(DEV), k.to(dtype).to(DEV), 1, q_pos=[L] * rows, keep=0).cpu()
    assert got[0, 0, 3] == 0.0 and torch.isfinite(got[0]).all()
    # each row's probabilities: logits below 16, rounded by 2^-24 of that some twenty times
    assert abs(got[0, 0].double().sum() - rows) <= 16 * 20 * 2.0 ** -24 * rows


@pytest.mark.parametrize("L", [300, 512, 700])
@pytest.mark.parametrize("values", ["equal", "two", "steps", "wide", "crowd"])
def test_ranking_of_equal_and_crowded_scores(values, L):
    """Scores made to order: one query of one element per key value.  Ties go to the lower position; a bin of many keys is
    counted again."""
    import paper_2505_20334_amd as laq
    g = torch.Generator().manual_seed(L)
    n, d = 80, 64
    if values == "equal":
        x = torch.zeros(n, 1, L)
    elif values == "two":
        x = torch.randint(0, 2, (n, 1, L), generator=g).float()
    elif values == "steps":
        x = torch.randint(0, 9, (n, 1, L), generator=g).float() / 8
    elif values == "wide":
        x = 12 * torch.randn(n, 1, L, generator=g)
    else:                                    # all but a few within a thousandth, those far away
        x = 2.0 ** -10 * torch.rand(n, 1, L, generator=g)
        x[:, :, ::97] = -80.0
        x[:, :, 5] = 9.0
    q, k = torch.zeros(n, 1, 1, d), torch.zeros(n, 1, L, d)
    q[..., 0] = 1.0
    k[..., 0] = x
    for budget in (1, 2, 63, 64, 65, L // 2, L - 1):
        for pool in (1, 7):
            scores, idx, ko, _ = laq.laq_evict(q.to(DEV), k.to(DEV), None, [budget] * n, pool, scale=1.0, q_pos=[L], keep=0)
            got = idx.cpu().reshape(n, 1, budget)
            for i in (0, n // 2, n - 1):
                want = oracle.select(scores[i].cpu(), 0, budget)
                assert torch.equal(got[i], want)
            assert torch.equal(ko.cpu().reshape(n, budget, d)[..., 0], torch.gather(k[:, 0, :, 0], 1, got[:, 0].long()))


@pytest.mark.parametrize("dtype,d", [(BF16, 64), (BF16, 128), (BF16, 256), (F32, 64), (F32, 96)])
def test_values_that_are_not_finite_stay_in_their_head(dtype, d):
    import paper_2505_20334_amd as laq
    n, L, W = 24, 400, 4
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(n, 2, W, d, generator=g).abs().to(dtype), torch.randn(n, 1, L, d, generator=g).to(dtype)
    pos = [L + w for w in range(W)]
    clean = laq.laq_evict(q.to(DEV), k.to(DEV), None, [50] * n, 5, q_pos=pos, keep=0)
    bad = k.clone()
    bad[3, 0, 17, 2] = float("nan")
    bad[5, 0, 399, 0] = float("inf")
    bad[7, 0, 0, 1] = -float("inf")          # logits of -inf only: the score 0
    got = laq.laq_evict(q.to(DEV), bad.to(DEV), None, [50] * n, 1, q_pos=pos, keep=0)
    raw = laq.laq_score(q.to(DEV), k.to(DEV), 1, q_pos=pos, keep=0)
    assert got[0][3].isnan().all() and got[0][5].isnan().all() and got[0][7, 0, 0] == 0 and not got[0][7].isnan().any()
    keep = [i for i in range(n) if i not in (3, 5, 7)]
    assert torch.equal(got[0][keep], raw[keep]) and not clean[0].isnan().any()
    idx = got[1].cpu().reshape(n, 50)
    assert (idx.diff(dim=1) > 0).all() and int(idx.min()) >= 0 and int(idx.max()) < L


def test_paged_and_captured():
    """Blocks behind a shuffled table give the bits of the dense cache; a captured call replays with new inputs."""
    import paper_2505_20334_amd as laq
    n, H, L, d, br, W = 5, 4, 700, 128, 256, 16
    g = torch.Generator(device=DEV).manual_seed(3)
    q = torch.randn(n, 2 * H, W, d, generator=g, device=DEV).to(BF16)
    k, v = (torch.randn(n, H, L, d, generator=g, device=DEV).to(BF16) for _ in range(2))
    per = -(-L // br)
    table = torch.randperm(n * per, generator=g, device=DEV).reshape(n, per).int()
    kp, vp = (torch.full((n * per, H, br, d), float("nan"), device=DEV, dtype=BF16) for _ in range(2))
    for i in range(n):
        for b in range(per):
            m = min(br, L - b * br)
            kp[table[i, b], :, :m], vp[table[i, b], :, :m] = k[i, :, b * br:b * br + m], v[i, :, b * br:b * br + m]
    dense = laq.laq_evict(q, k, v, [64] * n, 7)
    paged = laq.laq_evict(q, kp, vp, [64] * n, 7, block_table=table, L=L)
    for a, b in zip(dense, paged):
        assert torch.equal(a, b)
    out = dict(scores=torch.empty_like(dense[0]), idx=torch.empty_like(dense[1]), k_out=torch.empty_like(dense[2]), v_out=torch.empty_like(dense[3]),
               ws=torch.empty(laq.laq_workspace_bytes(n, 2 * H, H, d, L, W, BF16), dtype=torch.uint8, device=DEV))
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        laq.laq_evict(q, k, v, [64] * n, 7, **out)
    for turn in range(3):
        k.copy_(torch.randn(n, H, L, d, generator=g, device=DEV))
        want = laq.laq_evict(q, k, v, [64] * n, 7)
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(want, (out["scores"], out["idx"], out["k_out"], out["v_out"])):
            assert torch.equal(a, b)
