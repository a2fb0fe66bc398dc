"""laq_select at the edges of its variants against the oracle's full sort (needs an MI355X)."""
import pytest
import torch

import oracle
from parity_util import split_packed

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (n, Hkv, L, W, budgets): prefixes around the sizes at which a variant ends (4096, 8192, 16384 and 32768 keys;
# with many heads 2048, 8192 and 32768), rows that start 0 .. 3 scores behind a 16-byte boundary, and numbers of
# wanted keys around those up to which a group of keys is a thread's, half or a quarter of it
CASES = [
    (1, 3, 4093 + 8, 8, [8 + 1, ]), (1, 3, 4096 + 8, 8, [8 + 1023]), (1, 3, 4097 + 8, 8, [8 + 1024]),
    (1, 3, 8189 + 5, 5, [5 + 2049]), (1, 3, 16381 + 3, 3, [3 + 4097]), (1, 3, 16382 + 3, 3, [3 + 2048]),
    (1, 3, 32765, 0, [1024]), (1, 3, 32766, 0, [1023]), (1, 3, 30011, 8, [1024]), (1, 2, 517, 16, [516]),
    (400, 2, 2045 + 4, 4, [4 + 255, 4 + 2044]), (400, 2, 2046 + 4, 4, [4 + 256, 4 + 513]),
    (400, 2, 8189 + 4, 4, [4 + 300, 4 + 4000]), (400, 2, 8190 + 4, 4, [4 + 512, 4 + 1100]),
    (384, 2, 32765, 0, [512, 1500]), (384, 2, 32766, 0, [700, 2100]),
    # aligned rows: these fill a variant's registers exactly
    (1, 3, 4096, 0, [1024]), (1, 3, 16384 + 4, 4, [4 + 1024]), (1, 3, 32768, 0, [1024]), (1, 3, 32772, 4, [4 + 2048]),
    (400, 2, 2048, 0, [256, 2040]), (400, 2, 8192, 0, [512, 1100]), (384, 2, 32768, 0, [700, 2100]),
]


@pytest.mark.parametrize("values", ["spread", "few", "equal", "plateaus", "masked"])
@pytest.mark.parametrize("n,Hkv,L,W,budgets", CASES)
def test_select_at_the_edges_of_its_variants(n, Hkv, L, W, budgets, values):
    import paper_2505_20334_amd as laq
    print("case:", n, Hkv, L, W, budgets, values, flush=True)
    g = torch.Generator(device=DEV).manual_seed(L)
    if values == "spread":                  # many orders of magnitude
        s = torch.exp(6 * torch.randn(n, Hkv, L, generator=g, device=DEV))
    elif values == "few":
        s = torch.randint(0, 9, (n, Hkv, L), generator=g, device=DEV).float() / 7
    elif values == "equal":
        s = torch.full((n, Hkv, L), 0.25, device=DEV)
    elif values == "masked":                # fewer scores than wanted keys: the others tie at -inf
        s = torch.rand(n, Hkv, L, generator=g, device=DEV)
        s.masked_fill_(torch.rand(n, Hkv, L, generator=g, device=DEV) < 0.999, float("-inf"))
    else:                                   # what the pooling makes of scores
        s = torch.exp(torch.randn(n * Hkv, 1, L, generator=g, device=DEV))
        s = torch.nn.functional.max_pool1d(s, 7, 1, 3).reshape(n, Hkv, L)
    s = s.contiguous()
    b = [budgets[i % len(budgets)] for i in range(n)]
    idx = laq.laq_select(s, b, 1, W)
    torch.cuda.synchronize()
    parts = split_packed(idx.cpu(), b, Hkv, L)
    for i in sorted({0, 1, n // 2, n - 1} & set(range(n))):
        assert torch.equal(parts[i], oracle.select(s[i].cpu(), W, b[i])), i


# (n, P, waves): the variants with lists; a wave's list holds 204 quads of neighbouring keys
@pytest.mark.parametrize("n,P,waves", [(1, 32768, 16), (1, 16388, 16), (768, 8192, 4), (768, 32768, 8)])
@pytest.mark.parametrize("crowded", [64, 203, 204, 205, 512])
def test_select_where_one_waves_part_is_crowded(n, P, waves, crowded):
    """`crowded` quads of the first wave's part hold a high score, and one of every lane of the others."""
    import paper_2505_20334_amd as laq
    print("case:", n, P, waves, crowded, flush=True)
    part = 64 * 64 if waves == 8 else 64 * 32
    g = torch.Generator(device=DEV).manual_seed(crowded)
    s = torch.rand(n, 1, P, generator=g, device=DEV) * 1e-3
    for w in range(-(-P // part)):
        quads = torch.arange(crowded) if w == 0 else torch.arange(64) + 64 * (torch.arange(64) * 7 % (part // 256))
        pos = w * part + 4 * quads + quads % 4
        pos = pos[pos < P].to(DEV)
        s[:, 0, pos] = 1 + torch.randint(0, 50, (n, len(pos)), generator=g, device=DEV).float() / 64
    high = int((s[0, 0] >= 1).sum())
    budgets = [min(high - 5, P // 40), 37, high]
    b = [budgets[i % 3] for i in range(n)]
    parts = split_packed(laq.laq_select(s, b, 1, 0).cpu(), b, 1, P)
    for i in sorted({0, 1 % n, 2 % n, n - 1}):
        assert torch.equal(parts[i], oracle.select(s[i].cpu(), 0, b[i])), i


def test_a_prefix_of_a_variants_size_takes_that_variant():
    """32768 aligned scores per head fit the registers; the kernel that re-reads longer prefixes takes three times as long."""
    import paper_2505_20334_amd as laq

    def fastest(L):
        s = torch.rand(32, 8, L, device=DEV)
        idx = laq.laq_select(s, [512] * 32, 1, 0)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                laq.laq_select(s, [512] * 32, 1, 0, idx=idx)
        best = float("inf")
        for _ in range(20):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        return best

    assert fastest(32768) < 2 * fastest(32764)
