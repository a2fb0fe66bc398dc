"""The single-read scoring kernel (a head's unnormalised probabilities stay in registers until the
softmax denominators are known) vs the CPU oracle (needs an MI355X).

laq_score takes that kernel for bf16 caches with d = 128 and at most 64 score rows per KV head
(R = G * W), by itself from some size of the call on and below that when the shape asks for it, as
the cases here do; a team of workgroups shares a head, 512 keys each with more than 32 score rows,
1024 otherwise.  The cases walk the team sizes (one workgroup, a ragged last workgroup, a key count
one past a boundary) for both, the row counts, heads fewer and more than the teams the device
holds, strided caches, explicit query positions, and check after every call that all the kernel's
waits completed (status of the workspace).
"""
import numpy as np
import pytest
import torch

import oracle
from parity_util import check_scores

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
D = 128


@pytest.fixture(scope="module")
def laq():
    import paper_2505_20334_amd as m
    m.load_library()
    assert torch.cuda.is_available()
    return m


def draw(n, Hkv, G, L, W, seed, sinks=True):
    g = torch.Generator().manual_seed(seed)
    q = torch.randn(n, Hkv * G, W, D, generator=g)
    k = torch.randn(n, Hkv, L, D, generator=g)
    if sinks:
        # a few keys that every query likes (attention sinks), and one query row with a large norm
        k[:, :, :2] += 0.6 * q.reshape(n, Hkv, G * W, D).mean(2, keepdim=True)
        q[:, 0, 0] *= 4.0
    return q.bfloat16(), k.bfloat16()


def score_and_check(laq, q, k, pool, what, heads, k_dev=None, **kw):
    n, Hq, W, _ = q.shape
    _, Hkv, L, _ = k.shape
    G = Hq // Hkv
    print("case:", what, "n=%d Hkv=%d G=%d L=%d W=%d pool=%d" % (n, Hkv, G, L, W, pool), flush=True)
    qd = q.to(DEV)
    kd = k.to(DEV) if k_dev is None else k_dev
    strides = (0, 0, 0) if kd.is_contiguous() else (kd.stride(0), kd.stride(1), kd.stride(2))
    assert laq.laq_score_kernel(n, Hq, Hkv, D, L, W, torch.bfloat16, kw.get("q_pos"), kw.get("keep"),
                                strides, choose="single-read") == "single-read", what
    kw = dict(kw, choose="single-read")
    nb = laq.laq_workspace_bytes(n, Hq, Hkv, D, L, W, torch.bfloat16)
    ws = torch.zeros(nb, dtype=torch.uint8, device=DEV)
    s = laq.laq_score(qd, kd, pool, ws=ws, **kw)
    again = laq.laq_score(qd, kd, pool, ws=ws, **kw)
    torch.cuda.synchronize()
    assert laq.laq_workspace_status(ws, n, Hq, Hkv, D, L, W, torch.bfloat16) == 0, what + ": a wait was given up"
    assert torch.equal(s, again), what + ": two runs differ"
    assert torch.isfinite(s).all()
    sc = s.cpu()
    okw = {key: kw[key] for key in ("scale", "q_pos") if key in kw}
    keep = kw.get("keep", W)
    for (i, h) in heads:
        raw = oracle.raw_scores(q[i, h * G:(h + 1) * G], k[i, h:h + 1], **okw)
        want = oracle.maxpool(raw, keep, pool)
        check_scores(sc[i, h], want[0], torch.bfloat16, "%s inst %d head %d" % (what, i, h))
    return s


SHAPES = [
    # name, n, Hkv, G, L, W, pool
    ("one-workgroup", 3, 2, 4, 300, 8, 7),
    ("exactly-one-workgroup-32-rows", 2, 2, 4, 1024, 8, 1),
    ("exactly-one-workgroup-64-rows", 2, 2, 4, 512, 16, 1),
    ("one-key-past-a-boundary-32-rows", 2, 2, 4, 1025, 8, 7),
    ("one-key-past-a-boundary-64-rows", 2, 2, 4, 513, 16, 7),
    ("window-straddles-a-boundary-32-rows", 2, 2, 4, 2054, 8, 7),
    ("window-straddles-a-boundary-64-rows", 2, 2, 4, 1030, 16, 7),
    ("pool-window-straddles-boundaries", 2, 2, 4, 1540, 12, 15),
    ("ragged-team-of-ten", 2, 3, 4, 4700, 16, 7),
    ("rows-not-a-multiple-of-32", 2, 2, 4, 2100, 5, 5),
    ("48-rows", 2, 2, 4, 3000, 12, 3),
    ("64-rows-no-group", 2, 4, 1, 2500, 64, 7),
    ("group-of-eight", 2, 2, 8, 2049, 8, 7),
    ("one-query", 2, 2, 4, 1500, 1, 1),
    ("wide-pool", 2, 2, 4, 2600, 8, 31),
    # 65 ... 128 score rows: 256 keys per workgroup
    ("exactly-one-workgroup-128-rows", 2, 2, 4, 256, 32, 1),
    ("one-key-past-a-boundary-128-rows", 2, 2, 4, 257, 32, 7),
    ("window-straddles-a-boundary-128-rows", 2, 2, 4, 530, 32, 7),
    ("128-rows-team-of-eleven", 2, 3, 4, 2700, 32, 7),
    ("96-rows", 2, 2, 4, 1900, 24, 5),
    ("68-rows", 2, 2, 4, 1300, 17, 7),
    ("128-rows-group-of-eight", 2, 2, 8, 1111, 16, 3),
    ("128-rows-one-head-per-query", 1, 2, 1, 900, 128, 7),
]


@pytest.mark.parametrize("name,n,Hkv,G,L,W,pool", SHAPES, ids=[c[0] for c in SHAPES])
def test_shapes(laq, name, n, Hkv, G, L, W, pool):
    q, k = draw(n, Hkv, G, L, W, seed=L + W)
    score_and_check(laq, q, k, pool, name, [(0, 0), (n - 1, Hkv - 1)])


def test_more_heads_than_teams_and_fewer(laq):
    # L = 16384, 64 score rows: 32 workgroups per team, the device holds 16 teams; 40 heads take three
    # rounds with an unequal share, 3 heads leave most of the device idle
    for (n, Hkv) in ((5, 8), (1, 3)):
        q, k = draw(n, Hkv, 4, 16384, 16, seed=n * 100 + Hkv, sinks=False)
        score_and_check(laq, q, k, 7, "heads-%d" % (n * Hkv), [(0, 0), (n - 1, Hkv - 1), (n // 2, 1)])


def test_long_head_small_team_count(laq):
    # L = 70000: 137 workgroups per team with 64 score rows (3 teams on the device), 69 with 32 (7 teams)
    q, k = draw(1, 5, 4, 70000, 16, seed=7, sinks=False)
    score_and_check(laq, q, k, 7, "long-head-64-rows", [(0, 0), (0, 4)])
    q, k = draw(1, 9, 4, 70000, 8, seed=8, sinks=False)
    score_and_check(laq, q, k, 7, "long-head-32-rows", [(0, 0), (0, 8)])


def test_strided_and_token_major_caches(laq):
    n, Hkv, G, L, W = 2, 3, 4, 2300, 16
    q, k = draw(n, Hkv, G, L, W, seed=11)
    dense = score_and_check(laq, q, k, 7, "dense", [(0, 0), (1, 2)])
    # head-padded cache: every head is followed by 40 unused rows
    padded = torch.zeros(n, Hkv, L + 40, D, dtype=torch.bfloat16, device=DEV)
    padded[:, :, :L] = k.to(DEV)
    s_pad = score_and_check(laq, q, k, 7, "head-padded", [(1, 1)], k_dev=padded[:, :, :L])
    # token-major cache [n, L, Hkv, d] viewed as [n, Hkv, L, d]
    tm = k.to(DEV).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert not tm.is_contiguous()
    s_tm = score_and_check(laq, q, k, 7, "token-major", [(0, 2)], k_dev=tm)
    assert torch.equal(dense, s_pad) and torch.equal(dense, s_tm)


def test_explicit_query_positions_and_scale(laq):
    n, Hkv, G, L, W = 2, 2, 4, 1800, 8
    q, k = draw(n, Hkv, G, L, W, seed=5)
    # queries in the middle of the sequence: keys behind a query's position are invisible to it
    q_pos = [700, 701, 900, 1100, 1101, 1102, 1500, 1799]
    score_and_check(laq, q, k, 1, "positions", [(0, 0), (1, 1)], q_pos=q_pos, keep=0)
    score_and_check(laq, q, k, 7, "positions-pooled", [(0, 1)], q_pos=q_pos, keep=0)
    # a sharper softmax (large logits): the probabilities span hundreds of binary orders of magnitude
    score_and_check(laq, q, k, 1, "scale-1.5", [(0, 0), (1, 1)], scale=1.5)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("order", ["spread", "falling"])
@pytest.mark.parametrize("W", [8, 16])
def test_denormal_scores(laq, W, order, paged):
    """Logits 0, -1/4, -1/2, ...: lists that end among scores below 2^-126, in workgroups with large ones and (falling, 64 rows) in one without."""
    n, Hq, Hkv, L = 2, 8, 2, 1800
    rank = torch.arange(L) * 11 // 16 if order == "falling" else torch.randperm(L, generator=torch.Generator().manual_seed(W))
    q, k = torch.zeros(n, Hq, W, D), torch.zeros(n, Hkv, L, D)
    q[..., :2] = 1.0
    k[..., 0], k[..., 1] = -8.0 * (rank // 32).clamp(max=64), -0.25 * (rank % 32)
    pos = [L + w for w in range(W)]
    kd, kw = k.bfloat16().to(DEV), {}
    if paged:
        table = torch.randperm(n * 8, generator=torch.Generator().manual_seed(3)).reshape(n, 8).int().to(DEV)
        pool = torch.zeros(n * 8, Hkv, 256, D, dtype=torch.bfloat16, device=DEV)
        pool[table.long()] = torch.nn.functional.pad(kd, (0, 0, 0, 8 * 256 - L)).reshape(n, Hkv, 8, 256, D).transpose(1, 2)
        kd, kw = pool, dict(block_table=table, L=L)
    below = int((rank < 400).sum())                  # (2^-126 lies at rank 349, 2^-149 at 413; equal ranks: the lower positions)
    scores, idx, _, _ = laq.laq_evict(q.bfloat16().to(DEV), kd, None, [below] * n, 1, scale=1.0, q_pos=pos, keep=0, choose="single-read", **kw)
    torch.cuda.synchronize()
    assert torch.equal(idx.cpu().reshape(n * Hkv, below), torch.nonzero(rank < 400).flatten().int().expand(n * Hkv, below))
    want = oracle.raw_scores(q[0].bfloat16(), k[0].bfloat16(), 1.0, q_pos=pos)
    rows = Hq // Hkv * W                             # (the bound of the other kernels' test of such scores)
    assert ((scores.cpu().double() - want).abs() <= 1.2e-5 * want + rows * 2.0 ** -149).all()


def test_which_kernel(laq):
    bf, f32 = torch.bfloat16, torch.float32
    want = "single-read"
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 8, bf) == "two-pass"            # 16 MiB of keys: not worth it
    assert laq.laq_score_kernel(64, 32, 8, 128, 4096, 8, bf) == "single-read"        # 512 MiB
    assert laq.laq_score_kernel(16, 32, 8, 128, 4096, 16, bf) == "single-read"       # 128 MiB, 64 rows
    assert laq.laq_score_kernel(64, 32, 8, 128, 4096, 8, bf, choose="two-pass") == "two-pass"
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 8, bf, choose=want) == "single-read"     # 32 rows
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 16, bf, choose=want) == "single-read"    # 64 rows
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 17, bf, choose=want) == "single-read"    # 68 rows
    assert laq.laq_score_kernel(64, 32, 8, 128, 32768, 32, bf, choose=want) == "single-read"  # 128 rows
    assert laq.laq_score_kernel(64, 32, 8, 128, 32768, 32, bf) == "two-pass"                  # ... but not by itself
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 33, bf, choose=want) == "two-pass"       # 132 rows
    assert laq.laq_score_kernel(2, 32, 8, 64, 4096, 8, bf, choose=want) == "two-pass"         # d = 64
    assert laq.laq_score_kernel(2, 32, 8, 128, 4096, 8, f32, choose=want) == "vector"
    assert laq.laq_score_kernel(1, 4, 1, 128, 600000, 8, bf, choose=want) == "two-pass"       # a team longer than the device holds
    with pytest.raises(laq.LaqError):
        laq.laq_score_kernel(2, 32, 8, 128, 4096, 0, bf)


@pytest.mark.parametrize("n,L,W,light", [(3, 6827, 16, True), (3, 6750, 16, False), (5, 4916, 8, True), (5, 4900, 8, False), (24, 1281, 8, True),
                                          (26, 1280, 8, False), (1, 32768, 16, True), (1, 32769, 16, False)])
def test_which_kernel_by_the_size_of_the_call(laq, n, L, W, light):
    # either side of the lines (40 MiB of keys with 64 score rows, 48 with 32, there beyond 1280 keys a head; 64 workgroups per team below
    # 128 MiB); a captured call takes the same kernels: every replay gives the eager bits
    bf = torch.bfloat16
    kind = laq.laq_score_kernel(n, 32, 8, D, L, W, bf)
    assert kind == ("single-read" if light else "two-pass")
    q, k = draw(n, 8, 4, L, W, seed=L, sinks=False)
    q, k = q.to(DEV), k.to(DEV)
    ws = torch.full((laq.laq_workspace_bytes(n, 32, 8, D, L, W, bf),), 0xFF, dtype=torch.uint8, device=DEV)
    out, pooled = torch.empty(n, 8, L, device=DEV), torch.empty(n, 8, L, device=DEV)
    laq.laq_score(q, k, 7, scores=out, ws=ws)
    assert torch.equal(out, laq.laq_score(q, k, 7, choose=kind))
    assert laq.laq_workspace_status(ws, n, 32, 8, D, L, W, bf) == 0
    got = laq.laq_evict(q, k, k, [200] * n, 7, ws=ws)             # (pooled in another kernel, from the same raw scores)
    assert torch.equal(got[0], out) and torch.equal(got[1], laq.laq_select(out, [200] * n, 1, W))
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        laq.laq_score(q, k, 7, scores=pooled, ws=ws)
    two = laq.laq_score(q, k, 7, choose="two-pass")
    for _ in range(3):
        pooled.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(pooled, out)
    assert laq.laq_workspace_status(ws, n, 32, 8, D, L, W, bf) == 0
    np.testing.assert_allclose(out.cpu().numpy(), two.cpu().numpy(), rtol=2e-5, atol=1e-30)


def test_status_is_defined_after_every_kind_of_call(laq):
    # a workspace full of ones: whichever kernels score, the call leaves "all waits completed" behind
    for (W, d, dt, kind) in ((8, 128, torch.bfloat16, "single-read"), (32, 128, torch.bfloat16, "two-pass"),
                             (8, 128, torch.bfloat16, "two-pass"), (8, 64, torch.float32, "vector")):
        n, Hq, Hkv, L = 1, 8, 2, 1200
        assert laq.laq_score_kernel(n, Hq, Hkv, d, L, W, dt, choose=kind if kind != "vector" else "auto") == kind
        g = torch.Generator().manual_seed(W)
        q = torch.randn(n, Hq, W, d, generator=g).to(dt).to(DEV)
        k = torch.randn(n, Hkv, L, d, generator=g).to(dt).to(DEV)
        ws = torch.full((laq.laq_workspace_bytes(n, Hq, Hkv, d, L, W, dt),), 0xFF, dtype=torch.uint8, device=DEV)
        laq.laq_score(q, k, 7, ws=ws, choose=kind if kind != "vector" else "auto")
        assert laq.laq_workspace_status(ws, n, Hq, Hkv, d, L, W, dt) == 0, kind


def test_both_kernels_on_the_same_call(laq):
    # the two designs sum in different orders: equal to within fp32 rounding, not bit for bit
    n, Hkv, G, L, W = 3, 4, 4, 6000, 16
    q, k = draw(n, Hkv, G, L, W, seed=21)
    a = laq.laq_score(q.to(DEV), k.to(DEV), 7, choose="single-read")
    b = laq.laq_score(q.to(DEV), k.to(DEV), 7, choose="two-pass")
    torch.cuda.synchronize()
    np.testing.assert_allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=2e-5, atol=1e-30)
    # and the whole path agrees wherever the ranking is not decided inside that rounding
    budgets = [300, 301, 302]
    ia = laq.laq_evict(q.to(DEV), k.to(DEV), None, budgets, 7, choose="single-read")[1]
    ib = laq.laq_evict(q.to(DEV), k.to(DEV), None, budgets, 7, choose="two-pass")[1]
    assert (ia != ib).float().mean().item() < 0.01


def test_constant_keys_give_uniform_probabilities(laq):
    # all keys equal: every visible key gets probability 1 / (number visible), whatever the team split
    n, Hkv, G, L, W = 1, 2, 4, 1300, 8
    g = torch.Generator().manual_seed(3)
    q = torch.randn(n, Hkv * G, W, D, generator=g).bfloat16()
    k = torch.randn(1, 1, 1, D, generator=g).expand(n, Hkv, L, D).contiguous().bfloat16()
    s = laq.laq_score(q.to(DEV), k.to(DEV), 1, choose="single-read").cpu().double()
    P = L - W
    want = torch.zeros(L, dtype=torch.float64)
    for w in range(W):
        want[: P + w + 1] += G / (P + w + 1)
    np.testing.assert_allclose(s[0, 0].numpy(), want.numpy(), rtol=2e-6)
    np.testing.assert_allclose(s[0, 1].numpy(), want.numpy(), rtol=2e-6)


@pytest.mark.parametrize("L,W,heads", [((1500,) * 3, 8, 40), ((8200,) * 3, 8, 24), ((16384,) * 3, 16, 9), ((16640,) * 3, 16, 40), ((32768,) * 3, 16, 10),
                                       ((33280,) * 3, 16, 10), ((32768, 300, 65000, 9000), 16, 5), ((2100, 32768, 257), 32, 6)])
def test_calls_side_by_side(laq, L, W, heads):
    # several launches on the device at once, each with teams of which some are there only in part: places are drawn in the order
    # of start, so every call completes, with the bits of a call that is alone; sizes: few and many workgroups per team (2, 9, 32, 33, and 64, the
    # longest that draw from two counters, 65 from one), more and fewer heads than teams, unlike launches (64, 1, 127 and 18 workgroups per
    # team; with 128 score rows 9, 128, the longest that are covered, and 2)
    calls = []
    for i, L in enumerate(L):
        q, k = draw(1, heads, 4, L, W, seed=L + i, sinks=False)
        q, k = q.to(DEV), k.to(DEV)
        ws = torch.full((laq.laq_workspace_bytes(1, heads * 4, heads, D, L, W, torch.bfloat16),), 0xFF, dtype=torch.uint8, device=DEV)
        assert laq.laq_score_kernel(1, heads * 4, heads, D, L, W, torch.bfloat16, choose="single-read") == "single-read"
        calls.append((q, k, ws, torch.cuda.Stream(), laq.laq_score(q, k, 7, ws=ws, choose="single-read"), torch.empty(1, heads, L, device=DEV)))
    torch.cuda.synchronize()
    for _ in range(4):
        for q, k, ws, stream, alone, out in calls:
            with torch.cuda.stream(stream):
                laq.laq_score(q, k, 7, scores=out, ws=ws, choose="single-read")
    torch.cuda.synchronize()
    for q, k, ws, stream, alone, out in calls:
        assert laq.laq_workspace_status(ws, 1, heads * 4, heads, D, k.shape[2], W, torch.bfloat16) == 0
        assert torch.equal(out, alone)


@pytest.mark.parametrize("L,W,kind", [(65536, 16, "single-read"), (65537, 16, "two-pass"), (131072, 8, "single-read"), (131073, 8, "two-pass")])
def test_teams_that_are_not_covered_are_taken_on_request_only(laq, L, W, kind):
    # 128 workgroups are the longest team whose waits end whatever else the device runs (tests/test_team_places.py)
    assert laq.laq_score_kernel(1, 32, 8, D, L, W, torch.bfloat16) == kind
    assert laq.laq_score_kernel(1, 32, 8, D, L, W, torch.bfloat16, choose="single-read") == "single-read"


def test_ordinary_launch_gives_the_same_bits(laq, tmp_path):
    # LAQ_COOPERATIVE_LAUNCH=0 (read once per process, so a child process): the same kernel on the same
    # grid, started without the cooperative guarantee, for profilers that cannot follow cooperative launches
    import os
    import subprocess
    import sys
    n, Hkv, G, L, W = 2, 3, 4, 5000, 16
    q, k = draw(n, Hkv, G, L, W, seed=77)
    want = laq.laq_score(q.to(DEV), k.to(DEV), 7, choose="single-read").cpu()
    torch.save({"q": q, "k": k}, tmp_path / "in.pt")
    code = (
        "import sys, torch\n"
        "sys.path.insert(0, %r)\n"
        "import paper_2505_20334_amd as laq\n"
        "d = torch.load(%r, weights_only=True)\n"
        "s = laq.laq_score(d['q'].to('cuda:0'), d['k'].to('cuda:0'), 7, choose='single-read')\n"
        "torch.cuda.synchronize()\n"
        "torch.save(s.cpu(), %r)\n"
    ) % (os.path.dirname(os.path.dirname(os.path.abspath(__file__))), str(tmp_path / "in.pt"), str(tmp_path / "out.pt"))
    env = dict(os.environ, LAQ_COOPERATIVE_LAUNCH="0")
    res = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, res.stderr[-2000:]
    got = torch.load(tmp_path / "out.pt", weights_only=True)
    assert torch.equal(got, want)
