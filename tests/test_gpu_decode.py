"""Decode attention at the edges of its kernels' variants, against the oracle (needs an MI355X)."""
import pytest
import torch

import oracle
from parity_util import split_packed
from test_gpu_parity import check_decode

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F32, BF16 = torch.float32, torch.bfloat16


def _inputs(dtype, n, Hq, Hkv, d, L, budgets):
    import paper_2505_20334_amd as laq
    g = torch.Generator().manual_seed(d + L)
    total, _ = laq.packed_rows(budgets, Hkv, L)
    return ((torch.randn(n, Hq, d, generator=g) * 1.5).to(dtype), torch.randn(total, d, generator=g).to(dtype),
            torch.randn(total, d, generator=g).to(dtype))


# (dtype, Hq, Hkv, d, budgets): every head batch (one KV head's queries in one workgroup, and in several), every
# number of lanes per row with full and missing pieces; one row, ends of turns, one part and several, the most parts
CASES = [
    (BF16, 4, 4, 64, [1, 63, 64, 65]), (BF16, 6, 3, 24, [129, 257]), (BF16, 8, 2, 72, [2048, 640]), (BF16, 7, 1, 128, [64, 65, 1000]),
    (BF16, 8, 1, 96, [9000]), (BF16, 9, 1, 128, [700]), (BF16, 40, 2, 256, [513, 70]), (BF16, 6, 2, 200, [128, 128, 128]),
    (F32, 3, 3, 8, [65, 5]), (F32, 4, 2, 64, [320, 1]), (F32, 8, 2, 128, [512]), (F32, 28, 4, 136, [333, 64]), (F32, 5, 1, 256, [1100]),
    (BF16, 1, 1, 128, [20000]),
    # parts as even as their steps allow, and longer ones where the last parts would make too many workgroups
    (BF16, 16, 8, 64, [200] * 60), (F32, 8, 8, 72, [1000 - 900 * i // 11 for i in range(12)]), (BF16, 8, 8, 128, [321, 320, 2000] * 5),
    # one long cache among short ones, that makes more workgroups than the others leave room for; and whole caches that do alone
    (BF16, 8, 8, 128, [3000] + [64] * 95), (F32, 16, 8, 64, [5000] + [64] * 99), (BF16, 8, 8, 64, [300, 200] * 55),
]


@pytest.mark.parametrize("dtype,Hq,Hkv,d,budgets", CASES)
def test_decode_variants(dtype, Hq, Hkv, d, budgets):
    import paper_2505_20334_amd as laq
    print("case:", dtype, Hq, Hkv, d, budgets, flush=True)
    n, L = len(budgets), max(budgets)
    q, kc, vc = _inputs(dtype, n, Hq, Hkv, d, L, budgets)
    k_l, v_l = split_packed(kc, budgets, Hkv, L), split_packed(vc, budgets, Hkv, L)
    for split in (True, False):
        out = laq.laq_decode_attention(q.to(DEV), kc.to(DEV), vc.to(DEV), budgets, Hkv, L, split=split)
        torch.cuda.synchronize()
        for i in range(n):
            check_decode(out[i].cpu(), q[i], k_l[i].contiguous(), v_l[i].contiguous(), dtype, "inst %d split %s" % (i, split))


@pytest.mark.parametrize("offset", [0, 4])
def test_captured_decode_in_parts(offset):
    # replays with new inputs (sums left over from the replay before would show), the workspace left alone and overwritten in
    # between; a workspace of any alignment
    import paper_2505_20334_amd as laq
    n, Hq, Hkv, d, L, budgets = 3, 8, 2, 128, 1500, [1500, 700, 64]
    q, kc, vc = (x.to(DEV) for x in _inputs(BF16, n, Hq, Hkv, d, L, budgets))
    need = laq.laq_decode_workspace_bytes(n, Hq, Hkv, d, L, BF16, budgets)
    area = torch.randint(0, 256, (need + 8,), dtype=torch.uint8, device=DEV)
    ws, out = area[offset:offset + need], torch.empty(n, Hq, d, device=DEV)
    laq.laq_decode_attention(q, kc, vc, budgets, Hkv, L, ws=ws)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        laq.laq_decode_attention(q, kc, vc, budgets, Hkv, L, out=out, ws=ws)
    for replay in range(6):
        out.fill_(7.0)
        for x in (q, kc, vc):
            x.normal_()
        want = laq.laq_decode_attention(q, kc, vc, budgets, Hkv, L)           # (in a workspace of its own)
        if replay % 3 == 2:
            area[: need // 2].random_(0, 256)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), "replay %d" % replay
