"""The merge of split partials by the workgroups that stored them, against the merge by a second launch (needs an MI355X).

Both do the same arithmetic on the same partials; the sums over the splits differ in their order, that is by some 1e-6 of the terms
before the final rounding to bf16, which may then fall to the neighbouring number (spacing: at most 2^-7 of it).  The second launch's
parity with the oracle is test_gpu_attn.py's and test_gpu_fp8kv.py's.  All ways of the merge by workgroups give the same bits.  Every way a workgroup can take is forced: it waits for the
others, it leaves at once (the last one then merges for all), and (merge = 3) it shares its rows with workgroups on other XCDs, whose
L2s do not see what it stores unless it is written back and theirs are invalidated.
"""
import pytest
import torch

from paper_2605_29727_amd import binding as btv
from paper_2605_29727_amd import synth

pytestmark = pytest.mark.gpu

WAYS = [dict(merge=2), dict(merge=2, wait_ticks=-1), dict(merge=3), dict(merge=3, wait_ticks=-1), dict(merge=0)]


def _inputs(seed, L, M, Hq, Hkv, D, fp8):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=g, device="cuda")
    Q, K, V = r(M, Hq, D).bfloat16(), r(L + M, Hkv, D), r(L + M, Hkv, D)
    K, V = ([x.to(torch.float8_e4m3fn).view(torch.uint8) for x in (K, V)] if fp8 else [x.bfloat16() for x in (K, V)])
    return Q, K, V, torch.from_numpy(synth.tree_parents(seed, M, "random")).cuda()


def _call(x, L, ws, nsplit, shape, **how):
    O = torch.full_like(x[0], float("nan"))
    btv.btv_tree_verify_attn_merge_tuned(x[0], x[1], x[2], x[3], L, O, ws, 0.0, nsplit, shape, **how)
    return O


def _xcds(ws, n):
    """The XCDs that the first group's workgroups of the last call ran on: the first n words behind the workspace's header (256 bytes)
    hold tag << 8 | XCD.  None where no call has merged inside."""
    words = ws[256:256 + 8 * n].view(torch.int64).tolist()
    assert len({w >> 8 for w in words}) == 1
    return {w & 255 for w in words} if words[0] >> 8 else None


def _close(O, ref):
    o, r = O.float(), ref.float()
    return bool(((o - r).abs() <= r.abs() * 2.0 ** -7 + 1e-6).all())


# (L, M, Hq, Hkv, D, fp8, shape, splits): one row block and several, a ragged last one, a single row in it, heads that fill the
# XCDs and heads that only do so with their row blocks, the most splits, two workgroups on a CU, no room for all at once, few heads
CASES = [(8192, 64, 32, 8, 128, False, 2, 16), (3001, 33, 32, 8, 128, False, 1, 9), (2000, 65, 16, 8, 128, False, 2, 5),
         (4000, 256, 32, 8, 128, False, 3, 8), (1531, 23, 32, 8, 64, False, 1, 13), (900, 128, 8, 2, 128, False, 1, 7),
         (700, 97, 16, 4, 64, False, 2, 4), (5000, 7, 64, 8, 128, False, 1, 32), (12003, 33, 32, 8, 128, True, 1, 20),
         (500, 100, 32, 8, 128, True, 2, 3), (333, 5, 16, 16, 64, False, 1, 2), (4000, 200, 32, 8, 128, False, 1, 8),
         (1000, 40, 8, 2, 128, False, 1, 6), (20000, 3, 8, 8, 64, False, 3, 32), (8192, 64, 32, 8, 128, False, 3, 29)]


@pytest.mark.parametrize("case", CASES)
def test_same_as_the_second_launch(case):
    L, M, Hq, Hkv, D, fp8, shape, nsplit = case
    x = _inputs(L, L, M, Hq, Hkv, D, fp8)
    ws = btv.alloc_workspace(btv.btv_tree_verify_attn_tuned_workspace(M, L, Hq, Hkv, D, fp8, nsplit, shape))
    ref = _call(x, L, ws, nsplit, shape, merge=1)
    assert torch.isfinite(ref).all()
    first = _call(x, L, ws, nsplit, shape, merge=2)
    assert _close(first, ref)
    for how in WAYS + WAYS[:2]:
        O = _call(x, L, ws, nsplit, shape, **how)
        assert torch.equal(O, first), how
        on = _xcds(ws, 2)
        if on and how["merge"] and torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert len(on) == (2 if how["merge"] == 3 else 1), how
    assert btv.btv_workspace_status(ws) == 0


def test_a_workspace_over_changing_sizes_and_ways():
    """Tags count on per group, so calls of other sizes (other groups and numbers of splits) in between, calls that leave early and a
    batch over pages on the same workspace change nothing."""
    cases = [CASES[0], CASES[8], CASES[4], CASES[3], CASES[7]]
    ws = btv.alloc_workspace(max(btv.btv_tree_verify_attn_tuned_workspace(M, L, Hq, Hkv, D, fp8, n, s) for L, M, Hq, Hkv, D, fp8, s, n in cases)
                             + btv.btv_tree_verify_attn_paged_workspace(1, 64, 512, 32, 8, 128))
    ins = [_inputs(i, c[0], *c[1:6]) for i, c in enumerate(cases)]
    refs = [_call(x, c[0], ws, c[7], c[6], merge=1) for x, c in zip(ins, cases)]
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")
    Q, K, V, par = _inputs(9, 512, 64, 32, 8, 128, False)
    pages = lambda t: t.reshape(36, btv.BTV_PAGE, 8, 128)
    for k in range(3):
        for i, (x, c) in enumerate(zip(ins, cases)):
            O = _call(x, c[0], ws, c[7], c[6], **WAYS[(i + k) % len(WAYS)])
            assert _close(O, refs[i]), (k, c)
        O = torch.full_like(Q, float("nan"))
        btv.btv_tree_verify_attn_paged(Q, pages(K), pages(V), torch.arange(36, dtype=torch.int32, device="cuda").reshape(1, 36), i32(0, 64),
                                       i32(512), par, 64, 512, O, ws)
        assert torch.isfinite(O).all()
    assert btv.btv_workspace_status(ws) == 0


def test_replays_of_a_graph():
    """Recorded once and replayed with other inputs, with eager calls on the same workspace in between."""
    L, M, Hq, Hkv, D, fp8, shape, nsplit = CASES[0]
    x, y = _inputs(1, L, M, Hq, Hkv, D, fp8), _inputs(2, L, M, Hq, Hkv, D, fp8)
    ws = btv.alloc_workspace(btv.btv_tree_verify_attn_tuned_workspace(M, L, Hq, Hkv, D, fp8, nsplit, shape))
    ref = [_call(z, L, ws, nsplit, shape, merge=2) for z in (x, y)]
    st = [t.clone() for t in x]
    O = torch.empty_like(x[0])
    run = lambda: btv.btv_tree_verify_attn_merge_tuned(st[0], st[1], st[2], st[3], L, O, ws, 0.0, nsplit, shape, merge=0)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
        with torch.cuda.graph(graph, stream=side):
            run()
            run()
    torch.cuda.current_stream().wait_stream(side)
    for k in range(4):
        for a, b in zip(st, (x, y)[k % 2]):
            a.copy_(b)
        O.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, ref[k % 2]), k
        assert torch.equal(_call(y, L, ws, nsplit, shape, merge=2), ref[1]), k


@pytest.mark.parametrize("case", [CASES[0], CASES[4], CASES[11][:6] + (3, 8), CASES[12]])
def test_beside_a_kernel_that_holds_compute_units(case):
    """Workgroups whose peers cannot start leave, and the last one merges for them: the same bits, and the calls on the other stream end
    while that kernel runs or after it, whichever way the two are scheduled."""
    L, M, Hq, Hkv, D, fp8, shape, nsplit = case
    x = _inputs(3, L, M, Hq, Hkv, D, fp8)
    ws = btv.alloc_workspace(btv.btv_tree_verify_attn_tuned_workspace(M, L, Hq, Hkv, D, fp8, nsplit, shape))
    ref = _call(x, L, ws, nsplit, shape, merge=2)
    sink = torch.zeros(4096, dtype=torch.int32, device="cuda")
    here, there = torch.cuda.Stream(), torch.cuda.Stream()
    for held in (64, 192):
        torch.cuda.synchronize()
        with torch.cuda.stream(there):
            btv.btv_mfma_peak(held, 20000, sink)                # (2 ms)
        with torch.cuda.stream(here):
            outs = [_call(x, L, ws, nsplit, shape, merge=2) for _ in range(10)]
        torch.cuda.synchronize()
        assert all(torch.equal(O, ref) for O in outs)
    assert btv.btv_workspace_status(ws) == 0
