"""Parity of the HIP acceptance walks with the CPU oracle: argmax, path, n_acc and bonus are bit-exact."""
import numpy as np
import pytest

from paper_2605_29727_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _depths(parent):
    d = np.zeros(len(parent), dtype=np.int32)
    for i in range(len(parent)):
        d[i] = 1 if parent[i] < 0 else d[parent[i]] + 1
    return d


def _greedy_case(G, oracle, store, f32, bits, parent, token):
    ref = oracle.accept_greedy(f32, parent, token)
    got = G.run_accept_greedy(store, bits, parent, token)
    assert np.array_equal(got["argmax"], ref["argmax"])
    assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]) and got["bonus"] == ref["bonus"]
    return ref


def test_greedy_config1(G, oracle):
    w = synth.C1
    tree = oracle.tree_build(synth.marginals(w.seed, w.B, w.V, w.marg_sigma), w.N)
    store, f = synth.target_logits(w.seed, w.N + 1, w.V, w.logit_sigma, "fp32")
    _greedy_case(G, oracle, store, f, False, tree["parent"], tree["token"])
    for leaf in range(w.N):
        x = synth.plant_path(f, tree["parent"], tree["token"], leaf)
        r = _greedy_case(G, oracle, x, x, False, tree["parent"], tree["token"])
        assert r["n_acc"] >= tree["depth"][leaf]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_greedy_config2_full_vocab_with_planted_paths(G, oracle, dtype):
    w = synth.C2
    tree = oracle.tree_build(synth.marginals(w.seed, w.B, w.V, w.marg_sigma), w.N)
    _, f = synth.target_logits(w.seed, w.N + 1, w.V, w.logit_sigma, "fp32")
    deep = int(np.argmax(tree["depth"]))
    for leaf in (-1, deep, 0, w.N // 2):
        x = synth.plant_path(f, tree["parent"], tree["token"], leaf)
        store, xf = synth.round_to_dtype(x.astype(np.float64), dtype)
        r = _greedy_case(G, oracle, store, xf, dtype == "bf16", tree["parent"], tree["token"])
        if leaf >= 0:
            assert r["n_acc"] >= tree["depth"][leaf]
    # bf16 logits tie often at 128k draws: the argmax must still be the lowest index
    store, xf = synth.round_to_dtype(np.round(f.astype(np.float64) * 4) / 4, dtype)
    _greedy_case(G, oracle, store, xf, dtype == "bf16", tree["parent"], tree["token"])


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [2049, 4099, 20001, 32768, 49152, 49153])
def test_stochastic_exchanges_in_one_l2_and_through_memory(G, V, dtype):
    """The library's own choice (up to 24 workgroups on one XCD) and the same number of them dealt out over the chip do the same arithmetic: the same
    path and bonus for wide fans that are rejected, followed drafts and what lies between, call after call on one workspace."""
    import torch
    from paper_2605_29727_amd import binding as btv
    N, B = 90, 10
    g = torch.Generator(device="cuda"); g.manual_seed(V)
    wgs = -(-V // 2048)
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(N, V, True))
    z = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
    for k, (kind, noise) in enumerate([("star", 3.0), ("random", 2.0), ("chain", 0.3), ("deep", 0.5), ("star", 0.5)]):
        marg = torch.softmax(3 * torch.randn((B, V), generator=g, device="cuda"), 1)
        parent = synth.tree_parents(V + k, N, kind)
        depth = _depths(parent)
        keep = depth <= B
        parent = torch.from_numpy(np.where(keep, parent, -1).astype(np.int32)).cuda()
        order = marg.argsort(1, descending=True)
        rank = {}
        token = []
        for i, pa in enumerate(parent.tolist()):
            rank[pa] = rank.get(pa, -1) + 1
            token.append(int(order[min(int(depth[i]), B) - 1, rank[pa]]))
        x = torch.randn((N + 1, V), generator=g, device="cuda") * noise
        if kind in ("chain", "deep"):
            x += marg.clamp(min=1e-30).log()[torch.from_numpy(np.concatenate([[0], depth])).clamp(max=B - 1).long().cuda()]
        x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        u = torch.rand(N + 1, generator=g, device="cuda")
        tok = torch.tensor(token, dtype=torch.int32, device="cuda")
        res = []
        for most in (0, wgs, 0):
            path, n, b = z(N), z(1), z(1)
            btv.btv_tree_accept_stochastic_tuned(x, marg, parent, tok, u, path, n, b, ws, most)
            res.append((int(n), path[:int(n)].tolist(), int(b)))
        assert res[0] == res[1] == res[2], (kind, res)
    assert btv.btv_workspace_status(ws) == 0


@pytest.mark.parametrize("V, walks", [(20001, 4), (40000, 2), (49152, 3), (49152, 4)])
def test_stochastic_walks_on_several_streams(G, V, walks):
    """Walks that are laid out for one XCD, each on a stream and a workspace of its own: the results of a walk that has the chip to itself, and none of
    them waits for another until its limit and is done alone.  Every slice has been counted in twice per call."""
    import torch
    from paper_2605_29727_amd import binding as btv
    N, B, calls = 100, 4, 20
    g = torch.Generator(device="cuda"); g.manual_seed(V)
    marg = torch.softmax(3 * torch.randn((B, V), generator=g, device="cuda"), 1)
    x = torch.randn((N + 1, V), generator=g, device="cuda") * 3
    u = torch.rand(N + 1, generator=g, device="cuda")
    parent = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    tok = marg[0].argsort(descending=True)[:N].to(torch.int32)
    ws = [btv.alloc_workspace(btv.btv_tree_accept_workspace(N, V, True)) for _ in range(walks)]
    out = lambda: [torch.zeros(n, dtype=torch.int32, device="cuda") for n in (N, 1, 1)]
    ref = out()
    btv.btv_tree_accept_stochastic(x, marg, parent, tok, u, *ref, ws[0])
    outs = [[out() for _ in range(calls)] for _ in range(walks)]
    streams = [torch.cuda.Stream() for _ in range(walks)]
    sink = torch.zeros(4096, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    btv.btv_mfma_peak(256, 20000, sink)                          # (2 ms: all calls are queued behind it)
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for k in range(calls):
        for s, w, o in zip(streams, ws, outs):
            with torch.cuda.stream(s):
                btv.btv_tree_accept_stochastic(x, marg, parent, tok, u, *o[k], w)
    torch.cuda.synchronize()
    for w, o in zip(ws, outs):
        for path, n, bonus in o:
            assert int(n) == int(ref[1]) and int(bonus) == int(ref[2]) and torch.equal(path[:int(n)], ref[0][:int(n)])
        assert w[72:80].view(torch.int32).tolist() == [0, 0]     # nobody has claimed a walk alone
        ran = calls + (w is ws[0])
        slices = -(-V // 2048)
        assert w[128:256].view(torch.int32).tolist() == [2 * ran] * slices + [0] * (32 - slices)
        assert btv.btv_workspace_status(w) == 0


@pytest.mark.parametrize("V, N, step", [(4097, 40, 1), (20001, 100, 1), (20001, 100, 3), (49152, 100, 1), (49152, 100, 5)])
def test_stochastic_slices_walked_by_stand_ins(G, V, N, step):
    """Every step-th slice looks as if it had been taken already when its workgroup starts (its count is odd), so that the workgroup leaves and the
    stand-in on another XCD walks the slice.  The path, the bonus and the counts are those of a walk by the first workgroups."""
    import torch
    from paper_2605_29727_amd import binding as btv
    g = torch.Generator(device="cuda"); g.manual_seed(V)
    marg = torch.softmax(3 * torch.randn((4, V), generator=g, device="cuda"), 1)
    u = torch.rand(N + 1, generator=g, device="cuda")
    parent = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    parent[N // 2:] = torch.arange(N - N // 2, dtype=torch.int32, device="cuda")
    tok = marg[0].argsort(descending=True)[:N].to(torch.int32)
    slices, calls = -(-V // 2048), 3
    for scale in (3.0, 0.0):                                     # a target of its own; one that follows the draft
        x = marg.log()[:1] * (scale == 0.0) + torch.randn((N + 1, V), generator=g, device="cuda") * max(scale, 0.2)
        got = []
        for odd in (0, 1):
            ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(N, V, True))
            turn = ws[128:256].view(torch.int32)
            turn[:slices:step] = odd
            want = turn + 2 * calls * (torch.arange(32, device="cuda") < slices)
            for _ in range(calls):
                out = [torch.zeros(n, dtype=torch.int32, device="cuda") for n in (N, 1, 1)]
                btv.btv_tree_accept_stochastic(x, marg, parent, tok, u, *out, ws)
                got.append([o.tolist() for o in out])
            assert turn.tolist() == want.tolist()
            assert ws[72:80].view(torch.int32).tolist() == [0, 0]     # nobody has claimed a walk alone
            assert btv.btv_workspace_status(ws) == 0
        assert all(o == got[0] for o in got)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [257, 300, 511, 1021, 4089, 4095, 4096, 4103, 8190, 8193, 8201, 12287])
def test_greedy_rows_at_any_element(G, oracle, V, dtype):
    """The first row, and with it all others, begins 0 .. 7 elements behind a multiple of 16 bytes.  The largest value is among a row's or a unit's first and
    last few elements (which are no whole 16 bytes) as often as inside; it occurs more than once; rows of -inf and NaN have their rule."""
    import torch
    from paper_2605_29727_amd import binding as btv
    M, nb = 17, 3
    rows = M + nb
    rng = np.random.default_rng(V)
    x = np.round(rng.standard_normal((rows, V)) * 2).astype(np.float32) / 2          # few values: ties everywhere
    ends = [0, 1, 6, 7, 8, V - 9, V - 8, V - 2, V - 1] + [v for v in (4088, 4095, 4096, 8184, 8191, 8192) if v < V]
    for r in range(rows - 4):
        for v in rng.choice(ends, 2, replace=False):
            x[r, v] = 9.0
    x[rows - 4] = -np.inf
    x[rows - 3] = np.nan
    x[rows - 2] = -np.inf; x[rows - 2, V - 1] = -3.0
    x[rows - 1] = -np.inf; x[rows - 1, 0] = np.nan
    want = [int(np.argmax(np.where(np.isnan(r), -np.inf, r))) if (r > -np.inf).any() or not np.isnan(r).any() else
            int(np.argmax(~np.isnan(r))) for r in x]
    parent, token = synth.tree_parents(V, M, "random"), np.arange(M, dtype=np.int32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    z = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
    for shift in range(8 if dtype == "bf16" else 4):
        room = torch.zeros(rows * V + shift, dtype=dt, device="cuda")
        room[shift:] = torch.from_numpy(x.reshape(-1)).to(dt).cuda()
        rows_at = room[shift:].view(rows, V)
        am = z(rows)
        btv.btv_tree_accept_greedy(rows_at[nb - 1:], G.dev(parent), G.dev(token), z(M), z(1), z(1), am[:M + 1],
                                   btv.alloc_workspace(btv.btv_tree_accept_workspace(M, V, False)))
        assert am[:M + 1].tolist() == want[nb - 1:], shift
        offsets = np.array([0, 2, 3, M], dtype=np.int32)
        forest = np.concatenate([synth.tree_parents(r, int(n), "random") for r, n in enumerate(np.diff(offsets))]).astype(np.int32)
        btv.btv_tree_accept_greedy_batch(rows_at, G.dev(forest), G.dev(token), G.dev(offsets), M, z(M), z(nb), z(nb), am,
                                         btv.alloc_workspace(btv.btv_tree_accept_batch_workspace(nb, M, V)))
        assert am.tolist() == want, shift


@pytest.mark.parametrize("kind", ["chain", "star", "binary", "random", "deep"])
@pytest.mark.parametrize("M,V", [(1, 1), (7, 13), (256, 1000), (100, 8193), (33, 128256)])
def test_greedy_tree_kinds_and_odd_vocabularies(G, oracle, kind, M, V):
    parent = synth.tree_parents(5, M, kind)
    fan = max(np.bincount(parent + 1).max(), 1)
    if fan > V:
        pytest.skip("fan-out exceeds the vocabulary")
    token = synth.sibling_distinct_tokens(5, parent, V)
    for dtype in ("bf16", "fp32"):
        _, f = synth.target_logits(6, M + 1, V, 1.0, "fp32", tag=f"{kind}{M}{V}")
        leaf = int(np.argmax(_depths(parent)))
        x = synth.plant_path(f, parent, token, leaf)
        store, xf = synth.round_to_dtype(x.astype(np.float64), dtype)
        _greedy_case(G, oracle, store, xf, dtype == "bf16", parent, token)


def test_greedy_all_equal_and_neg_inf_rows(G, oracle):
    M, V = 5, 300
    parent = synth.tree_parents(0, M, "chain")
    token = np.zeros(M, dtype=np.int32)
    x = np.zeros((M + 1, V), dtype=np.float32)
    r = _greedy_case(G, oracle, x, x, False, parent, token)     # every row ties everywhere: argmax 0 -> full chain
    assert r["n_acc"] == M and r["bonus"] == 0
    x[:] = -np.inf
    _greedy_case(G, oracle, x, x, False, parent, token)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_greedy_neg_inf_in_whole_units(G, oracle, dtype):
    """Rows that are -inf nearly everywhere, over a vocabulary of two whole scan units and a ragged one: a lane
    whose elements are all -inf has nothing "larger than the start value", which is the case the scan's cheap pass
    hands back to the exact one."""
    M, V = 4, 2 * 4096 + 777
    parent = synth.tree_parents(0, M, "chain")
    x = np.full((M + 1, V), -np.inf, dtype=np.float32)
    x[1, 5000] = -3.0                       # one finite value in the second unit
    x[2, V - 1] = 0.5                       # only the last element of the ragged unit
    x[3, :] = np.linspace(-4.0, 4.0, V, dtype=np.float32)[::-1]
    x[3, 4096] = 9.0
    x[4, 4095], x[4, 4096] = 2.0, 2.0       # a tie across two units
    token = np.array([0, 5000, V - 1, 4096], dtype=np.int32)
    store, xf = synth.round_to_dtype(x.astype(np.float64), dtype)
    r = _greedy_case(G, oracle, store, xf, dtype == "bf16", parent, token)
    assert r["n_acc"] == 4 and r["bonus"] == 4095


def test_greedy_signed_zeros_tie_and_workspace_reuse(G, oracle):
    """-0.0 and +0.0 are the same value: the lower index wins whichever sign it carries.  One workspace then serves
    calls of different sizes in a row: the slots that the workgroups leave their keys in are back at zero after each."""
    import torch
    from paper_2605_29727_amd import binding as btv
    M, V = 3, 9000
    parent = synth.tree_parents(0, M, "chain")
    x = np.full((M + 1, V), -1.0, dtype=np.float32)
    x[0, 5000], x[0, 17] = 0.0, -0.0
    x[1, 17], x[1, 8999] = 0.0, -0.0
    x[2, 8999], x[2, 4096] = -0.0, -0.0
    x[3, 1] = 0.0
    token = np.array([17, 17, 4096], dtype=np.int32)
    r = _greedy_case(G, oracle, x, x, False, parent, token)
    assert r["n_acc"] == 3 and r["bonus"] == 1

    V = 128256
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(256, V, False))
    for M, kind, seed in ((64, "random", 1), (5, "chain", 2), (256, "deep", 3), (64, "random", 1)):
        parent = synth.tree_parents(seed, M, kind)
        token = synth.sibling_distinct_tokens(seed, parent, V)
        _, f = synth.target_logits(seed, M + 1, V, 1.0, "fp32", tag=f"reuse{M}")
        x = synth.plant_path(f, parent, token, int(np.argmax(_depths(parent))))
        store, xf = synth.round_to_dtype(x.astype(np.float64), "bf16")
        ref = oracle.accept_greedy(xf, parent, token)
        d = G.dev(store, True)
        par, tok = G.dev(parent.astype(np.int32)), G.dev(token.astype(np.int32))
        path = torch.full((M,), -7, dtype=torch.int32, device="cuda")
        n_acc = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        bonus = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        am = torch.full((M + 1,), -7, dtype=torch.int32, device="cuda")
        for _ in range(2):                                   # twice in a row on the same workspace
            btv.btv_tree_accept_greedy(d, par, tok, path, n_acc, bonus, am, ws)
        torch.cuda.synchronize()
        n = int(n_acc.item())
        assert n == ref["n_acc"] and bonus.item() == ref["bonus"], (M, kind)
        assert np.array_equal(path.cpu().numpy()[:n], ref["path"]) and np.array_equal(am.cpu().numpy(), ref["argmax"])
    assert torch.count_nonzero(ws).item() == 0               # the workspace is left as it was handed over


def test_greedy_collector_gives_up_within_its_limit(G, oracle):
    """The workgroup that collects the others' keys waits for them with a limit on the wall clock.  A negative
    limit makes it give up before its first look: the kernel ends normally, the workspace's flag reports it, and
    the outputs are those of all-zero argmax rows.  The same call with a real limit, on a workspace zero-filled
    again, then gives the oracle's result."""
    import torch
    from paper_2605_29727_amd import binding as btv
    M, V = 40, 20000
    parent = synth.tree_parents(5, M, "random")
    token = synth.sibling_distinct_tokens(5, parent, V)
    _, f = synth.target_logits(5, M + 1, V, 1.0, "fp32", tag="limit")
    x = synth.plant_path(f, parent, token, int(np.argmax(_depths(parent))))
    store, xf = synth.round_to_dtype(x.astype(np.float64), "bf16")
    ref = oracle.accept_greedy(xf, parent, token)
    d = G.dev(store, True)
    par, tok = G.dev(parent.astype(np.int32)), G.dev(token.astype(np.int32))
    path = torch.full((M,), -7, dtype=torch.int32, device="cuda")
    n_acc = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    bonus = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    am = torch.full((M + 1,), -7, dtype=torch.int32, device="cuda")
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(M, V, False))
    btv.btv_tree_accept_greedy_tuned(d, par, tok, path, n_acc, bonus, am, ws, -1)
    torch.cuda.synchronize()
    assert btv.btv_workspace_status(ws) == btv.BTV_EDATA
    assert torch.count_nonzero(am).item() == 0 and 0 <= n_acc.item() <= M
    ws.zero_()
    btv.btv_tree_accept_greedy_tuned(d, par, tok, path, n_acc, bonus, am, ws, 100_000_000)
    torch.cuda.synchronize()
    assert btv.btv_workspace_status(ws) == 0
    n = int(n_acc.item())
    assert n == ref["n_acc"] and bonus.item() == ref["bonus"]
    assert np.array_equal(path.cpu().numpy()[:n], ref["path"]) and np.array_equal(am.cpu().numpy(), ref["argmax"])
    assert torch.count_nonzero(ws).item() == 0


AMBIGUOUS, AMBIGUOUS_GAP = 1e-4, 1e-6


def _ambiguous(ref):
    return ref["margin"] < AMBIGUOUS or ref["bonus_gap"] < AMBIGUOUS_GAP


@pytest.mark.parametrize("logit_dtype", ["fp32", "bf16"])
def test_stochastic_parity(G, oracle, logit_dtype):
    """Seeds whose accept tests sit within AMBIGUOUS (relative) of the threshold, or whose bonus draw sits within
    AMBIGUOUS_GAP (absolute) of a CDF step, are skipped: there the outcome
    depends on the rounding of vocabulary-wide sums and either result is correct."""
    B, V, N = 8, 5000, 48
    checked = 0
    for seed in range(12):
        marg = synth.marginals(100 + seed, B, V, 2.0)
        tree = oracle.tree_build(marg, N)
        # target close to the draft so that acceptances and rejections both happen
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(200 + seed, "noise", z.shape, 1.0)
        store, xf = synth.round_to_dtype(z, logit_dtype)
        u = synth.uniform(300 + seed, "u", (N + 1,)).astype(np.float32)
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, logit_dtype == "bf16", marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]), seed
        assert got["bonus"] == ref["bonus"], seed
        checked += 1
    assert checked >= 8


def test_stochastic_extremes(G, oracle):
    B, V, N = 4, 640, 20
    marg = synth.marginals(7, B, V, 2.0)
    tree = oracle.tree_build(marg, N)
    store, xf = synth.target_logits(8, N + 1, V, 1.0, "fp32")
    for u in (np.zeros(N + 1, dtype=np.float32), np.full(N + 1, 0.999999, dtype=np.float32)):
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        got = G.run_accept_stochastic(store, False, marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]) and got["bonus"] == ref["bonus"]


def test_config5_stochastic_full_vocab(G, oracle):
    w = synth.C5
    marg = synth.marginals(w.seed, w.B, w.V, w.marg_sigma)
    tree = oracle.tree_build(marg, w.N)
    store, xf = synth.target_logits(w.seed, w.N + 1, w.V, w.logit_sigma, w.logit_dtype)
    done = 0
    for k in range(6):
        u = synth.uniform(w.seed, f"uniforms{k}", (w.N + 1,)).astype(np.float32)
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, False, marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]) and got["bonus"] == ref["bonus"]
        done += 1
    assert done >= 3


@pytest.mark.parametrize("V,fan", [(300, 120), (5000, 200), (40000, 64), (2048 * 64 + 200, 48)])
def test_stochastic_wide_fans(G, oracle, V, fan):
    """Nodes with many children have their rejections solved together (Newton's method on sums over each slice's tokens, sorted
    into bins of e/q): flat marginals give a wide fan under the root, a target close to the draft makes acceptances late in the
    fan likely, and one workgroup, few, and slices of 2048 and of 4096 tokens are covered."""
    B = 3
    checked = 0
    for seed in range(8):
        marg = synth.marginals(700 + seed, B, V, 0.7)
        tree = oracle.tree_build(marg, fan)
        assert int((tree["parent"] == -1).sum()) >= min(fan, 40)
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(800 + seed, "noise", z.shape, [0.3, 1.0, 2.0][seed % 3])
        store, xf = synth.round_to_dtype(z, "fp32")
        u = synth.uniform(900 + seed, "u", (fan + 1,)).astype(np.float32)
        if seed % 4 == 3:
            u[:] = 0.999999           # everything that can be rejected is: the whole fan is walked
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, False, marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]), (V, fan, seed)
        assert got["bonus"] == ref["bonus"], (V, fan, seed)
        checked += 1
    assert checked >= 4


@pytest.mark.parametrize("V,fan", [(4000, 12), (4096, 255), (6000, 255), (10000, 130), (2048 * 15, 255), (2048 * 31, 66), (2048 * 33, 33),
                                   (2048 * 33, 34), (2048 * 63, 255), (2048 * 64, 20), (2048 * 64, 65)])
def test_stochastic_fans_over_the_workgroups(G, oracle, V, fan):
    """The sums at a fan's points are shared out among the workgroups in runs of a power of two: numbers of workgroups and of
    children that leave some with a shorter run or with none, one part per wavefront of the adding and many."""
    B = 2
    checked = 0
    for seed in range(5):
        marg = synth.marginals(730 + seed, B, V, 0.7)
        tree = oracle.tree_build(marg, fan)
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(830 + seed, "noise", z.shape, [0.3, 1.0, 2.0][seed % 3])
        store, xf = synth.round_to_dtype(z, "fp32")
        u = synth.uniform(930 + seed, "u", (fan + 1,)).astype(np.float32)
        if seed % 2 == 1:
            u[:] = 0.999999
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, False, marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]), (V, fan, seed)
        assert got["bonus"] == ref["bonus"], (V, fan, seed)
        checked += 1
    assert checked >= 2


def test_stochastic_wide_fan_long_vocabulary(G, oracle):
    """A vocabulary of 300000: slices of 8192 tokens, eight per thread where a fan is sorted, and a ragged last one.  With
    probabilities this small most seeds fall under the ambiguity margins; those that do not must agree."""
    B, V, fan = 3, 300000, 40
    checked = 0
    for seed in range(8):
        marg = synth.marginals(700 + seed, B, V, 0.7)
        tree = oracle.tree_build(marg, fan)
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(800 + seed, "noise", z.shape, [0.3, 1.0, 2.0][seed % 3])
        store, xf = synth.round_to_dtype(z, "fp32")
        u = synth.uniform(900 + seed, "u", (fan + 1,)).astype(np.float32)
        if seed % 4 == 3:
            u[:] = 0.999999
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, False, marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]), seed
        assert got["bonus"] == ref["bonus"], seed
        checked += 1
    assert checked >= 2


@pytest.mark.parametrize("V", [1, 5, 2047, 2049, 30000, 131072, 131073, 262148, 524301])
@pytest.mark.parametrize("logit_dtype", ["fp32", "bf16"])
def test_stochastic_slices(G, oracle, V, logit_dtype):
    """Vocabularies around the limits of the slices that the workgroups take (2048, 4096 and 8192 tokens, 64 workgroups at
    most, longer slices above), whole and ragged, over a deep tree whose first children are mostly accepted and over
    one with a fan of 24 at the root."""
    checked = 0
    for seed, (B, N, sigma, noise) in enumerate([(6, 12, 4.0, 0.3), (2, 24, 0.5, 2.0), (6, 12, 4.0, 0.0)]):
        marg = synth.marginals(40 + seed, B, V, sigma)
        tree = oracle.tree_build(marg, N)
        M = len(tree["parent"])
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(50 + seed, "noise", z.shape, noise)
        store, xf = synth.round_to_dtype(z, logit_dtype)
        u = synth.uniform(60 + seed, "u", (M + 1,)).astype(np.float32)
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if V > 1 and _ambiguous(ref):
            continue
        got = G.run_accept_stochastic(store, logit_dtype == "bf16", marg, tree["parent"], tree["token"], u)
        assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]), (V, seed)
        assert got["bonus"] == ref["bonus"], (V, seed)
        checked += 1
    assert checked >= 1


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 7, 8, 9, 13])
def test_stochastic_first_children_taken_to_any_depth(G, oracle, M):
    """Chains (read four rows at a time) of M nodes, with a second child at the root in half of them, that are followed to the end, or to the child
    whose uniform rejects it, at every level: the last row of a read, the first of the next, the end of the tree."""
    V, B = 3000, 14
    marg = synth.marginals(74, B, V, 3.0)
    order = np.argsort(-marg, axis=1, kind="stable")
    for second in (False, True):
        parent = [-1] + [i for i in range(M - 1)]
        depth = list(range(M))
        if second and M > 1:
            parent[1:] = [-1] + [0 if i == 2 else i - 1 for i in range(2, M)]
            depth = [0, 0] + [i - 1 for i in range(2, M)]
        token = [int(order[min(d, B - 1), 1 if (second and i == 1) else 0]) for i, d in enumerate(depth)]
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], np.asarray(depth) + 1]), B - 1)].astype(np.float64), 1e-30))
        store, xf = synth.round_to_dtype(z, "fp32")
        for stop in range(M + 1):
            u = np.full(M + 1, 0.25, dtype=np.float32)
            if stop < M:
                u[stop] = 0.99999
                xf2, store2 = xf.copy(), store.copy()
                row = parent[stop] + 1                   # this row's target has little on that child
                store2[row, token[stop]] -= 6
                xf2[row, token[stop]] -= 6
            else:
                xf2, store2 = xf, store
            ref = oracle.accept_stochastic(xf2, marg, np.asarray(parent, dtype=np.int32), np.asarray(token, dtype=np.int32), np.asarray(depth, dtype=np.int32), u)
            if _ambiguous(ref):
                continue
            got = G.run_accept_stochastic(store2, False, marg, parent, token, u)
            assert got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]) and got["bonus"] == ref["bonus"], (second, stop)


@pytest.mark.parametrize("V", [3, 4, 6, 7, 2049, 5000, 5001, 5002, 5003, 9996])
@pytest.mark.parametrize("logit_dtype", ["fp32", "bf16"])
def test_stochastic_rows_at_any_element(G, oracle, V, logit_dtype):
    """Rows that begin on any element and end in any part of a piece of four (the last one is loaded from V - 4 on), in one slice and in several:
    the same walk as from aligned arrays, and the oracle's."""
    import torch
    from paper_2605_29727_amd import binding as btv
    marg = synth.marginals(71, 6, V, 4.0)
    tree = oracle.tree_build(marg, 24)
    M = len(tree["parent"])
    z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), 5)].astype(np.float64), 1e-30)) + synth.normal(72, "noise", (M + 1, V), 0.3)
    store, xf = synth.round_to_dtype(z, logit_dtype)
    u = synth.uniform(73, "u", (M + 1,)).astype(np.float32)
    ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
    whole = G.run_accept_stochastic(store, logit_dtype == "bf16", marg, tree["parent"], tree["token"], u)
    if not _ambiguous(ref):
        assert whole["n_acc"] == ref["n_acc"] and np.array_equal(whole["path"], ref["path"]) and whole["bonus"] == ref["bonus"]
    x, m = G.dev(store, logit_dtype == "bf16"), G.dev(marg.astype(np.float32))
    par, tok, uni = G.dev(np.asarray(tree["parent"], dtype=np.int32)), G.dev(np.asarray(tree["token"], dtype=np.int32)), G.dev(u)
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(M, V, True))

    def at(t, off):                                  # a copy that begins `off` elements behind an aligned address
        flat = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")
        flat[off:off + t.numel()] = t.flatten()
        return flat[off:off + t.numel()].view(t.shape)

    for dx, dm in ((1, 0), (2, 0), (4, 0), (8, 1), (0, 2), (4, 4), (3, 3)):
        out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (M, 1, 1)]
        btv.btv_tree_accept_stochastic(at(x, dx), at(m, dm), par, tok, uni, *out, ws)
        n = int(out[1].item())
        assert n == whole["n_acc"] and out[2].item() == whole["bonus"], (dx, dm)
        assert np.array_equal(out[0].cpu().numpy()[:n], whole["path"]), (dx, dm)


def test_stochastic_token_outside_vocabulary_is_flagged_not_faulting():
    """A token id outside [0, V) is never used as an index: that child counts as rejected, the data flag is raised,
    and the walk goes on with the valid children."""
    import torch
    import gpu_util as G
    from paper_2605_29727_amd import binding as btv
    B, V, M = 4, 300, 6
    marg = synth.marginals(97, B, V, 2.0)
    parent = np.array([-1, -1, 0, 0, 1, 2], dtype=np.int32)
    token = np.array([10 ** 9, 7, 5, -3, 9, 11], dtype=np.int32)
    st, _ = synth.target_logits(97, M + 1, V, 1.0, "fp32")
    path = torch.full((M,), -7, dtype=torch.int32, device="cuda")
    n_acc = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    bonus = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(M, V, True))
    btv.btv_tree_accept_stochastic(G.dev(st), G.dev(marg.astype(np.float32)), G.dev(parent), G.dev(token),
                                   G.dev(np.zeros(M + 1, dtype=np.float32)), path, n_acc, bonus, ws)
    torch.cuda.synchronize()
    assert btv.btv_workspace_status(ws) == btv.BTV_EDATA
    n = int(n_acc.item())
    assert 0 <= n <= M and 0 <= int(bonus.item()) < V
    assert 0 not in path.cpu().numpy()[:n].tolist()          # node 0 carries the invalid id: never accepted


def _walk_cases(oracle, V, logit_dtype):
    """A deep tree whose first children are mostly accepted, one whose first children are mostly not, and a fan of 24 all of
    which is rejected; without the ambiguous ones."""
    for seed, (B, N, sigma, noise) in enumerate([(6, 12, 4.0, 0.3), (6, 24, 3.0, 2.0), (2, 24, 0.5, 2.0)]):
        marg = synth.marginals(40 + seed, B, V, sigma)
        tree = oracle.tree_build(marg, N)
        M = len(tree["parent"])
        z = np.log(np.maximum(marg[np.minimum(np.concatenate([[0], tree["depth"]]), B - 1)].astype(np.float64), 1e-30))
        z += synth.normal(50 + seed, "noise", z.shape, noise)
        store, xf = synth.round_to_dtype(z, logit_dtype)
        u = synth.uniform(60 + seed, "u", (M + 1,)).astype(np.float32)
        if seed == 2:
            u[:24] = 0.999999
        ref = oracle.accept_stochastic(xf, marg, tree["parent"], tree["token"], tree["depth"], u)
        if not _ambiguous(ref):
            yield (store, logit_dtype == "bf16", marg, tree["parent"], tree["token"], u), ref


def _same(got, ref):
    return got["n_acc"] == ref["n_acc"] and np.array_equal(got["path"], ref["path"]) and got["bonus"] == ref["bonus"]


@pytest.mark.parametrize("V,workgroups", [(5000, 2), (5003, 1), (30000, 8), (30000, 4), (30001, 3), (128256, 32), (128256, 1)])
@pytest.mark.parametrize("logit_dtype", ["fp32", "bf16"])
def test_stochastic_on_few_compute_units(G, oracle, V, workgroups, logit_dtype):
    """Where fewer workgroups than the vocabulary has slices can run at once, the slices get longer (the register
    shapes at 4096 and 8192 tokens, slices read again from memory above), down to one workgroup."""
    checked = 0
    for args, ref in _walk_cases(oracle, V, logit_dtype):
        got = G.run_accept_stochastic(*args, tuned=(workgroups, 1000000))
        assert _same(got, ref) and got["status"] == 0, (V, workgroups)
        checked += 1
    assert checked >= 1


@pytest.mark.parametrize("V,workgroups", [(5000, 0), (30001, 0), (128256, 0), (128256, 32), (128256, 16), (131072, 5)])
@pytest.mark.parametrize("logit_dtype", ["fp32", "bf16"])
def test_stochastic_when_the_workgroups_do_not_run_at_once(G, oracle, V, workgroups, logit_dtype):
    """A wait limit below zero makes a workgroup leave the exchange at the first part it does not find: one of those that
    left walks the tree alone.  The results are the oracle's all the same, no flag is raised, and the next calls on the
    workspace, with and without the limit, are right too."""
    import torch
    from paper_2605_29727_amd import binding as btv
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(24, V, True))
    checked = 0
    for args, ref in _walk_cases(oracle, V, logit_dtype):
        for wait in (-1, -1, 1000000, -1, 1000000):
            got = G.run_accept_stochastic(*args, tuned=(workgroups, wait), ws=ws)
            assert _same(got, ref) and got["status"] == 0, (V, workgroups, wait)
        checked += 1
    torch.cuda.synchronize()
    words = ws[64:80].view(torch.int32).cpu().tolist()
    assert words[0] >= 1 << 20 and words[3] == 1                 # a walk was done alone, and its tags are left behind
    assert checked >= 1


def test_stochastic_workspace_serves_changing_sizes(G, oracle):
    """One workspace over calls of other vocabularies, other numbers of workgroups and walks that had to be done alone: the
    words of earlier calls, at other places, are taken for nothing."""
    from paper_2605_29727_amd import binding as btv
    ws = btv.alloc_workspace(btv.btv_tree_accept_workspace(24, 131072, True))
    cases = [(V, args, ref) for V in (1500, 5000, 30001, 131072) for args, ref in _walk_cases(oracle, V, "fp32")]
    assert len(cases) >= 6
    for turn in range(3):
        for k, (V, args, ref) in enumerate(cases[turn:] + cases[:turn]):
            got = G.run_accept_stochastic(*args, tuned=((0, 3, 17)[(turn + k) % 3], -1 if k % 4 == 3 else 1000000), ws=ws)
            assert _same(got, ref) and got["status"] == 0, (turn, V)


@pytest.mark.parametrize("bits", [False, True])
@pytest.mark.parametrize("V,M", [(1, 3), (15, 127), (16, 128), (64, 127), (64, 128), (65, 63), (128, 63), (128, 64), (129, 31), (256, 31), (256, 32), (257, 31),
                                 (64, 95), (64, 96), (128, 47), (128, 48), (200, 23), (256, 23), (256, 24)])
def test_greedy_small_vocabularies(G, oracle, V, M, bits):
    """Around the sizes up to which one workgroup takes all rows: last rows and last tokens, ties (the lowest id), rows of -inf and of
    signed zeros."""
    parent = synth.tree_parents(V + M, M, "random")
    token = (np.arange(M) % V).astype(np.int32)
    x = np.round(synth.target_logits(V + M, M + 1, V, 2.0, "fp32")[1] * 2) / 2
    x[0] = -np.inf
    x[min(2, M), :] = -0.0
    x[min(2, M), V // 2] = 0.0
    x[M, V - 1] = 50.0                                                        # the very last element
    store, xf = synth.round_to_dtype(x.astype(np.float64), "bf16" if bits else "fp32")
    _greedy_case(G, oracle, store, xf, bits, parent, token)
