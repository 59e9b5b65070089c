"""Parity of the HIP tree-verify attention with the CPU oracle (needs an MI355X; all calls go through the C ABI).

Tolerances: max-abs 1e-5 for the fp32 path, 2e-2 for bf16 (outputs are O(1) convex combinations of N(0,1) values;
one bf16 rounding of the output alone is up to 2^-9 * |O| ~ 8e-3 at |O| = 4).
"""
import numpy as np
import pytest

from paper_2605_29727_amd import synth

pytestmark = pytest.mark.gpu

TOL_BF16, TOL_F32 = 2e-2, 1e-5
KINDS = ["chain", "star", "binary", "caterpillar", "random", "deep"]


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def test_config1_fp32_full_parity(G, oracle):
    w = synth.C1
    marg = synth.marginals(w.seed, w.B, w.V, w.marg_sigma)
    tree = oracle.tree_build(marg, w.N)
    t = synth.qkv(w.seed, w.N, w.L, w.Hq, w.Hkv, w.D, "fp32")
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], tree["parent"], w.L)
    out = G.run_verify_attn(t, tree["parent"], w.L, "fp32")
    assert np.abs(out - ref).max() <= TOL_F32


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,L,Hq,Hkv,D", [(16, 128, 1, 1, 64), (37, 300, 4, 2, 128), (5, 0, 2, 1, 64), (1, 77, 2, 2, 128)])
def test_fp32_shapes_and_trees(G, oracle, kind, M, L, Hq, Hkv, D):
    parent = synth.tree_parents(7, M, kind)
    t = synth.qkv(31, M, L, Hq, Hkv, D, "fp32", tag=kind)
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
    out = G.run_verify_attn(t, parent, L, "fp32")
    assert np.abs(out - ref).max() <= TOL_F32


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("M,L", [(1, 127), (1, 255), (2, 126), (3, 254), (17, 240), (256, 0), (200, 313)])
def test_fp32_around_the_chunks_of_keys(G, oracle, M, L, D):
    for kind in ("random", "star", "chain"):
        parent = synth.tree_parents(8, M, kind)
        t = synth.qkv(32, M, L, 4, 2, D, "fp32", tag=kind)
        out = G.run_verify_attn(t, parent, L, "fp32")
        assert np.abs(out - oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)).max() <= TOL_F32


# (M, L, Hq, Hkv, D): spans all three kernel configurations (G*M <= 64, <= 128, > 128 with several row blocks),
# ragged tails (M, L not multiples of 32 / 64), L = 0, L smaller than a tile, and a prefix/tree boundary inside a tile.
BF16_SHAPES = [
    (16, 256, 32, 8, 128), (1, 100, 4, 1, 128), (5, 0, 8, 2, 128), (33, 31, 8, 2, 128), (64, 777, 32, 8, 128),
    (100, 1000, 8, 2, 128), (256, 300, 8, 2, 128), (37, 513, 64, 8, 128), (16, 200, 8, 8, 64), (70, 129, 16, 4, 64),
    (13, 64, 4, 4, 128), (128, 96, 16, 2, 128),
]


@pytest.mark.parametrize("shape", BF16_SHAPES)
def test_bf16_elementwise_parity(G, oracle, shape):
    M, L, Hq, Hkv, D = shape
    for kind in ("random", "deep", "chain"):
        parent = synth.tree_parents(M + L, M, kind)
        t = synth.qkv(41, M, L, Hq, Hkv, D, "bf16", tag=f"{kind}{shape}")
        ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
        out = G.run_verify_attn(t, parent, L, "bf16")
        assert np.isfinite(out).all()
        assert np.abs(out - ref).max() <= TOL_BF16, (kind, shape, np.abs(out - ref).max())


@pytest.mark.parametrize("kind", KINDS)
def test_bf16_tree_kinds_with_split(G, oracle, kind):
    M, L, Hq, Hkv, D = 48, 1500, 16, 4, 128
    parent = synth.tree_parents(3, M, kind)
    t = synth.qkv(42, M, L, Hq, Hkv, D, "bf16", tag=kind)
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
    outs = [G.run_verify_attn(t, parent, L, "bf16", nsplit=ns) for ns in (1, 2, 5, 25)]
    for o in outs:
        assert np.abs(o - ref).max() <= TOL_BF16
    for o in outs[1:]:       # any split count gives the single-split result up to the final bf16 rounding
        assert np.abs(o - outs[0]).max() <= 2 ** -7


def test_bf16_scale_argument(G, oracle):
    M, L = 20, 150
    parent = synth.tree_parents(1, M, "random")
    t = synth.qkv(43, M, L, 8, 2, 128, "bf16")
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L, scale=0.05)
    out = G.run_verify_attn(t, parent, L, "bf16", scale=0.05)
    assert np.abs(out - ref).max() <= TOL_BF16


def test_bf16_deterministic_and_mask_tight(G, oracle):
    """Same input twice -> identical bits; changing K/V of a non-ancestor tree row leaves a node's output bit-identical."""
    M, L, Hq, Hkv, D = 40, 600, 8, 2, 128
    parent = synth.tree_parents(11, M, "random")
    t = synth.qkv(44, M, L, Hq, Hkv, D, "bf16")
    a = G.run_verify_attn(t, parent, L, "bf16", nsplit=4)
    b = G.run_verify_attn(t, parent, L, "bf16", nsplit=4)
    assert np.array_equal(a, b)
    anc = oracle.ancestor_mask(parent)
    victim = 7
    t2 = dict(t)
    for nm in ("K", "V"):
        bits = t[nm].copy()
        bits[L + victim] ^= np.uint16(0x0180)            # flip mantissa/exponent bits of that tree row
        t2[nm] = bits
        t2[nm + "f"] = synth.bf16_bits_to_f32(bits)
    c = G.run_verify_attn(t2, parent, L, "bf16", nsplit=4)
    for i in range(M):
        sees = bool((anc[i, victim // 32] >> np.uint32(victim % 32)) & np.uint32(1))
        assert np.array_equal(c[i], a[i]) != sees, i


def test_ancestor_mask_bit_exact(G, oracle):
    import torch
    from paper_2605_29727_amd import binding as btv
    for kind in KINDS:
        for M in (1, 31, 32, 33, 200, 256):
            parent = synth.tree_parents(M, M, kind)
            anc = torch.zeros((M, 8), dtype=torch.int32, device="cuda")
            ws = btv.alloc_workspace(256)
            btv.btv_tree_ancestor_mask(G.dev(parent), anc, ws)
            torch.cuda.synchronize()
            assert np.array_equal(anc.cpu().numpy().view(np.uint32), oracle.ancestor_mask(parent))


@pytest.mark.parametrize("shape_id", [1, 2, 3])
@pytest.mark.parametrize("M", [1, 31, 33, 64, 65, 128, 129, 255, 256])
def test_bf16_every_node_sees_its_ancestors_alone(G, oracle, M, shape_id):
    """Keys of zero give every visible row the same weight, and channel d of tree row a is 64 where a % 128 == d, 0 elsewhere:
    O[i, d] is 64 times the number of ancestors a of i with a % 128 == d (0, 1 or 2), over L + the number of all of them.  The output is rounded
    by 2^-9 of itself, a partial by 2^-10 of the row's largest value, which is at most twice as large."""
    L, D = 5, 128
    for kind in KINDS:
        parent = synth.tree_parents(M + 1, M, kind)
        rows = np.zeros((L + M, 1, D), dtype=np.float32)
        rows[L + np.arange(M), 0, np.arange(M) % D] = 64.0
        t = {"Q": np.full((M, 2, D), 0x3F80, dtype=np.uint16), "K": np.zeros((L + M, 1, D), dtype=np.uint16),
             "V": (rows.view(np.uint32) >> 16).astype(np.uint16)}
        anc = np.unpackbits(oracle.ancestor_mask(parent).view(np.uint8), axis=1, bitorder="little")[:, :M].astype(np.float64)
        ref = anc @ rows[L:, 0] / (L + anc.sum(1, keepdims=True))
        for ns in (1, 3):
            out = G.run_verify_attn(t, parent, L, "bf16", nsplit=ns, shape=shape_id)
            assert np.all(np.abs(out - ref[:, None]) <= 2 ** -7 * ref[:, None]), (kind, ns)


def test_invalid_parent_is_flagged_not_faulting(G):
    import torch
    from paper_2605_29727_amd import binding as btv
    M, L = 8, 64
    t = synth.qkv(45, M, L, 4, 2, 128, "bf16")
    parent = synth.tree_parents(0, M, "chain")
    parent[3] = 5                                             # parent >= own index: invalid
    Q, K, V = G.dev(t["Q"], True), G.dev(t["K"], True), G.dev(t["V"], True)
    O = torch.zeros_like(Q)
    ws = btv.alloc_workspace(btv.btv_tree_verify_attn_workspace(M, L, 4, 2, 128, btv.BTV_BF16))
    btv.btv_tree_verify_attn(Q, K, V, G.dev(parent), L, O, ws)
    torch.cuda.synchronize()
    assert btv.btv_workspace_status(ws) == btv.BTV_EDATA
    assert btv.btv_workspace_status(ws) == btv.BTV_OK        # the flag is cleared by the read
    assert torch.isfinite(O.float()).all()


def _full_size_check(G, oracle, w, N, seed_tag):
    """Every (node, head) row of the full-size configuration against the oracle (the oracle runs all rows of the
    largest configuration in well under a minute on the GPU machine's host cores)."""
    marg = synth.marginals(w.seed, w.B, w.V, w.marg_sigma)
    tree = oracle.tree_build(marg, N)
    t = synth.qkv(w.seed, N, w.L, w.Hq, w.Hkv, w.D, "bf16", tag=seed_tag)
    out = G.run_verify_attn(t, tree["parent"], w.L, "bf16")
    assert np.isfinite(out).all()
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], tree["parent"], w.L)
    assert out.shape == ref.shape
    assert np.abs(out - ref).max() <= TOL_BF16, np.abs(out - ref).max()
    return out


def test_config2_full_size(G, oracle):
    _full_size_check(G, oracle, synth.C2, synth.C2.N, "c2")


@pytest.mark.parametrize("N", synth.C3_SIZES)
@pytest.mark.parametrize("sharp", [True, False])
def test_config3_budget_sweep_full_size(G, oracle, N, sharp):
    _full_size_check(G, oracle, synth.c3(N, sharp), N, f"c3{N}{sharp}")


def test_config5_70b_shape_full_size(G, oracle):
    _full_size_check(G, oracle, synth.C5, synth.C5.N, "c5")


# Every kernel shape on inputs the heuristic would give to another one: (M, L, Hq, Hkv, D), ragged tails in M and L,
# prefix/tree boundary inside a tile, fewer rows than the workgroup holds, several row blocks, one and several splits.
FORCED_SHAPES = [(16, 700, 32, 8, 128), (100, 1000, 8, 2, 128), (37, 513, 64, 8, 128), (70, 129, 16, 4, 64),
                 (5, 0, 8, 2, 128), (256, 300, 8, 2, 128)]


@pytest.mark.parametrize("shape_id", [1, 2, 3])
@pytest.mark.parametrize("dims", FORCED_SHAPES)
def test_bf16_every_kernel_shape_elementwise(G, oracle, shape_id, dims):
    M, L, Hq, Hkv, D = dims
    for kind, ns in (("random", 0), ("deep", 3)):
        parent = synth.tree_parents(M + L + shape_id, M, kind)
        t = synth.qkv(46, M, L, Hq, Hkv, D, "bf16", tag=f"{kind}{dims}")
        ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
        out = G.run_verify_attn(t, parent, L, "bf16", nsplit=ns, shape=shape_id)
        assert np.isfinite(out).all()
        assert np.abs(out - ref).max() <= TOL_BF16, (kind, dims, shape_id, np.abs(out - ref).max())


@pytest.mark.parametrize("steep", [2, 8])
@pytest.mark.parametrize("shape_id", [1, 2, 3])
@pytest.mark.parametrize("dims", [(16, 700, 32, 8, 128), (70, 1029, 16, 4, 64), (250, 650, 8, 2, 128)])
def test_bf16_maxima_that_grow_along_the_prefix(G, oracle, shape_id, dims, steep):
    """Scores of a standard deviation of 16 to 90 in log2 units: a row's maximum passes the reference taken from its first tile
    by more than 16 in most rows, by more than exp2 can hold in some."""
    M, L, Hq, Hkv, D = dims
    parent = synth.tree_parents(M + L, M, "random")
    t = synth.qkv(48, M, L, Hq, Hkv, D, "bf16", tag=f"grow{dims}")
    scale = steep * np.log(2)            # (a power of two times log2(e): the queries are not rounded again)
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L, scale=scale)
    out = G.run_verify_attn(t, parent, L, "bf16", nsplit=1, shape=shape_id, scale=scale)
    assert np.abs(out - ref).max() <= TOL_BF16


@pytest.mark.parametrize("dims,kind", [((256, 16384, 32, 8, 128), "random"), ((131, 16397, 16, 2, 128), "deep"),
                                       ((250, 16415, 64, 8, 128), "chain")])
def test_bf16_long_prefix_many_rows_elementwise(G, oracle, dims, kind):
    """Sizes at which the heuristic itself picks the 256-row workgroup (at least 1024 packed rows per KV head over a
    prefix of at least 16384 keys): every element, with ragged tails in both dimensions and deep trees."""
    M, L, Hq, Hkv, D = dims
    parent = synth.tree_parents(M + L, M, kind)
    t = synth.qkv(47, M, L, Hq, Hkv, D, "bf16", tag=f"{kind}{dims}")
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
    out = G.run_verify_attn(t, parent, L, "bf16")
    assert np.isfinite(out).all()
    assert np.abs(out - ref).max() <= TOL_BF16, (dims, kind, np.abs(out - ref).max())


def _paged_case(G, oracle, Ls, Ns, Hq, Hkv, D, seed, alike=1):
    """Every element against the oracle.  alike: so many times these heads, all with the same queries, keys and values, and so the same results.
    Returns what the workgroups left of their plan (G.batch_plan)."""
    import torch
    from paper_2605_29727_amd import binding as btv
    batch = len(Ls)
    bt, nb = synth.paged_layout(seed, [l + n for l, n in zip(Ls, Ns)])
    Kp = np.zeros((nb, synth.PAGE, Hkv, D), dtype=np.uint16)
    Vp = np.zeros_like(Kp)
    # unused pool slots hold NaN so that any stray read shows up
    Kp[:] = 0x7FC0
    Vp[:] = 0x7FC0
    qoff = np.zeros(batch + 1, dtype=np.int32)
    qoff[1:] = np.cumsum(Ns)
    Qall = np.zeros((int(qoff[-1]), Hq, D), dtype=np.uint16)
    parents = np.zeros(int(qoff[-1]), dtype=np.int32)
    reqs = []
    for r in range(batch):
        t = synth.qkv(seed, Ns[r], Ls[r], Hq, Hkv, D, "bf16", tag=f"req{r}")
        kinds = ["random", "deep", "binary", "chain", "star", "caterpillar"]
        parent = synth.tree_parents(seed + r, Ns[r], kinds[r % len(kinds)])
        synth.scatter_to_pages(t["K"], bt[r], Kp)
        synth.scatter_to_pages(t["V"], bt[r], Vp)
        Qall[qoff[r]:qoff[r + 1]] = t["Q"]
        parents[qoff[r]:qoff[r + 1]] = parent
        reqs.append((t, parent))
    Q, K, V = (G.dev(x, True).repeat(*(1,) * (x.ndim - 2), alike, 1) for x in (Qall, Kp, Vp))
    O = torch.full_like(Q, float("nan"))
    M_max, L_max = max(Ns), max(Ls)
    ws = btv.alloc_workspace(btv.btv_tree_verify_attn_paged_workspace(batch, M_max, L_max, Hq * alike, Hkv * alike, D))
    btv.btv_tree_verify_attn_paged(Q, K, V, G.dev(bt), G.dev(qoff), G.dev(np.asarray(Ls, dtype=np.int32)),
                                   G.dev(parents), M_max, L_max, O, ws)
    torch.cuda.synchronize()
    assert btv.btv_workspace_status(ws) == 0
    out = G.host(O).astype(np.float64)
    assert np.isfinite(out).all()
    assert np.array_equal(out, np.tile(out[:, :Hq], (1, alike, 1)))
    out = out[:, :Hq]
    Kpf, Vpf = synth.bf16_bits_to_f32(Kp), synth.bf16_bits_to_f32(Vp)
    for r, (t, parent) in enumerate(reqs):
        o = out[qoff[r]:qoff[r + 1]]
        ref = oracle.tree_attn(t["Qf"], Kpf, Vpf, parent, Ls[r], block_table=bt[r], page=synth.PAGE)
        assert np.abs(o - ref).max() <= TOL_BF16, r
    return G.batch_plan(ws)


@pytest.mark.parametrize("shape_id", [1, 2, 3])
@pytest.mark.parametrize("D", [64, 128])
def test_bf16_around_the_rings_and_the_trips(G, oracle, shape_id, D):
    """One part of as many tiles as the ring's stages, the rounds of two and the groups of eight trips make different paths of (all keys there
    or not, prefix rows only or not), whole tiles at the end of the prefix, of the sequence, and neither."""
    for tiles in (3, 4, 5, 6, 7, 8, 9, 10, 14, 15, 16, 17, 22, 23, 24, 25, 31):
        for L, M in ((32 * tiles, 3), (32 * tiles - 3, 3), (32 * tiles - 17, 5)):
            parent = synth.tree_parents(tiles, M, "random")
            t = synth.qkv(91, M, L, 2, 1, D, "bf16", tag=f"{L}")
            ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
            out = G.run_verify_attn(t, parent, L, "bf16", nsplit=1, shape=shape_id)
            assert np.abs(out - ref).max() <= TOL_BF16, (L, M, np.abs(out - ref).max())


@pytest.mark.parametrize("D", [64, 128])
def test_paged_around_the_windows_of_pages(G, oracle, D):
    """A grid of parts, and in it requests of 31 to 34 and 63 to 66 tiles, ending in either half of a tile and with it: with 64 channels around the windows of 32 tiles
    whose page ids are kept, with 128, which leave no room for them, with ids loaded one by one."""
    for tiles in (31, 33, 64):
        plan = _paged_case(G, oracle, [32 * tiles - 3, 32 * tiles + 13, 32 * tiles + 29, 32 * tiles + 45], [3, 3, 3, 19], 4, 1, D, seed=92 + tiles)
        assert plan == (0, 0)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N_lo, N_hi", [(33, 36), (20, 24)])         # 256-row blocks, the pipelined loop; 128-row blocks, two key-waves
def test_paged_around_the_windows_of_pages_of_whole_requests(G, oracle, N_lo, N_hi, D):
    """The work shared out, two whole requests a share: pieces of 31 to 33, 63 to 65 and 95 to 97 tiles, where the windows of 32 tiles' page ids turn with all loads in flight
    and at the ends of the requests."""
    Ls, Ns = G.whole_shares(64, N_lo, N_hi)
    share, head = _paged_case(G, oracle, Ls, Ns, 4, 1, D, seed=95, alike=8)
    assert head == 32 * share > 0                                     # (256 teams, none of which begins or ends within a request)


def test_paged_ragged_small(G, oracle):
    _paged_case(G, oracle, [100, 0, 333, 17, 1025], [9, 5, 33, 1, 64], 8, 2, 128, seed=61)
    _paged_case(G, oracle, [640, 64], [70, 130], 8, 2, 64, seed=62)


def test_config4_ragged_paged_full_size(G, oracle):
    Ls, Ns = synth.c4_request_shapes()
    _paged_case(G, oracle, Ls, Ns, 32, 8, 128, seed=synth.C4.seed)


def test_paged_ragged_several_splits(G, oracle):
    """Prefixes long enough for several key splits per request, of very different lengths: the split index is
    rotated per (request, head), short requests skip the splits they do not have, every element is compared."""
    _paged_case(G, oracle, [5000, 300, 2500, 4097, 64, 9000], [40, 64, 7, 100, 130, 16], 8, 2, 128, seed=63)
    _paged_case(G, oracle, [2100, 2047, 2049], [33, 32, 31], 4, 4, 64, seed=64)


def long_batch(batch, M_max, L_long, long_at):
    """Request sizes around the edges of the plan of a batch with much to do: stretches of 16 tiles, just longer ones, no prefix at all, one very long request; trees around the ends of row blocks."""
    Ls = [(0, 1, 31, 32, 495, 511, 513, 530, 700)[r % 9] for r in range(batch)]
    Ns = [(1, 2, M_max // 2, M_max // 2 + 1, M_max)[r % 5] for r in range(batch)]
    Ls[long_at] = L_long
    return Ls, Ns


@pytest.mark.parametrize("batch, M_max, L_long, long_at, Hq, Hkv, D", [
    (66, 33, 2900, 64, 16, 2, 128),      # 256-row blocks, teams of two, two chunks of requests
    (130, 33, 2900, 3, 16, 2, 64),
    (66, 16, 8100, 65, 16, 2, 128),      # 128-row blocks, teams of one
    (130, 9, 8100, 129, 16, 4, 64),
])
def test_paged_batches_that_share_the_work_out(G, oracle, batch, M_max, L_long, long_at, Hq, Hkv, D):
    Ls, Ns = long_batch(batch, M_max, L_long, long_at)
    assert _paged_case(G, oracle, Ls, Ns, Hq, Hkv, D, seed=65)[0] > 0


@pytest.mark.parametrize("batch, M_max, L_long, long_at, Hq, Hkv, D", [(66, 33, 3200, 60, 16, 2, 128), (70, 16, 8100, 0, 16, 2, 128), (130, 9, 8100, 64, 16, 4, 64)])
def test_paged_batches_around_stretches_that_are_cut(G, oracle, batch, M_max, L_long, long_at, Hq, Hkv, D):
    """Stretches of 6 to 13 tiles: up to 8 are not cut, a cut within two of an end moves there, beside one that many workgroups share."""
    Ls, Ns = long_batch(batch, M_max, L_long, long_at)
    Ls = [(180, 222, 230, 255, 256, 270, 289, 320, 350, 383, 400)[r % 11] if r != long_at else l for r, l in enumerate(Ls)]
    assert _paged_case(G, oracle, Ls, Ns, Hq, Hkv, D, seed=67)[0] > 0


@pytest.mark.parametrize("batch, M_max, L_long, Hq, Hkv, D, shared", [
    (64, 33, 3300, 16, 2, 128, True), (65, 33, 3300, 16, 2, 128, True), (130, 33, 3300, 16, 2, 64, True), (65, 16, 8100, 16, 2, 128, True), (130, 16, 8100, 16, 2, 64, True),
    (65, 16, 3300, 16, 2, 128, False), (65, 16, 3300, 16, 4, 64, False)])
def test_paged_batches_around_a_chunk_of_requests(G, oracle, batch, M_max, L_long, Hq, Hkv, D, shared):
    """The work shared out: several small pieces a workgroup, found in the first chunk of 64 requests (kept in LDS) and in later ones, before and behind a long request.  And
    as many requests in a grid of parts."""
    Ls, Ns = long_batch(batch, M_max, L_long, batch - 1)
    Ls[0] = 2500
    assert (_paged_case(G, oracle, Ls, Ns, Hq, Hkv, D, seed=69)[0] > 0) == shared


@pytest.mark.parametrize("batch, M_max, L, Hq, Hkv, D", [(6, 128, 700, 16, 2, 64), (7, 110, 710, 16, 2, 64), (6, 128, 700, 16, 2, 128), (7, 110, 710, 16, 2, 128),
                                                         (2, 8, 5000, 8, 1, 128), (2, 9, 5100, 8, 1, 64)])
def test_paged_batches_of_parts(G, oracle, batch, M_max, L, Hq, Hkv, D):
    """The merge of a short batch's parts: on either side of the number of rows that changes its lanes, and of more parts than it asks for at once."""
    Ls, Ns = [L - 13 * r for r in range(batch)], [M_max - r % 3 for r in range(batch)]
    _paged_case(G, oracle, Ls, Ns, Hq, Hkv, D, seed=68)


@pytest.mark.parametrize("M, L", [(1, 24000), (9, 9000), (130, 24000)])     # many parts; more than 32; the work shared out
def test_paged_batch_of_one(G, oracle, M, L):
    assert (_paged_case(G, oracle, [L], [M], 16, 2, 128, seed=66)[0] > 0) == (M == 130)


def test_paged_bad_requests_are_skipped_where_the_work_is_shared_out(G):
    import torch
    from paper_2605_29727_amd import binding as btv
    Ls, Ns = long_batch(66, 33, 2900, 64)
    bt, nb = synth.paged_layout(5, [l + n for l, n in zip(Ls, Ns)])
    qoff = np.concatenate([[0], np.cumsum(Ns)]).astype(np.int32)
    run = {}
    for bad in (None, 7, 64):
        torch.manual_seed(0)
        Q = torch.randn(int(qoff[-1]), 16, 128, device="cuda", dtype=torch.bfloat16)
        K, V = (torch.randn(nb, synth.PAGE, 2, 128, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        L = np.asarray(Ls, dtype=np.int32)
        if bad is not None:
            L[bad] = -1
        par = G.dev(np.concatenate([np.arange(n) - 1 for n in Ns]).astype(np.int32))
        O = torch.full_like(Q, 7.0)
        ws = btv.alloc_workspace(btv.btv_tree_verify_attn_paged_workspace(66, 33, 2900, 16, 2, 128))
        btv.btv_tree_verify_attn_paged(Q, K, V, G.dev(bt), G.dev(qoff), G.dev(L), par, 33, 2900, O, ws)
        torch.cuda.synchronize()
        assert (btv.btv_workspace_status(ws) != 0) == (bad is not None)
        run[bad] = O.float()
    for bad in (7, 64):
        rows = slice(int(qoff[bad]), int(qoff[bad + 1]))
        assert (run[bad][rows] == 7.0).all()
        run[bad][rows] = run[None][rows]
        assert (run[bad] - run[None]).abs().max() <= TOL_BF16      # (the others' parts may be cut elsewhere)


@pytest.mark.parametrize("seed", range(24))
def test_bf16_random_shapes(G, oracle, seed):
    """Seeded random shapes inside the documented limits (ragged M and L, every GQA ratio up to 16, both head sizes,
    every tree kind), each compared element by element."""
    r = lambda tag, lo, hi: int(synth.integers(1000 + seed, tag, (1,), lo, hi)[0])
    D = (64, 128)[r("D", 0, 1)]
    Hkv = (1, 2, 4, 8)[r("Hkv", 0, 3)]
    Gq = (1, 2, 4, 8, 16)[r("G", 0, 4)]
    M = r("M", 1, 256) if seed % 3 else r("M", 1, 40)
    L = (0, r("L", 1, 31), r("L", 32, 700), r("L", 701, 3000))[r("Lk", 0, 3)]
    kind = KINDS[r("kind", 0, len(KINDS) - 1)]
    if M * Gq * Hkv * (L + M) > 6_000_000:      # keep the oracle's share of the test short
        L = min(L, 600)
    parent = synth.tree_parents(seed, M, kind)
    t = synth.qkv(2000 + seed, M, L, Hkv * Gq, Hkv, D, "bf16", tag="fz")
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
    out = G.run_verify_attn(t, parent, L, "bf16")
    assert np.isfinite(out).all()
    assert np.abs(out - ref).max() <= TOL_BF16, (M, L, Hkv * Gq, Hkv, D, kind, np.abs(out - ref).max())


@pytest.mark.parametrize("value", ["inf", "-inf", "nan"])
@pytest.mark.parametrize("dims", [(64, 700, 8, 2, 128), (70, 1029, 16, 4, 64)])
def test_bf16_non_finite_values_stay_in_their_channel(G, oracle, dims, value):
    """An infinite or NaN value in the cache costs a row that channel alone, into however many parts the keys are cut: the
    partials' scale is the row's largest finite magnitude."""
    M, L, Hq, Hkv, D = dims
    parent = synth.tree_parents(5, M, "random")
    t = synth.qkv(91, M, L, Hq, Hkv, D, "bf16")
    ref = oracle.tree_attn(t["Qf"], t["Kf"], t["Vf"], parent, L)
    t["V"][5, 0, 7] = synth.round_to_dtype(np.array([float(value)]), "bf16")[0][0]
    hit = np.zeros(ref.shape, dtype=bool)
    hit[:, :Hq // Hkv, 7] = True
    for shape in (1, 2, 3):
        for nsplit in (1, 2, 6, 40):
            out = G.run_verify_attn(t, parent, L, "bf16", nsplit=nsplit, shape=shape)
            assert not np.isfinite(out[hit]).any(), (shape, nsplit)
            assert np.abs(out - ref)[~hit].max() <= TOL_BF16, (shape, nsplit)


def test_paged_non_finite_values_stay_in_their_channel(G):
    """The same where a batch's rows come in parts: equal parts of short requests, and parts of an equal share of the work."""
    import torch
    from paper_2605_29727_amd import binding as btv
    for Ls, Ns in (([5000, 300, 2500], [40, 64, 7]), long_batch(66, 33, 2900, 64)):
        bt, nb = synth.paged_layout(5, [l + n for l, n in zip(Ls, Ns)])
        qoff = np.concatenate([[0], np.cumsum(Ns)]).astype(np.int32)
        torch.manual_seed(0)
        Q = torch.randn(int(qoff[-1]), 16, 128, device="cuda", dtype=torch.bfloat16)
        K, V = (torch.randn(nb, synth.PAGE, 2, 128, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        par = G.dev(np.concatenate([np.arange(n) - 1 for n in Ns]).astype(np.int32))
        ws = btv.alloc_workspace(btv.btv_tree_verify_attn_paged_workspace(len(Ls), max(Ns), max(Ls), 16, 2, 128))
        run = []
        for value in (0.0, float("inf")):
            V[:, 3, 0, 7] = value                         # a token of every page
            O = torch.zeros_like(Q)
            btv.btv_tree_verify_attn_paged(Q, K, V, G.dev(bt), G.dev(qoff), G.dev(np.asarray(Ls, dtype=np.int32)), par, max(Ns), max(Ls), O, ws)
            run.append(O.float())
        long_rows = torch.from_numpy(np.repeat(np.asarray(Ls) >= 32, Ns)).cuda()
        assert not run[1][long_rows, :8, 7].isfinite().any()
        for x in run:
            x[:, :8, 7] = 0
        assert (run[0] - run[1]).abs().max() <= 2.0 ** -8       # (two bf16 roundings of values below 2, partials scaled otherwise)
        assert run[0].abs().max() > 0.1
