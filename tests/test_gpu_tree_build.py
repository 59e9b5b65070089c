"""Bit-exact parity of the HIP best-first tree build with the CPU oracle (topology, tokens, depth, rho bits)."""
import numpy as np
import pytest

from paper_2605_29727_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _check(G, oracle, marg, N):
    """The library's own choice of expansion, then each of the two expansions forced."""
    ref = oracle.tree_build(marg, N)
    for algo in (0, 1, 2):
        got = G.run_tree_build(marg, N, algo)
        assert got["n"] == ref["n"], algo
        for k in ("parent", "token", "depth"):
            assert np.array_equal(got[k], ref[k]), (k, algo)
        assert np.array_equal(got["rho"].view(np.uint32), ref["rho"].view(np.uint32)), algo
        assert abs(got["ahat"] - ref["ahat"]) <= 1e-5 * ref["ahat"], algo
    return ref


def test_config1(G, oracle):
    w = synth.C1
    _check(G, oracle, synth.marginals(w.seed, w.B, w.V, w.marg_sigma), w.N)


@pytest.mark.parametrize("sigma,seed", [(3.0, 2), (5.0, 3), (1.0, 4), (8.0, 9)])
@pytest.mark.parametrize("N", [1, 16, 64, 100, 256])
def test_full_vocabulary(G, oracle, sigma, seed, N):
    marg = synth.marginals(seed, 16, 128256, sigma)
    ref = _check(G, oracle, marg, N)
    if sigma == 1.0 and N == 256:
        assert ref["depth"].max() == 1          # flat marginals: the tree is a depth-1 star
    if sigma >= 5.0 and N >= 64:
        assert ref["depth"].max() >= 3          # sharp marginals: deep chains


@pytest.mark.parametrize("B,V,N", [(1, 1, 1), (2, 3, 12), (4, 64, 200), (16, 2049, 256), (3, 5000, 77), (16, 300, 256)])
def test_small_and_ragged_vocabularies(G, oracle, B, V, N):
    for seed in range(3):
        _check(G, oracle, synth.marginals(50 + seed, B, V, 2.5), N)


@pytest.mark.parametrize("V", [1, 2, 15, 16, 17, 32, 33, 64, 65, 127, 128, 129, 256, 257, 512, 513])
@pytest.mark.parametrize("B", [1, 3, 4, 5, 16])
def test_small_vocabularies_whole_and_by_position(G, oracle, B, V):
    """Where one workgroup takes all positions (up to 512 marginals, both sizes rounded up to powers of two), where a position's marginals are
    ranked whole (up to 256) and where they have a bound; probabilities of few distinct values too, so that most of them tie."""
    for N in (1, 20, 256):
        marg = synth.marginals(90, B, V, 2.0)
        _check(G, oracle, marg, N)
        _check(G, oracle, np.round(marg * 24).astype(np.float32) / 32, N)


@pytest.mark.parametrize("V", [4097, 8192, 16390, 40001, 131072])
def test_marginals_at_any_float(G, oracle, V):
    """Rows, and the first of them, that begin 4, 8 or 12 bytes past a multiple of 16."""
    import torch
    from paper_2605_29727_amd import binding as btv
    B, N = 5, 40
    marg = synth.marginals(91, B, V, 3.0)
    ref = oracle.tree_build(marg, N)
    for shift in (0, 1, 2, 3):
        room = torch.zeros(B * V + shift, device="cuda")
        room[shift:] = torch.from_numpy(marg.reshape(-1)).cuda()
        out = {k: torch.zeros(N, dtype=torch.int32, device="cuda") for k in ("parent", "token", "depth")}
        rho, n_out, ahat = torch.zeros(N, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda")
        btv.btv_tree_build(room[shift:].view(B, V), N, out["parent"], out["token"], out["depth"], rho, n_out, ahat,
                           btv.alloc_workspace(btv.btv_tree_build_workspace(B, V, N)))
        for k in out:
            assert np.array_equal(out[k].cpu().numpy(), ref[k]), (k, shift)
        assert np.array_equal(rho.cpu().numpy().view(np.uint32), ref["rho"].view(np.uint32)), shift


@pytest.mark.parametrize("extra", [-1, 0, 1, 2])
@pytest.mark.parametrize("N", [63, 127, 255, 256])
def test_number_of_candidates_around_the_ways_of_ranking_them(G, oracle, N, extra):
    """N + extra tokens of one probability's bin above all others: they are what the ranking orders, by 16 or 8 lanes a key or by bins."""
    marg = np.full((4, 6000), 1e-6, dtype=np.float32)
    rng = np.random.default_rng(N + extra)
    for row in marg:
        row[rng.permutation(6000)[:N + extra]] = (1.0 + rng.integers(0, 3, N + extra) / 64.0).astype(np.float32) / 512
    _check(G, oracle, marg, N)


@pytest.mark.parametrize("V", [255, 256, 257, 4096, 4097, 16384, 16387, 65536, 65541, 131072, 131075])
def test_vocabularies_around_the_slot_sizes(G, oracle, V):
    """The ranking sees a row as slots whose size follows the vocabulary's: single marginals up to 4096, then 4 to 32 of them."""
    for seed, (B, N, sigma) in enumerate([(3, 256, 2.5), (16, 64, 6.0), (2, 1, 1.0)]):
        _check(G, oracle, synth.marginals(70 + seed, B, V, sigma), N)


@pytest.mark.parametrize("V", [4097, 4098, 4099, 5119, 5121, 6146, 16383, 20481, 65539, 70001, 131069])
def test_rows_that_end_with_their_best_tokens(G, oracle, V):
    """The last tokens of a row, in a chunk whose loads are moved back into the row, are the largest, in rising and falling order and tied."""
    rng = np.random.default_rng(V)
    marg = (rng.random((3, V)) * 1e-5).astype(np.float32)
    marg[0, -9:] = np.linspace(0.05, 0.2, 9)
    marg[1, -9:] = np.linspace(0.2, 0.05, 9)
    marg[2, -9:] = 0.1
    _check(G, oracle, marg, 24)


@pytest.mark.parametrize("N", [1, 2, 40, 97, 256])
@pytest.mark.parametrize("step", [-1, 0, 1])
def test_star_and_its_first_deeper_node(G, oracle, N, step):
    """The best second-level node just below the N-th best first token, level with it (the lesser depth comes first), just above."""
    q0 = (0.5 * 0.97 ** np.arange(300)).astype(np.float32)
    q1 = np.full(300, 1e-4, dtype=np.float32)
    q1[7] = q0[N - 1] * np.float32(2)
    q1[7] = np.nextafter(q1[7], np.float32(step)) if step else q1[7]
    _check(G, oracle, np.stack([q0, q1, q1]), N)


def test_more_candidates_than_the_sweep_holds(G, oracle):
    """Marginals near 1 for many tokens (no probabilities, but finite and at most 1) make every level of the lattice larger than
    the sweep's lists: the frontier loop takes over, whichever expansion was asked for."""
    marg = np.sort(synth.uniform(5, "near_one", (16, 40)), axis=1)[:, ::-1]
    marg = (1.0 - 1e-3 * (1.0 - marg)).astype(np.float32)
    for N in (40, 256):
        _check(G, oracle, marg, N)


def test_ties_zeros_one_hot_and_budget_beyond_lattice(G, oracle):
    cases = [
        np.full((4, 8), 0.125, dtype=np.float32),                                   # everything ties
        np.array([[0.0, 1.0, 0.0], [0.5, 0.5, 0.0], [0.0, 0.0, 1.0]], dtype=np.float32),
        np.array([[0.5, 0.25, 0.25], [0.75, 0.25, 0.0]], dtype=np.float32),
        np.array([[0.6, 0.4]], dtype=np.float32),                                   # lattice of 2 prefixes
    ]
    for marg in cases:
        for N in (1, 2, 5, 12, 40, 256):
            _check(G, oracle, marg, N)
    # many exact ties in a large vocabulary: probabilities quantised to multiples of 2^-12
    marg = synth.marginals(77, 8, 4096, 2.0)
    marg = (np.floor(marg * 4096) / 4096).astype(np.float32)
    _check(G, oracle, marg, 256)


def test_tiny_scores_keep_their_bits(G, oracle):
    """Products deep in the tree reach the subnormal range; rho must still match bit for bit."""
    marg = np.full((16, 4), 1e-3, dtype=np.float32)
    marg[:, 0] = 3e-3
    _check(G, oracle, marg, 256)


def test_more_candidates_than_the_selection_keeps(G, oracle):
    """Rows whose probabilities tie heavily, or grow with the token id, defeat the cheap bound of the top-K
    selection (most of the row stays a candidate): the exact byte-wise selection must take over."""
    V = 20000
    uniform = np.full((3, V), 1.0 / V, dtype=np.float32)                         # every key ties on the probability
    ramp = np.tile(np.arange(1, V + 1, dtype=np.float64), (2, 1))                 # best tokens at the highest ids
    ramp = (ramp / ramp.sum(axis=1, keepdims=True)).astype(np.float32)
    steps = np.repeat(np.arange(1, 6, dtype=np.float64), V // 5)[None, :]        # five plateaus of 4000 equal values
    steps = np.tile(steps / steps.sum(), (4, 1)).astype(np.float32)
    mixed = synth.marginals(91, 4, V, 2.0)
    mixed[1] = uniform[0]                                                         # only one row takes the slow path
    for marg in (uniform, ramp, steps, mixed):
        for N in (7, 64, 256):
            _check(G, oracle, marg, N)


@pytest.mark.parametrize("N", [5, 64, 97, 256])
def test_wide_fans_along_the_chain(G, oracle, N):
    """What the thin levels of the sweep do with fans: one and several nodes of a level with more than 4 and more than 68 children above the
    threshold, with and without ties, down to a threshold that scores lie on exactly (powers of two are edges of its bins)."""
    B, V = 16, 400
    flat = np.tile(1e-3 * 0.9995 ** np.arange(V), (B, 1))
    one = flat.copy(); one[:, 17] = 0.6                                       # a chain with many near-equal siblings at every depth
    two = flat.copy(); two[:, 17] = 0.5; two[:, 18] = 0.4999                  # 2^depth chains
    tied = np.full((B, V), 2.0 ** -9); tied[:, 3] = 0.5                       # all siblings tie, on an edge
    halves = np.tile(2.0 ** -np.arange(1.0, 11.0), (B, 1))                    # every score a power of two
    first = one.copy(); first[0] = 0.002 * 0.998 ** np.arange(V)             # a wide first level, confident from there on
    for marg in (one, two, tied, halves, first):
        _check(G, oracle, marg.astype(np.float32), N)


@pytest.mark.parametrize("N", [5, 64, 97, 256])
def test_sweep_from_a_confident_chain(G, oracle, N):
    """The same on either side of the confidence from which the sweep starts from the chain, and with more wide fans than one
    wavefront goes through."""
    B, V = 16, 400
    flat = np.tile(1e-3 * 0.9995 ** np.arange(V), (B, 1))
    two = flat.copy(); two[:, 17] = 0.55; two[:, 18] = 0.4399                 # 2^depth chains, each node with a wide fan
    tied = np.full((B, V), 2.0 ** -9); tied[:, 3] = 0.75                      # all siblings tie, on an edge
    halves = np.tile(2.0 ** -np.arange(10.0), (B, 1))                         # every score a power of two, the chain's all one
    below, above = flat.copy(), flat.copy()
    below[:, 5] = 0.547; above[:, 5] = 0.548                                  # a second node of probability a little less, and more, than 0.3
    for marg in (two, tied, halves, below, above):
        _check(G, oracle, marg.astype(np.float32), N)
