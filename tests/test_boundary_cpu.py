"""The C-ABI library loads without a GPU, exports every symbol the header declares, and rejects
bad arguments on the host before anything is launched (no compute call is made here)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_29727_amd", "libbastion_tv.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2605_29727_amd import build
        build.build()
    L = C.CDLL(LIB)
    L.btv_last_error.restype = C.c_char_p
    for n in ("btv_tree_build_workspace", "btv_tree_verify_attn_workspace", "btv_tree_verify_attn_paged_workspace",
              "btv_tree_accept_workspace"):
        getattr(L, n).restype = C.c_size_t
    return L


def _declared():
    names = set()
    for f in os.listdir(os.path.join(ROOT, "include")):
        if f.endswith(".h"):
            names |= set(re.findall(r"\b(btv_[a-z_0-9]+)\s*\(", open(os.path.join(ROOT, "include", f)).read()))
    return sorted(names)


def test_every_declared_symbol_is_exported(lib):
    names = _declared()
    assert len(names) >= 12
    for n in names:
        assert getattr(lib, n) is not None


def test_binding_names_match_header():
    from paper_2605_29727_amd import binding
    assert sorted(binding.EXPORTS) == _declared()
    for n in binding.EXPORTS:
        if n != "btv_last_error":
            assert hasattr(binding, n), n


def test_version_and_workspace_queries(lib):
    assert lib.btv_version() >= 1
    assert lib.btv_tree_verify_attn_workspace(64, 8192, 32, 8, 128, 1) > 64 * 8 * 4
    assert lib.btv_tree_verify_attn_workspace(16, 128, 1, 1, 64, 0) >= 256
    assert lib.btv_tree_verify_attn_workspace(0, 128, 1, 1, 64, 0) == 0          # invalid shape -> 0
    assert lib.btv_tree_verify_attn_workspace(16, 128, 3, 2, 64, 0) == 0
    assert lib.btv_tree_verify_attn_fp8kv_workspace(64, 8192, 32, 8, 128) > 64 * 8 * 4
    assert lib.btv_tree_verify_attn_fp8kv_workspace(64, 8192, 32, 8, 64) == 0        # D = 64 is not built for FP8 K/V
    assert lib.btv_tree_verify_attn_paged_fp8kv_workspace(8, 64, 8192, 32, 8, 128) > 0
    assert lib.btv_tree_build_workspace(16, 128256, 64) > 0
    assert lib.btv_tree_build_workspace(17, 128256, 64) == 0
    assert lib.btv_tree_accept_workspace(64, 128256, 0) > 0
    assert lib.btv_tree_accept_workspace(64, 128256, 1) >= 128256 * 4      # two sets of words for each of the walk's workgroups


def test_bad_arguments_are_rejected_on_the_host(lib):
    fake = C.c_void_p(4096)   # never dereferenced: every call below fails validation first
    f0 = C.c_float(0.0)
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 1000, 10, 8, 8, 128, 1, f0, fake, None, C.c_size_t(0), None)
    assert rc == -1 and b"M=1000" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn(None, fake, fake, fake, 16, 10, 8, 8, 128, 1, f0, fake, None, C.c_size_t(0), None)
    assert rc == -1
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 16, 10, 8, 8, 96, 1, f0, fake, None, C.c_size_t(0), None)
    assert rc == -1 and b"D=96" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 16, 10, 8, 8, 128, 7, f0, fake, None, C.c_size_t(0), None)
    assert rc == -1
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 16, 10, 8, 8, 128, 1, f0, fake, None, C.c_size_t(0), None)
    assert rc == -2 and b"workspace" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 16, 10, 8, 8, 128, 1, f0, fake, C.c_void_p(4096 + 8),
                                  C.c_size_t(1 << 20), None)
    assert rc == -2 and b"aligned" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, 16, 10, 8, 8, 128, 1, f0, fake, fake, C.c_size_t(16), None)
    assert rc == -2 and b"too small" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn(C.c_void_p(4096 + 8), fake, fake, fake, 16, 10, 8, 8, 128, 1, f0, fake, None, C.c_size_t(0),
                                  None)
    assert rc == -1 and b"16-byte aligned" in lib.btv_last_error()
    # FP8 KV cache: D = 128 only, positive finite scales, the same shape checks
    one, zero, nan = C.c_float(1.0), C.c_float(0.0), C.c_float(float("nan"))
    rc = lib.btv_tree_verify_attn_fp8kv(fake, fake, fake, one, one, fake, 16, 10, 8, 8, 64, f0, fake, None, C.c_size_t(0), None)
    assert rc == -1 and b"D=64" in lib.btv_last_error()
    for ks, vs in ((zero, one), (one, zero), (nan, one), (one, C.c_float(float("inf"))), (C.c_float(-2.0), one)):
        rc = lib.btv_tree_verify_attn_fp8kv(fake, fake, fake, ks, vs, fake, 16, 10, 8, 8, 128, f0, fake, None,
                                            C.c_size_t(0), None)
        assert rc == -1 and b"scales" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn_fp8kv(fake, fake, fake, one, one, fake, 1000, 10, 8, 8, 128, f0, fake, None,
                                        C.c_size_t(0), None)
    assert rc == -1 and b"M=1000" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn_fp8kv(fake, fake, fake, one, one, fake, 16, 10, 8, 8, 128, f0, fake, None,
                                        C.c_size_t(0), None)
    assert rc == -2 and b"workspace" in lib.btv_last_error()
    rc = lib.btv_tree_verify_attn_paged_fp8kv(fake, fake, fake, one, one, 10, fake, 4, fake, fake, fake, 2, 10, 8, 1 << 20,
                                              8, 8, 128, f0, fake, fake, C.c_size_t(1 << 30), None)
    assert rc == -1 and b"max_blocks" in lib.btv_last_error()
    rc = lib.btv_tree_build(fake, 16, 128256, 1000, fake, fake, None, None, fake, None, fake, C.c_size_t(1 << 30), None)
    assert rc == -1
    rc = lib.btv_tree_build(fake, 99, 128256, 64, fake, fake, None, None, fake, None, fake, C.c_size_t(1 << 30), None)
    assert rc == -1
    rc = lib.btv_tree_accept_greedy(fake, 1, fake, fake, 0, 100, fake, fake, fake, None, fake, C.c_size_t(1 << 20), None)
    assert rc == -1
    rc = lib.btv_tree_accept_stochastic(fake, 0, None, 16, fake, fake, 8, 100, fake, fake, fake, fake, fake,
                                        C.c_size_t(1 << 20), None)
    assert rc == -1
    rc = lib.btv_tree_verify_attn_paged(fake, fake, fake, 10, fake, 4, fake, fake, fake, 2, 10, 8, 1 << 20, 8, 8, 128,
                                        f0, fake, fake, C.c_size_t(1 << 30), None)
    assert rc == -1 and b"max_blocks" in lib.btv_last_error()


def test_host_cost_model_matches_the_oracle(oracle):
    """btv_verify_cost is host arithmetic only (App. E), so it is compared here, without a GPU."""
    from paper_2605_29727_amd import binding as btv
    cfgs = [(64, 8192, 32, 4096, 32, 8, 128, 14336, 128256, 2, 2.5e15, 8e12, 1.0, 0.0),
            (128, 32768, 80, 8192, 64, 8, 128, 28672, 128256, 2, 2.5e15, 8e12, 1.3, 2e-4),
            (1, 2, 1, 2, 1, 1, 2, 3, 5, 1, 56.0, 37.0, 2.0, 0.5),
            (0, 100, 2, 16, 2, 1, 8, 32, 50, 4, 1e9, 1e9, 1.0, 0.0)]
    for cfg in cfgs:
        got, ref = btv.btv_verify_cost(*cfg), oracle.verify_cost(*cfg)
        for k in ("flops", "bytes", "roofline_s", "latency_s"):
            assert got[k] == pytest.approx(ref[k], rel=1e-14), (cfg, k)
    with pytest.raises(btv.BtvError):
        btv.btv_verify_cost(1, 1, 1, 0, 1, 1, 1, 1, 1, 1, 1.0, 1.0)          # zero hidden size
    with pytest.raises(btv.BtvError):
        btv.btv_verify_cost(1, 1, 1, 8, 1, 1, 1, 1, 1, 1, 0.0, 1.0)          # zero peak


def test_host_calibration_matches_the_oracle(oracle):
    """The calibration entry points (Sec. 5.2) and the controller's cost curve (Eq. 6) are host arithmetic only."""
    import numpy as np
    from paper_2605_29727_amd import binding as btv, synth
    for seed in range(3):
        pred = 1e-3 * (1.0 + 10.0 * synth.uniform(seed, "calib_pred", (30,)))
        obs = 1.4 * pred + 3e-4 + 1e-4 * synth.uniform(seed, "calib_noise", (30,))
        got, ref = btv.btv_calib_fit_linear(pred, obs), oracle.calib_fit(pred, obs)
        assert got[0] == pytest.approx(ref[0], rel=1e-11) and got[1] == pytest.approx(ref[1], rel=1e-11)
    with pytest.raises(btv.BtvError):
        btv.btv_calib_fit_linear([2.0, 2.0], [1.0, 3.0])
    with pytest.raises(btv.BtvError):
        btv.btv_calib_fit_linear([2.0], [1.0])
    c_lib = c_orc = 1.0
    for i in range(20):
        obs, pred = 2.0 + 0.1 * i, 1.5 + 0.05 * i
        c_lib, c_orc = btv.btv_calib_ema_update(c_lib, 0.2, obs, pred), oracle.calib_ema(c_orc, 0.2, obs, pred)
        assert c_lib == pytest.approx(c_orc, rel=1e-14)
    with pytest.raises(btv.BtvError):
        btv.btv_calib_ema_update(1.0, 1.5, 1.0, 1.0)                           # alpha outside [0, 1]
    with pytest.raises(btv.BtvError):
        btv.btv_calib_ema_update(1.0, 0.5, 1.0, 0.0)                           # zero prediction
    args = (8192, 32, 4096, 32, 8, 128, 14336, 128256, 2, 2.5e15, 8e12, 1.3, 2e-4, 0.9, 1e-3)
    got, ref = np.array(btv.btv_verify_cost_curve(256, *args)), oracle.cost_curve(256, *args)
    assert np.allclose(got, ref, rtol=1e-14, atol=0)
    assert btv.btv_verify_cost_curve(0, *args) == []
    with pytest.raises(btv.BtvError):
        btv.btv_verify_cost_curve(257, *args)


def _need(lib, fn, *args):
    """What a call needs by its own plan, from the refusal of a workspace of no bytes (nothing is launched)."""
    fake = C.c_void_p(4096)
    a = [fake if x is None else x for x in args]
    assert getattr(lib, fn)(*a, fake, fake, C.c_size_t(0), None) == -2       # BTV_EWORKSPACE
    return int(re.search(rb"too small: 0 < (\d+) bytes", lib.btv_last_error()).group(1))


def _attn_need(lib, M, L, Hq, Hkv, D, dtype):
    return _need(lib, "btv_tree_verify_attn", None, None, None, None, M, L, Hq, Hkv, D, dtype, C.c_float(0.0))


def _attn_fp8_need(lib, M, L, Hq, Hkv):
    one = C.c_float(1.0)
    return _need(lib, "btv_tree_verify_attn_fp8kv", None, None, None, one, one, None, M, L, Hq, Hkv, 128, C.c_float(0.0))


def _attn_tuned_need(lib, M, L, Hq, Hkv, nsplit, shape):
    one = C.c_float(1.0)
    return _need(lib, "btv_tree_verify_attn_tuned", None, None, None, 0, one, one, None, M, L, Hq, Hkv, 128, C.c_float(0.0), nsplit, shape)


# (most nodes, longest context, Hq, Hkv, D): the 8B shape with trees of all sizes (32 nodes at 10208 keys need more than at
# 32768), wide and narrow groups, one head, more heads than workgroups that the chip holds at once
@pytest.mark.parametrize("shape", [(32, 32768, 32, 8, 128), (24, 16384, 32, 8, 128), (16, 16384, 32, 8, 128), (256, 9000, 32, 8, 128), (65, 8192, 64, 8, 128),
                                   (23, 1531, 32, 8, 64), (64, 6000, 16, 1, 128), (33, 4000, 64, 64, 128), (16, 128, 1, 1, 64), (1, 31, 4, 4, 64),
                                   (128, 32768, 28, 4, 128)])
def test_a_workspace_for_the_largest_sizes_serves_all_smaller_ones(lib, shape):
    M, L, Hq, Hkv, D = shape
    for n in ("btv_tree_verify_attn_fp8kv_workspace", "btv_tree_verify_attn_tuned_workspace"):
        getattr(lib, n).restype = C.c_size_t
    trees = sorted({M, 1, max(1, M // 2), max(1, M - 1)} | {m for m in (4, 16, 17, 32, 33, 64, 65, 129) if m < M})
    contexts = [L, 0, max(0, L - 1)] + list(range(16, L, max(1, L // 512)))
    have = lib.btv_tree_verify_attn_workspace(M, L, Hq, Hkv, D, 1)
    assert max(_attn_need(lib, m, l, Hq, Hkv, D, 1) for m in trees for l in contexts) <= have
    assert max(_attn_need(lib, m, l, Hq, Hkv, D, 0) for m in trees for l in contexts[:9]) <= lib.btv_tree_verify_attn_workspace(M, L, Hq, Hkv, D, 0)
    assert have < (1 << 25)                       # (what the built-in array of the allocation-free form holds)
    if D != 128:
        return
    have = lib.btv_tree_verify_attn_fp8kv_workspace(M, L, Hq, Hkv, D)
    assert max(_attn_fp8_need(lib, m, l, Hq, Hkv) for m in trees for l in contexts) <= have
    for nsplit, form in ((0, 1), (0, 3), (7, 0), (32, 2), (100, 1)):
        have = lib.btv_tree_verify_attn_tuned_workspace(M, L, Hq, Hkv, D, 0, nsplit, form)
        assert max(_attn_tuned_need(lib, m, l, Hq, Hkv, nsplit, form) for m in trees for l in contexts[::4]) <= have


@pytest.mark.parametrize("heads", [(32, 8), (16, 2), (4, 1), (64, 16), (28, 4)])
def test_a_workspace_for_the_largest_batch_serves_all_smaller_ones(lib, heads):
    import random
    Hq, Hkv = heads
    rng = random.Random(Hq)
    lib.btv_tree_verify_attn_paged_fp8kv_workspace.restype = C.c_size_t
    one, f0, fake = C.c_float(1.0), C.c_float(0.0), [None] * 3

    def need(fp8, batch, M_max, L_max, D):
        sizes = (1, None, 1 << 20, None, None, None, batch, batch, M_max, L_max, Hq, Hkv, D, f0)
        if fp8:
            return _need(lib, "btv_tree_verify_attn_paged_fp8kv", *fake, one, one, *sizes)
        return _need(lib, "btv_tree_verify_attn_paged", *fake, *sizes)

    for _ in range(300):
        fp8, batch, M_max, L_max = rng.randrange(2), int(2 ** rng.uniform(0, 8)), int(2 ** rng.uniform(0, 8)), int(2 ** rng.uniform(2, 15.3))
        D = 128 if fp8 else rng.choice([64, 128])
        have = (lib.btv_tree_verify_attn_paged_fp8kv_workspace(batch, M_max, L_max, Hq, Hkv, D) if fp8
                else lib.btv_tree_verify_attn_paged_workspace(batch, M_max, L_max, Hq, Hkv, D))
        for k in range(40):
            b, m, l = [x if rng.random() < 0.4 else rng.randint(1, x) for x in (batch, M_max, L_max)]
            assert need(fp8, b, m, l, D) <= have, (fp8, batch, M_max, L_max, D, b, m, l)


def test_a_workspace_smaller_than_a_call_needs_is_refused(lib):
    fake, f0 = C.c_void_p(4096), C.c_float(0.0)
    for M, L in ((64, 8192), (32, 10208), (3, 100)):
        need = _attn_need(lib, M, L, 32, 8, 128, 1)
        rc = lib.btv_tree_verify_attn(fake, fake, fake, fake, M, L, 32, 8, 128, 1, f0, fake, fake, C.c_size_t(need - 1), None)
        assert rc == -2 and b"too small" in lib.btv_last_error()
