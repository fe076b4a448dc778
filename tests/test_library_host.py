"""Host-side checks of the C-ABI library that need no GPU: it loads, exports
every symbol declared in include/rocket.h, samples kernels bit-identically to
the oracle's separately written sampler, and validates its arguments."""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
from paper_2301_08527_amd import rocket

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "rocket.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(rocket_[a-z0-9_]+)\s*\(", header))
    assert declared == set(rocket.EXPORTS)
    lib = rocket.load_library()
    for name in declared:
        assert hasattr(lib, name), name
    assert isinstance(lib.rocket_transform, ctypes._CFuncPtr)


@pytest.mark.parametrize("seed,K,C,L", [
    (2000, 500, 1, 512), (2001, 2000, 1, 1000), (2002, 3000, 20, 50000),
    (2004, 1500, 20, 200000), (0, 64, 3, 11), (2**64 - 1, 64, 9, 4097), (12345, 200, 40, 333),
])
def test_sampler_bit_exact_against_oracle(seed, K, C, L):
    kr = oracle.sample_kernels(seed, K, C, L)
    h = rocket.rocket_make_kernels(seed, K, C, L)
    v = rocket.rocket_kernels_view_get(h)
    assert (v["K"], v["C"], v["L"]) == (K, C, L)
    for name in ("length", "dilation", "padding", "n_ch", "channels", "ch_off", "w_off"):
        assert np.array_equal(v[name], kr[name]), name
    assert np.array_equal(v["bias"].view(np.uint32), kr["bias"].view(np.uint32))
    assert np.array_equal(v["weights"].view(np.uint32), kr["weights"].view(np.uint32))
    h.free()


def test_import_round_trip_and_set_params():
    kr = oracle.sample_kernels(5, 50, 6, 300)
    h = rocket.rocket_kernels_import(50, 6, 300, kr["length"], kr["dilation"], kr["padding"], kr["bias"],
                                     kr["n_ch"], kr["channels"], kr["weights"])
    v = rocket.rocket_kernels_view_get(h)
    for name in ("length", "dilation", "padding", "n_ch", "channels", "bias", "weights", "ch_off", "w_off"):
        assert np.array_equal(v[name], kr[name]), name
    rocket.rocket_kernels_set_params(h, weights=kr["weights"] * 2, bias=None)
    v2 = rocket.rocket_kernels_view_get(h)
    assert np.array_equal(v2["weights"], kr["weights"] * 2) and np.array_equal(v2["bias"], kr["bias"])
    with pytest.raises(rocket.RocketError):
        rocket.rocket_kernels_set_params(h, weights=np.full_like(kr["weights"], np.nan))
    # a rejected call changes nothing, whichever array is the bad one
    bad_bias = kr["bias"].copy()
    bad_bias[3] = np.inf
    with pytest.raises(rocket.RocketError):
        rocket.rocket_kernels_set_params(h, weights=kr["weights"] * 3, bias=bad_bias)
    v3 = rocket.rocket_kernels_view_get(h)
    assert np.array_equal(v3["weights"], kr["weights"] * 2) and np.array_equal(v3["bias"], kr["bias"])
    fma, outs = rocket.rocket_work_per_series(h)
    n = 300 + 2 * kr["padding"].astype(np.int64) - (kr["length"] - 1) * kr["dilation"]
    assert outs == n.sum() and fma == (n * kr["n_ch"] * kr["length"]).sum()


def test_import_rejects_bad_kernels():
    kr = oracle.sample_kernels(6, 10, 4, 200)

    def attempt(**changes):
        a = {k: np.array(v, copy=True) for k, v in kr.items() if isinstance(v, np.ndarray)}
        for name, (idx, val) in changes.items():
            a[name][idx] = val
        return rocket.rocket_kernels_import(10, 4, 200, a["length"], a["dilation"], a["padding"], a["bias"],
                                            a["n_ch"], a["channels"], a["weights"])

    attempt().free()
    bad = [dict(length=(0, 8)), dict(dilation=(1, 0)), dict(padding=(2, 1 + int(kr["padding"][2]))),
           dict(dilation=(3, 1000), padding=(3, 0)), dict(channels=(0, 4)), dict(channels=(0, -1)),
           dict(bias=(0, np.inf)), dict(weights=(5, np.nan))]
    for ch in bad:
        with pytest.raises(rocket.RocketError) as e:
            attempt(**ch)
        assert e.value.code == rocket.ROCKET_ESHAPE
    # a repeated channel inside one kernel
    k2 = int(np.argmax(kr["n_ch"] >= 2))
    lo = int(kr["ch_off"][k2])
    with pytest.raises(rocket.RocketError):
        attempt(channels=(lo + 1, int(kr["channels"][lo])))


def test_argument_validation_without_gpu():
    with pytest.raises(rocket.RocketError) as e:
        rocket.rocket_make_kernels(1, 0, 1, 100)
    assert e.value.code == rocket.ROCKET_EINVAL and "K" in str(e.value)
    with pytest.raises(rocket.RocketError):
        rocket.rocket_make_kernels(1, 10, 1, 10)      # L < 11
    with pytest.raises(rocket.RocketError):
        rocket.rocket_make_kernels(1, 10, 0, 100)
    h = rocket.rocket_make_kernels(1, 10, 2, 100)
    assert rocket.rocket_num_features(0) == 0 and rocket.rocket_num_features(8) == 0
    assert [rocket.rocket_num_features(m) for m in range(1, 8)] == [1, 1, 2, 1, 2, 2, 3]
    assert rocket.rocket_workspace_bytes(h, 0, 3) == 0 and rocket.rocket_workspace_bytes(h, 4, 0) == 0
    fwd = rocket.rocket_workspace_bytes(h, 4, 3)
    bwd = rocket.rocket_workspace_bytes(h, 4, 5, backward=True)
    assert fwd >= 4 * 2 * 100 * 4 and fwd % 256 == 0 and bwd > fwd
    lib = rocket.load_library()
    # compute entry points reject bad arguments before touching the GPU
    dummy = ctypes.c_void_p(256)
    assert lib.rocket_transform(None, dummy, 1, 3, 10.0, -3.0, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_transform(h.handle, None, 1, 3, 10.0, -3.0, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_transform(h.handle, dummy, 0, 3, 10.0, -3.0, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_transform(h.handle, dummy, 1, 9, 10.0, -3.0, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_transform(h.handle, dummy, 1, 3, float("nan"), -3.0, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_transform(h.handle, dummy, 1, 3, 10.0, -3.0, dummy, dummy, 16, None) == rocket.ROCKET_EWORKSPACE
    assert lib.rocket_transform(h.handle, dummy, 1, 3, 10.0, -3.0, dummy, None, 1 << 30, None) == rocket.ROCKET_EWORKSPACE
    assert "workspace" in rocket.rocket_last_error()
    assert lib.rocket_transform(h.handle, dummy, 1, 3, 10.0, -3.0, None, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    # backward needs the softPPV plane
    assert lib.rocket_soft_ppv_backward(h.handle, dummy, 1, 3, dummy, 10.0, -3.0, 0, dummy, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    assert lib.rocket_soft_ppv_backward(h.handle, dummy, 1, 4, dummy, 10.0, -3.0, 1, dummy, dummy, dummy, 1 << 30, None) == rocket.ROCKET_EINVAL
    # the 8-bit, inference and training entry points validate the same way, before any GPU call
    E = rocket.ROCKET_EINVAL
    assert lib.rocket_transform_u8(h.handle, dummy, 0, 3, 10.0, -3.0, dummy, dummy, 1 << 30, None) == E
    assert lib.rocket_transform_u8(h.handle, None, 1, 3, 10.0, -3.0, dummy, dummy, 1 << 30, None) == E
    assert lib.rocket_soft_ppv_backward_u8(h.handle, dummy, 1, 3, dummy, 10.0, -3.0, 0, dummy, dummy, dummy, 1 << 30, None) == E
    assert lib.rocket_infer(h.handle, dummy, 0, 1, 3, 10.0, -3.0, None, dummy, dummy, dummy, dummy, 1 << 30, None) == E
    assert lib.rocket_infer(h.handle, dummy, 1, 0, 3, 10.0, -3.0, dummy, dummy, dummy, dummy, dummy, 1 << 30, None) == E
    assert lib.rocket_mse_grad(None, dummy, dummy, 4, 10, dummy, dummy, None) == E
    assert lib.rocket_mse_grad(dummy, dummy, dummy, 0, 10, dummy, dummy, None) == E
    assert lib.rocket_mse_grad(dummy, dummy, dummy, 70000, 10, dummy, dummy, None) == E
    assert lib.rocket_sgd_update(h.handle, None, dummy, 0.1, 0, None) == E
    assert lib.rocket_sgd_update(h.handle, dummy, dummy, float("inf"), 0, None) == E
    assert lib.rocket_train_workspace_bytes(h.handle, 0, 5) == 0
    need = lib.rocket_train_workspace_bytes(h.handle, 4, 5)
    assert need > rocket.rocket_workspace_bytes(h, 4, 5, backward=True) and need % 256 == 0
    args = (h.handle, dummy, 0, 4, 3, 10.0, -3.0, dummy, dummy, dummy, 0.1, 0, dummy, dummy, 1 << 40, None)
    assert lib.rocket_train_step(*args) == E                       # mask without softPPV
    args = (h.handle, dummy, 0, 4, 5, 10.0, -3.0, dummy, dummy, dummy, 0.1, 0, dummy, dummy, 16, None)
    assert lib.rocket_train_step(*args) == rocket.ROCKET_EWORKSPACE
    assert lib.rocket_kernels_subset(h.handle, None, 1, ctypes.byref(ctypes.c_void_p())) == E
    # the entry point that allocates nothing: bad sizes, then a handle whose parameters were never uploaded
    assert lib.rocket_transform_noalloc(None, dummy, 1, 3, 10.0, -3.0, dummy, None) == E
    assert lib.rocket_transform_noalloc(h.handle, dummy, 0, 3, 10.0, -3.0, dummy, None) == E
    assert lib.rocket_transform_noalloc(h.handle, dummy, 1, 8, 10.0, -3.0, dummy, None) == E
    assert lib.rocket_transform_noalloc(h.handle, dummy, 1, 3, 10.0, -3.0, dummy, None) == E
    assert "upload" in rocket.rocket_last_error()
    assert rocket.rocket_workspace_bytes(h, 100000, 3) > 64 << 20
    assert lib.rocket_transform_noalloc(h.handle, dummy, 100000, 3, 10.0, -3.0, dummy, None) == rocket.ROCKET_EWORKSPACE
    assert lib.rocket_jobs_view_get(h.handle, None, None, None, None, None, None) == E
    assert lib.rocket_calibrate_fma(None, None) == E
    assert lib.rocket_calibrate_units(None, 10, None) == E
    assert lib.rocket_calibrate_units((ctypes.c_double * 4)(), 4, None) == E      # too few slots
    h.free()
    rocket.load_library().rocket_free_kernels(None)


def test_minirocket_kernel_set_without_gpu():
    """host-only: the predetermined kernel set equals the oracle's, and bad arguments are errors"""
    kr = oracle.minirocket_kernels(9, 6, 20, 3000)
    h = rocket.rocket_minirocket_kernels(9, 6, 20, 3000)
    v = rocket.rocket_kernels_view_get(h)
    for name in ("length", "dilation", "padding", "n_ch", "channels", "ch_off", "w_off", "weights", "bias"):
        assert np.array_equal(v[name], kr[name]), name
    for bad in ((0, 20, 3000), (6, 0, 3000), (6, 20, 8)):
        with pytest.raises(rocket.RocketError):
            rocket.rocket_minirocket_kernels(9, *bad)
    lib = rocket.load_library()
    dummy = ctypes.c_void_p(256)
    assert rocket.rocket_minirocket_fit_workspace_bytes(h, 0) == 0
    need = rocket.rocket_minirocket_fit_workspace_bytes(h, 4)
    assert need % 256 == 0 and need > 4 * 20 * 3000 * 4
    E = rocket.ROCKET_EINVAL
    assert lib.rocket_minirocket_fit_bias(None, dummy, 4, 1, dummy, 1 << 40, None) == E
    assert lib.rocket_minirocket_fit_bias(h.handle, None, 4, 1, dummy, 1 << 40, None) == E
    assert lib.rocket_minirocket_fit_bias(h.handle, dummy, 0, 1, dummy, 1 << 40, None) == E
    assert lib.rocket_minirocket_fit_bias(h.handle, dummy, 4, 1, dummy, 16, None) == rocket.ROCKET_EWORKSPACE


@pytest.mark.parametrize("groups,C,L", [(1, 1, 9), (4, 2, 10), (9, 3, 73), (20, 4, 4105), (40, 20, 50000), (12, 9, 200001)])
def test_minirocket_plan_covers_every_position_once(groups, C, L):
    """host-only: the work items of the group kernel cover every output position of every group exactly once,
    and none stages more than the 4,864 samples of its LDS planes"""
    h = rocket.rocket_minirocket_kernels(17, groups, C, L)
    v = rocket.rocket_kernels_view_get(h)
    items = rocket.rocket_minirocket_jobs_view_get(h)
    assert np.all(items[:, 7] == 0) and set(items[:, 1].tolist()) <= {0, 1}
    kinds = set()
    for g in range(groups):
        d, p = int(v["dilation"][84 * g]), int(v["padding"][84 * g])
        n = L + 2 * p - 8 * d
        seen = np.zeros(n, np.int32)
        mine = items[items[:, 0] == g]
        assert len(mine) >= 1
        for _, mode, first, count, col0, width, rows, _ in mine.tolist():
            assert width % 64 == 0 and width >= 64
            kinds.add(mode)
            if mode == 0:
                assert d <= 256 and 1 <= count <= width < count + 64 and width + 8 * d <= 4864 and rows == 1
                seen[first:first + count] += 1
            else:
                assert d > 256 and width <= 256 and rows >= 1 and (rows + 8) * width <= 4864 and col0 < d
                cols = np.arange(col0, min(col0 + width, d))
                t = (first + np.arange(rows))[:, None] * d + cols[None, :]
                t = t[t < n]
                assert t.size > 0                  # no work item without work
                np.add.at(seen, t, 1)
        assert np.all(seen == 1), (g, d, p, int(seen.min()), int(seen.max()))
    if L >= 50000:
        assert kinds == {0, 1}
    plain = rocket.rocket_make_kernels(1, 84, C, max(L, 11))
    with pytest.raises(rocket.RocketError):
        rocket.rocket_minirocket_jobs_view_get(plain)
    assert rocket.rocket_minirocket_workspace_bytes(plain, 2) == 0 and rocket.rocket_minirocket_workspace_bytes(h, 2) > 0


def test_subset_keeps_the_chosen_kernels():
    """host-only: rocket_kernels_subset copies the selected kernels, in the given order"""
    h = rocket.rocket_make_kernels(3, 50, 6, 900)
    kr = rocket.rocket_kernels_view_get(h)
    idx = np.array([7, 0, 49, 7], np.int32)
    hs = rocket.rocket_kernels_subset(h, idx)
    ks = rocket.rocket_kernels_view_get(hs)
    assert len(ks["length"]) == 4
    for i, k in enumerate(idx):
        for name in ("length", "dilation", "padding", "n_ch", "bias"):
            assert ks[name][i] == kr[name][k]
        assert np.array_equal(ks["weights"][ks["w_off"][i]:ks["w_off"][i + 1]], kr["weights"][kr["w_off"][k]:kr["w_off"][k + 1]])
        assert np.array_equal(ks["channels"][ks["ch_off"][i]:ks["ch_off"][i + 1]], kr["channels"][kr["ch_off"][k]:kr["ch_off"][k + 1]])
    with pytest.raises(rocket.RocketError):
        rocket.rocket_kernels_subset(h, np.array([50], np.int32))


@pytest.mark.parametrize("K,C,L", [(300, 3, 700), (400, 20, 50000), (200, 1, 8193), (300, 5, 200001)])
def test_job_plan_partitions_every_kernel(K, C, L):
    """host-only: the jobs of a kernel cover its full rows exactly once, in order, exactly one
    of them owns the partial last row, and tile boundaries are whole bands"""
    h = rocket.rocket_make_kernels(11, K, C, L)
    kr = rocket.rocket_kernels_view_get(h)
    jobs = rocket.rocket_jobs_view_get(h)
    n = L + 2 * kr["padding"].astype(np.int64) - (kr["length"].astype(np.int64) - 1) * kr["dilation"]
    rows = n // kr["dilation"]
    assert set(jobs["kernel"].tolist()) == set(range(K))
    total_positions = 0
    for k in range(K):
        mine = np.nonzero(jobs["kernel"] == k)[0]
        r0, r1, fl = jobs["row0"][mine], jobs["row1"][mine], jobs["flags"][mine]
        order = np.argsort(r0, kind="stable")
        r0, r1, fl = r0[order], r1[order], fl[order]
        assert r0[0] == 0 and r1[-1] == rows[k]
        assert np.all(r0[1:] == r1[:-1])                       # contiguous, no overlap
        assert np.all(r1[:-1] > r0[:-1]) and r1[-1] >= r0[-1]  # only a last tile may hold no full row
        assert (fl & 1).sum() == 1 and fl[-1] & 1              # the last tile owns the partial last row
        assert np.all(((fl & 2) != 0) == (len(mine) == 1))
        d = int(kr["dilation"][k])
        if len(mine) > 1:
            unit = 17 * (256 // d) if d < 16 else 32          # whole LDS chunks / whole 32-row bands
            assert np.all(r1[:-1] % unit == 0)
            assert np.all((r1[:-1] - r0[:-1]) * d >= 16384)    # tiles of at least 16,384 positions
        total_positions += int(n[k])
    fma, outs = rocket.rocket_work_per_series(h)
    assert outs == total_positions
