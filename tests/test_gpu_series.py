"""GPU parity of the matrix-core kernel for short univariate series (sets of kernels of one dilation) against the CPU
oracle, at the sizes where its steps, sets and choice of path can go wrong.  Needs an MI355X."""
import numpy as np
import pytest

from kernels_of import sampled
from paper_2301_08527_amd import rocket
from parity import check_forward

pytestmark = pytest.mark.gpu


def _run(B, L, K, mask, lam=10.0, u8=False):
    import torch
    h, kr = sampled(L + K, K, 1, L)
    rng = np.random.default_rng(L)
    print("series", B, L, K, mask, lam, flush=True)
    if u8:
        import oracle
        raw = rng.integers(0, 256, size=(B, 1, L)).astype(np.uint8)
        out = rocket.rocket_transform_u8(h, torch.from_numpy(raw).cuda(), mask, lam).cpu().numpy()
        x = oracle.znormalize_u8(raw)
    else:
        x = rng.standard_normal((B, 1, L)).astype(np.float32)
        out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), mask, lam).cpu().numpy()
    check_forward(x, kr, out, mask, lam=lam)


@pytest.mark.parametrize("mask", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("B,L,K", [(2, 11, 9), (3, 33, 70), (5, 97, 200)])    # shorter than a step of 32; sets of one to sixteen kernels
def test_every_mask_on_small_series(B, L, K, mask):
    _run(B, L, K, mask)


@pytest.mark.parametrize("B,L,K,mask", [
    (3, 2400, 600, 7), (2, 4900, 300, 3), (2, 9700, 100, 7), (2, 10400, 100, 7),     # longer series, few kernels: the job kernels
    (11, 9700, 9700, 3), (10, 10400, 10400, 2),     # longer than the sets take
    (40, 3000, 3000, 3), (25, 4900, 4900, 7),       # workgroups of eight and of sixteen wavefronts
    (40, 1500, 3000, 3),
    (64, 3000, 300, 7), (40, 8000, 200, 2),
])
def test_long_and_thin(B, L, K, mask):
    _run(B, L, K, mask)


@pytest.mark.parametrize("lam", [-2.0, 0.0, 0.3, 1000.0])
def test_slope_of_any_sign(lam):
    _run(3, 150, 120, 7, lam=lam)


def test_raw_bytes():
    _run(5, 701, 333, 7, u8=True)


def _imported(rng, L, lengths, dilations, padded=True):
    """(handle, oracle arrays) of one-channel kernels of given lengths and dilations"""
    K = len(lengths)
    length, dilation = np.asarray(lengths, np.int32), np.asarray(dilations, np.int32)
    kr = dict(K=K, C=1, L=L, length=length, dilation=dilation,
              padding=((length - 1) // 2 * dilation if padded else np.zeros(K)).astype(np.int32),
              bias=rng.uniform(-1, 1, K).astype(np.float32), n_ch=np.ones(K, np.int32), channels=np.zeros(K, np.int32),
              ch_off=np.arange(K + 1, dtype=np.int64), w_off=np.concatenate([[0], np.cumsum(length)]).astype(np.int64),
              weights=rng.standard_normal(int(length.sum())).astype(np.float32))
    h = rocket.rocket_kernels_import(K, 1, L, length, dilation, kr["padding"], kr["bias"], kr["n_ch"], kr["channels"], kr["weights"])
    return h, kr


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5])
def test_series_shorter_than_a_vector_load(L):
    import torch
    rng = np.random.default_rng(L)
    h, kr = _imported(rng, L, [7, 9, 11] * 7, [1, 1, 2, 1, 3, 1, 1] * 3)
    x = rng.standard_normal((5, 1, L)).astype(np.float32)
    print("short series", L, flush=True)
    out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), 7).cpu().numpy()
    check_forward(x, kr, out, 7)


@pytest.mark.parametrize("what", ["large samples", "small samples", "large weights", "small weights"])
def test_numbers_beyond_the_split(what):
    """Finite samples and weights that three bf16 parts or their products do not carry, in one series of five and in one kernel
    of 16: fp32 arithmetic handles them, so the outputs keep fp32's error, (length + 1) roundings of the sum of magnitudes."""
    import torch
    rng = np.random.default_rng(5)
    B, L, K = 5, 300, 32
    h, kr = _imported(rng, L, [7, 9, 11, 11] * 8, [1, 1, 1, 1, 3, 3, 3, 3] * 4)
    x = rng.standard_normal((B, 1, L)).astype(np.float32)
    w, bias = kr["weights"].copy(), np.zeros(K, np.float32)
    lo, hi = int(kr["w_off"][7]), int(kr["w_off"][8])
    if what == "large samples":
        x[2, 0, ::37] = np.float32(3.4e38) * np.sign(x[2, 0, ::37])
        w *= np.float32(0.01)
    elif what == "small samples":
        x[2] *= np.float32(2.0 ** -120)
    elif what == "large weights":
        w[lo:hi] *= np.float32(3e38) / np.abs(w[lo:hi]).max()
        w[lo] = np.float32(3.4e38)
        x *= np.float32(0.01)
    else:
        w[lo:hi] *= np.float32(2.0 ** -120)
    rocket.rocket_kernels_set_params(h, w, bias)
    kr = dict(kr, weights=w, bias=bias)
    print("beyond the split:", what, flush=True)
    out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), 3).cpu().numpy().astype(np.float64)
    for b in range(B):
        for k in range(K):
            ln, d, p = int(kr["length"][k]), int(kr["dilation"][k]), int(kr["padding"][k])
            n = L + 2 * p - (ln - 1) * d
            xp = np.pad(x[b, 0].astype(np.float64), p)
            wk = w[kr["w_off"][k]:kr["w_off"][k + 1]].astype(np.float64)
            terms = np.stack([wk[j] * xp[j * d:j * d + n] for j in range(ln)])
            y, tol = terms.sum(0), (ln + 1) * 2.0 ** -24 * np.abs(terms).sum(0)
            assert np.abs(out[b, k] - y.max()) <= tol.max(), (b, k, out[b, k], y.max())
            count = np.rint(out[b, K + k] * n)
            assert abs(count - (y > 0).sum()) <= (np.abs(y) <= tol).sum(), (b, k)


@pytest.mark.parametrize("lam,shift,want", [(10.0, 3e38, 1.0), (10.0, -3e38, 0.0), (-2.0, 3e38, 1.0), (0.0, -3e38, 0.0)])
def test_extreme_shift(lam, shift, want):
    """every sigmoid saturates, those of positions that only some kernels of a set have included"""
    import torch
    rng = np.random.default_rng(8)
    h = rocket.rocket_make_kernels(8, 200, 1, 150)
    x = torch.from_numpy(rng.standard_normal((3, 1, 150)).astype(np.float32)).cuda()
    print("extreme shift", lam, shift, flush=True)
    out = rocket.rocket_transform(h, x, 4, lam, shift).cpu().numpy()
    assert np.all(out == np.float32(want))


def test_soft_features_are_as_precise_as_the_job_kernels():
    """The same kernels through the sets (one channel) and through the job kernels (a second channel that none of them reads):
    the sums of sigmoids of the first must not have the larger error.  Over 102,400 features the rms errors scatter by some
    0.3 %; 2 % are allowed.  (One chain of additions per lane had 8 % more.)"""
    import torch
    import oracle
    rng = np.random.default_rng(6)
    B, L, K = 64, 1500, 1600
    h, kr = sampled(17, K, 1, L)
    h2 = rocket.rocket_kernels_import(K, 2, L, kr["length"], kr["dilation"], kr["padding"], kr["bias"], kr["n_ch"], kr["channels"], kr["weights"])
    x = rng.standard_normal((B, 1, L)).astype(np.float32)
    print("precision of soft features", flush=True)
    sets = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), 4).cpu().numpy().astype(np.float64)
    jobs = rocket.rocket_transform(h2, torch.from_numpy(np.concatenate([x, np.zeros_like(x)], axis=1)).cuda(), 4).cpu().numpy().astype(np.float64)
    ref = oracle.transform(x, kr)["softppv"]
    rms = [float(np.sqrt(np.mean((got - ref) ** 2))) for got in (sets, jobs)]
    print("rms error: sets %.4e, job kernels %.4e" % tuple(rms), flush=True)
    assert rms[0] <= 1.02 * rms[1], rms


@pytest.mark.parametrize("L", [97, 500, 1000, 1025, 2000, 3199, 3201])       # 3,200 kernels: up to 3,200 samples in sets
def test_features_depend_on_neither_the_batch_nor_the_other_kernels(L):
    """a series alone, in a small and in a large batch, and through handles that keep many or few of the kernels: the same bits"""
    import torch
    rng = np.random.default_rng(L)
    K, B = 3200, 64
    h = rocket.rocket_make_kernels(8, K, 1, L)
    x = torch.from_numpy(rng.standard_normal((B, 1, L)).astype(np.float32)).cuda()
    print("independent of batch and handle", L, flush=True)
    full = rocket.rocket_transform(h, x, 7).view(B, 3, K)
    for n in (1, 5):
        assert torch.equal(rocket.rocket_transform(h, x[:n].contiguous(), 7).view(n, 3, K), full[:n]), n
    for count in (1600, 150, 1):
        keep = np.sort(rng.choice(K, size=count, replace=False)).astype(np.int32)
        part = rocket.rocket_transform(rocket.rocket_kernels_subset(h, keep), x, 7).view(B, 3, count)
        assert torch.equal(full[:, :, torch.from_numpy(keep.astype(np.int64)).cuda()], part), count


def test_kernels_wider_than_their_series():
    """imported dilations up to and beyond the length, beside ordinary ones: with as much padding as one LDS plane holds, and more"""
    import torch
    rng = np.random.default_rng(12)
    for L, widest in ((40, 1000003), (40, 1410), (40, 2100), (1000, 1330), (1000, 2000)):
        d = [1, 2, 5, L // 6, L // 2, L - 1, L, L + 1, widest, widest // 2] * 3
        h, kr = _imported(rng, L, [7, 9, 11] * 10, d)
        x = rng.standard_normal((3, 1, L)).astype(np.float32)
        print("wide kernels", L, flush=True)
        out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), 7).cpu().numpy()
        check_forward(x, kr, out, 7)


def _launch(kr, L, B):
    """(wavefronts to a workgroup, series to a workgroup, sets to a wavefront) of the sets' launch, from the kernels alone"""
    d, pad, ln = (np.asarray(kr[name], np.int64) for name in ("dilation", "padding", "length"))
    order = np.lexsort((np.arange(len(d)), ln, pad > 0, d))
    sets = [g[i:i + 16] for v in np.unique(d) for g in [order[d[order] == v]] for i in range(0, len(g), 16)]
    first = reach = 0
    for g in sets:
        lo = -((int(pad[g].max()) + 31) // 32 * 32)
        hi = int((L + pad[g] - (ln[g] - 1) * d[g]).max())
        first, reach = min(first, lo), max(reach, lo + (hi - lo + 31) // 32 * 32 + (int(ln[g].max()) - 1) * int(d[g[0]]))
    origin = (-first + 3) // 4 * 4
    nbytes = 8 * ((reach + origin + 3) // 4 * 4)
    waves = 4 if nbytes <= 39936 else 8 if nbytes <= 79872 else 16
    some = min(max(1, 39936 * (waves // 4) // nbytes), 32, B, max(1, len(sets) * B // 16384))
    tasks = -(-B // some) * len(sets)
    return waves, some, 4 if tasks >= 131072 else 2 if tasks >= 65536 else 1


@pytest.mark.parametrize("B,L,K,mask,want,last", [
    (3, 2000, 2000, 7, (4, 1, 1), 1), (2, 3000, 3000, 7, (8, 1, 1), 1), (2, 4900, 4900, 7, (16, 1, 1), 1),
    (302, 200, 3000, 5, (4, 3, 1), 2),            # several series to a workgroup, the last one with fewer
    (1502, 64, 1000, 3, (4, 6, 1), 2),
    (131, 1000, 10000, 3, (4, 2, 1), 1),
    (201, 1000, 10000, 7, (4, 2, 2), 1),          # two and four sets to a wavefront
    (401, 1000, 10000, 3, (4, 2, 4), 1),
])
def test_launch_shapes(B, L, K, mask, want, last):
    import torch
    h, kr = sampled(L + K, K, 1, L)
    waves, some, per = _launch(kr, L, B)
    assert (waves, some, per) == want and (B - 1) % some + 1 == last, (waves, some, per, (B - 1) % some + 1)
    x = np.random.default_rng(L).standard_normal((B, 1, L)).astype(np.float32)
    print("launch shape", B, L, K, mask, want, flush=True)
    out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), mask).cpu().numpy()
    check_forward(x, kr, out, mask, rows=sorted({0, B // 2, B - 2, B - 1}), sel=np.arange(0, K, max(1, K // 600), dtype=np.int32))
