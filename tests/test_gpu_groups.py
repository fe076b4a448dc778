"""Transform and backward pass over groups of interleaved short series (needs an MI355X): against the oracle, against the same kernels one
series at a time, and the backward pass's rule for exact ties."""
import numpy as np
import pytest

import oracle
from paper_2301_08527_amd import rocket
from parity import check_backward, check_forward

pytestmark = pytest.mark.gpu


def _gpu(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _raw(rng, shape):
    """8-bit samples and the floats that the entry points make of them"""
    x = rng.integers(0, 256, size=shape, dtype=np.uint8)
    v = x.astype(np.float64)
    return x, ((v - v.mean(axis=-1, keepdims=True)) / v.std(axis=-1, keepdims=True)).astype(np.float32)


def _width(h, B, C, L, mask, backward):
    """How many series of a batch lie interleaved in the copy that a pass leaves in its workspace (1: no groups)."""
    import torch
    x = torch.randn((B, C, L), device="cuda")
    x[-1, 0, 0], x[-1, 0, 1] = 123.25, 321.5        # neighbours in the series
    ws = torch.zeros(rocket.rocket_workspace_bytes(h, B, mask, backward), dtype=torch.uint8, device="cuda")
    if backward:
        gout = torch.zeros((B, rocket.rocket_num_features(mask) * h.K), device="cuda")
        rocket.rocket_soft_ppv_backward(h, x, mask, gout, 10.0, -3.0, bool(mask & 1), workspace=ws)
    else:
        rocket.rocket_transform(h, x, mask, workspace=ws)
    words = ws.view(torch.float32)
    at = [(words == v).nonzero().flatten().tolist() for v in (123.25, 321.5)]
    assert len(at[0]) == 1 and len(at[1]) == 1
    return at[1][0] - at[0][0]


# Widths that the rule gives (_width looks at what a call does), as (width, series of the first group).  Narrow groups reach
# the staged small dilations (width x dilation below 16) and bands of 32 rows, wide ones of short series the few-rows strips only; first
# groups of one series (and an empty place), as wide as the others and narrower, with all their series and with idle ones (3 of 4, 13 of 16).
CASES = [
    (9, 2, 2000, 4000, (2, 1)), (13, 3, 700, 3000, (4, 1)), (27, 2, 400, 2500, (8, 3)), (13, 2, 128, 6000, (16, 13)), (70, 1, 100, 4000, (32, 6)),
    (200, 1, 40, 6000, (64, 8)), (130, 1, 25, 4000, (64, 2)), (3, 1, 61, 9000, (4, 3)), (200, 9, 90, 700, (16, 8)), (6, 1, 11, 3000, (8, 6)),
    (60, 1, 12000, 1000, (2, 2)),      # beyond the one-wavefront kernels' series
    (149, 18, 1263, 600, (4, 1)),      # 38 groups: the first six one after the other, each on all XCDs
    (200, 20, 1200, 400, (4, 4)),      # 50: two by kernels, then 40 side by side and eight more
]


@pytest.mark.parametrize("B,C,L,K,groups", CASES)
@pytest.mark.parametrize("u8", [False, True])
def test_groups_against_the_oracle(B, C, L, K, groups, u8):
    import torch
    rng = np.random.default_rng(L + B)
    if u8:
        raw, x = _raw(rng, (B, C, L))
        entry, xd = rocket.rocket_soft_ppv_backward_u8, _gpu(raw)
    else:
        x = rng.standard_normal((B, C, L)).astype(np.float32)
        entry, xd = rocket.rocket_soft_ppv_backward, _gpu(x)
    h = rocket.rocket_make_kernels(L, K, C, L)
    kr = rocket.rocket_kernels_view_get(h)
    g = rng.standard_normal((B, 2 * K)).astype(np.float32)
    sel = np.arange(0, K, max(1, K // 150), dtype=np.int32)
    print("groups", B, C, L, K, groups, "u8" if u8 else "f32", flush=True)
    assert _width(h, B, C, L, 5, True) == groups[0] and (B - 1) % groups[0] + 1 == groups[1]
    gw, gb = entry(h, xd, 4, _gpu(g[:, K:]), 4.0, -3.0, False)
    check_backward(x, kr, gw.cpu().numpy(), gb.cpu().numpy(), g[:, K:], None, 4.0, -3.0, sel=sel)
    gw, gb = entry(h, xd, 5, _gpu(g), 4.0, -3.0, True)
    sel = sel[oracle.transform(x, kr, sel=sel)["gap"].min(axis=0) > 1e-4]      # the largest output is the same one in fp32 and fp64
    assert len(sel) > 20
    check_backward(x, kr, gw.cpu().numpy(), gb.cpu().numpy(), g[:, K:], g[:, :K], 4.0, -3.0, sel=sel)
    again = entry(h, xd, 5, _gpu(g), 4.0, -3.0, True)
    assert torch.equal(again[0], gw) and torch.equal(again[1], gb)


@pytest.mark.parametrize("B,C,L,K,groups", CASES)
def test_groups_equal_single_series(B, C, L, K, groups):
    """gradients add up over the batch: every kernel, with both planes, where no series alone is a group"""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn((B, C, L), generator=gen, device="cuda")
    gout = torch.randn((B, 2 * K), generator=gen, device="cuda")
    h = rocket.rocket_make_kernels(L + 1, K, C, L)
    print("groups and single series", B, C, L, K, groups, flush=True)
    assert _width(h, B, C, L, 5, True) == groups[0] and _width(h, 1, C, L, 5, True) == 1
    ws = torch.full((rocket.rocket_workspace_bytes(h, B, 5, True),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever nothing writes
    whole = rocket.rocket_soft_ppv_backward(h, x, 5, gout, 10.0, -3.0, True, workspace=ws)
    parts = [rocket.rocket_soft_ppv_backward(h, x[b:b + 1].contiguous(), 5, gout[b:b + 1].contiguous(), 10.0, -3.0, True) for b in range(B)]
    for i in (0, 1):
        a, want = whole[i].double(), sum(p[i].double() for p in parts)
        # fp32 sums of the same terms in another order: 2^-24 sqrt(B L terms) of sums around their rms, tenfold
        assert float((a - want).norm()) <= 1e-5 * float(want.norm())
        assert float((a - want).abs().max()) <= 1e-4 * float(want.abs().max())


@pytest.mark.parametrize("B,L", [(9, 1500), (24, 700), (30, 150)])
def test_exact_ties_in_groups(B, L):
    """small-integer samples and one non-zero tap per channel: all sums are exact, nearly every largest output is attained many times, and
    the first position of each series must get its gradient"""
    import torch
    rng = np.random.default_rng(L)
    C = 3
    spec = [(ln, d, p) for ln in (7, 9, 11) for d in sorted({1, 2, 3, 5, 7, 8, 15, 16, 31, 40, (L - 1) // (ln - 1)}) if d * (ln - 1) < L
            for p in (False, True)] * 20
    K = len(spec)
    length, dil = (np.array([s[i] for s in spec], np.int32) for i in (0, 1))
    pad = np.array([(s[0] - 1) * s[1] // 2 if s[2] else 0 for s in spec], np.int32)
    nch = rng.integers(1, C + 1, K).astype(np.int32)
    chans = np.concatenate([rng.permutation(C)[:m] for m in nch]).astype(np.int32)
    rows = []
    for k in range(K):
        for _ in range(nch[k]):
            row = np.zeros(length[k], np.float32)
            row[rng.integers(0, length[k])] = float(rng.choice([1.0, 2.0, -1.0]))
            rows.append(row)
    h = rocket.rocket_kernels_import(K, C, L, length, dil, pad, rng.integers(-2, 3, K).astype(np.float32) * 0.25, nch, chans, np.concatenate(rows))
    kr = rocket.rocket_kernels_view_get(h)
    x = rng.integers(-2, 3, size=(B, C, L)).astype(np.float32)
    g = np.zeros((B, 2 * K), np.float32)
    g[:, :K] = rng.integers(1, 4, size=(B, K)).astype(np.float32)
    print("ties in groups", B, L, flush=True)
    assert _width(h, B, C, L, 5, True) > 1
    gw, gb = rocket.rocket_soft_ppv_backward(h, _gpu(x), 5, _gpu(g), 10.0, -3.0, True)
    torch.cuda.synchronize()
    gw_ref, gb_ref = oracle.backward(x, kr, g[:, K:].astype(np.float64), g[:, :K].astype(np.float64), lam=10.0, shift=-3.0)
    assert np.array_equal(gw.cpu().numpy().astype(np.float64), gw_ref)
    assert np.array_equal(gb.cpu().numpy().astype(np.float64), gb_ref)


# (width, series of the first group) of a transform without softPPV; one series alone is never a group
AHEAD = [(28, 15, 134, 2351, (8, 4)), (149, 3, 166, 3236, (32, 21)), (3, 2, 200, 9000, (4, 3)), (20, 18, 1263, 4822, (4, 4)), (9, 4, 600, 6000, (4, 1)),
         (130, 2, 60, 4000, (64, 2)), (100, 4, 600, 200, (2, 2)), (149, 18, 1263, 600, (4, 1)), (200, 20, 1200, 400, (4, 4))]


@pytest.mark.parametrize("B,C,L,K,groups", AHEAD)
@pytest.mark.parametrize("u8", [False, True])
def test_features_of_groups(B, C, L, K, groups, u8):
    """the same bits as one series at a time, and within the oracle's tolerance; without allocation too"""
    import torch
    rng = np.random.default_rng(L)
    if u8:
        raw, x = _raw(rng, (B, C, L))
        entry, xd = rocket.rocket_transform_u8, _gpu(raw)
    else:
        x = rng.standard_normal((B, C, L)).astype(np.float32)
        entry, xd = rocket.rocket_transform, _gpu(x)
    h = rocket.rocket_make_kernels(L, K, C, L)
    print("features of groups", B, C, L, K, groups, "u8" if u8 else "f32", flush=True)
    assert all(_width(h, B, C, L, mask, False) == groups[0] for mask in (1, 2, 3)) and (B - 1) % groups[0] + 1 == groups[1]
    assert _width(h, 1, C, L, 3, False) == 1 and _width(h, B, C, L, 7, False) == 1
    alone = torch.cat([entry(h, xd[b:b + 1].contiguous(), 3) for b in range(B)])
    ws = torch.full((rocket.rocket_workspace_bytes(h, B, 3, False),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever nothing writes
    both = entry(h, xd, 3, workspace=ws)
    assert torch.equal(both, alone)
    assert torch.equal(entry(h, xd, 1), alone[:, :K]) and torch.equal(entry(h, xd, 2), alone[:, K:])
    kr = rocket.rocket_kernels_view_get(h)
    check_forward(x, kr, both.cpu().numpy(), 3, rows=sorted({0, B // 2, B - 1}), sel=np.arange(0, K, max(1, K // 200), dtype=np.int32))
    if not u8 and rocket.rocket_workspace_bytes(h, B, 3, False) <= 64 << 20:
        import ctypes
        out = torch.full_like(both, float("nan"))
        rc = rocket.load_library().rocket_transform_noalloc(h.handle, xd.data_ptr(), B, 3, 10.0, -3.0, out.data_ptr(),
                                                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == rocket.ROCKET_OK and torch.equal(out, both)


@pytest.mark.parametrize("C,L,K,B", [(14, 2857, 1724, 24), (2, 3000, 2000, 9), (5, 8192, 700, 40), (1, 1500, 300, 120), (3, 1030, 1100, 40)])
def test_four_wavefronts_give_the_same_bits(C, L, K, B):
    """one series alone takes four wavefronts to a kernel, a batch one or groups (tests/sanitize/groups_driver.cpp has the routes): all their features"""
    import torch
    x = np.random.default_rng(K).standard_normal((B, C, L)).astype(np.float32)
    h = rocket.rocket_make_kernels(K, K, C, L)
    xd = _gpu(x)
    print("four wavefronts", C, L, K, B, flush=True)
    for mask in (1, 2, 3):
        batch = rocket.rocket_transform(h, xd, mask)
        for b in (0, B // 2, B - 1):
            assert torch.equal(rocket.rocket_transform(h, xd[b:b + 1].contiguous(), mask), batch[b:b + 1]), (mask, b)
    kr = rocket.rocket_kernels_view_get(h)
    check_forward(x[:1], kr, rocket.rocket_transform(h, xd[:1].contiguous(), 3).cpu().numpy(), 3, sel=np.arange(0, K, max(1, K // 200), dtype=np.int32))


def test_groups_keep_their_series_apart():
    """infinite, undefined and huge samples in some series of a group leave the others' features as they are"""
    import torch
    B, C, L, K = 30, 3, 300, 2500
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((B, C, L), generator=gen, device="cuda")
    x[3, :, 70] = float("nan")
    x[5, 1, 10] = float("inf")
    x[12, 0] = 3e38
    h = rocket.rocket_make_kernels(6, K, C, L)
    print("groups keep their series apart", flush=True)
    assert _width(h, B, C, L, 3, False) > 1
    both = rocket.rocket_transform(h, x, 3)
    alone = torch.cat([rocket.rocket_transform(h, x[b:b + 1].contiguous(), 3) for b in range(B)])
    assert torch.equal(torch.nan_to_num(both, nan=-7.0), torch.nan_to_num(alone, nan=-7.0))
    clean = [b for b in range(B) if b not in (3, 5, 12)]
    assert torch.isfinite(both[clean]).all()


def test_groups_in_a_graph():
    """copy and kernel of a transform and of a backward pass are captured and replayed on new samples"""
    import torch
    B, C, L, K = 40, 3, 400, 1500
    gen = torch.Generator(device="cuda").manual_seed(5)
    h = rocket.rocket_make_kernels(7, K, C, L)
    x = torch.randn((B, C, L), generator=gen, device="cuda")
    gout = torch.randn((B, 2 * K), generator=gen, device="cuda")
    out = torch.empty((B, 2 * K), device="cuda")
    gw, gb = torch.empty(h.total_weights, device="cuda"), torch.empty(K, device="cuda")
    ws = torch.empty(max(rocket.rocket_workspace_bytes(h, B, 5, True), rocket.rocket_workspace_bytes(h, B, 3, False)), dtype=torch.uint8, device="cuda")

    def step():
        rocket.rocket_transform(h, x, 3, out=out, workspace=ws)
        rocket.rocket_soft_ppv_backward(h, x, 5, gout, 10.0, -3.0, True, grad_w=gw, grad_b=gb, workspace=ws)

    print("groups in a graph", flush=True)
    assert _width(h, B, C, L, 3, False) > 1 and _width(h, B, C, L, 5, True) > 1
    step()
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for _ in range(3):
        x.copy_(torch.randn((B, C, L), generator=gen, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (out, gw, gb)]
        step()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, (out, gw, gb)))
