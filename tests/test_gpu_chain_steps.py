"""The fma chain's int32 steps taken as one step, and when they must not be:
bit for bit against the oracle's step-by-step chain with scalars, inputs and
array elements at and beyond the bounds where one step rounds differently
(partial sums around 2^29, x off the 2^-24 grid, large elements), with
denormal and non-finite inputs, at ragged sizes around a wave's batch."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

I31 = (1 << 31) - 1


def scalars(kind, ni, rs):
    if kind == "small":
        return rs.randint(-(1 << 20), (1 << 20) + 1, ni).astype(np.int32)
    if kind == "at_bound":                    # partial sums reach 2^29 exactly
        s = np.zeros(ni, np.int32)
        s[0] = (1 << 29) - 1
        s[1:2] = 1
        s[2:] = np.tile([-3, 3], ni)[:max(0, ni - 2)]
        return s
    if kind == "over_bound":                  # one partial sum is 2^29 + 1
        s = scalars("at_bound", ni, rs)
        s[0] += 1
        return s
    if kind == "huge":                        # cancelling 31-bit scalars
        return np.tile(np.array([I31, -I31, I31 - 7, -I31 + 3], np.int32), ni)[:ni]
    return np.zeros(ni, np.int32)


def inputs(kind, n, rs):
    x = (rs.randint(-(1 << 23), 1 << 23, n) * 2.0 ** -23).astype(np.float32)
    if kind == "grid24":                      # the finest grid the array bound allows
        x = (rs.randint(-(1 << 24), 1 << 24, n) * 2.0 ** -24).astype(np.float32)
    elif kind == "off_grid":
        x[::5] = rs.standard_normal(len(x[::5])).astype(np.float32) * np.float32(2.0 ** -30)
    elif kind == "denormal":
        x[::3] = np.float32(1e-40)
        x[1::3] = -np.float32(0.0)
    elif kind == "wide":                      # large x on the grid
        x *= np.float32(2.0 ** 9)
    return x


def chain_region(ctx, form, n, teams, s_i, s_f, arr, x, y):
    img, size = D.fma_chain_frame(s_i, s_f, arr)
    ni, nf, alen = len(s_i), len(s_f), 0 if arr is None else len(arr)
    args = {"inp": x.data_ptr(), "out": y.data_ptr(), "ni": ni, "nf": nf, "alen": alen}
    r = D.dsr_region_begin(ctx, teams)
    f = D.dsr_push(r, size, img)
    if form == "list":
        refs = [(f, 0)] + [(f, 24 + 8 * nf + 4 * k) for k in range(ni)] + [(f, 24 + 8 * k) for k in range(nf)]
        if alen:
            refs.append((f, (24 + 8 * nf + 4 * ni + 15) // 16 * 16))
        D.dsr_publish_list(r, refs, D.DSR_BODY_FMA_CHAIN_REFS, n, **args)
    else:
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, n, **args)
    D.dsr_pop(r, f)
    return r


def exact_total(want):
    """The sum in units of 2^-75, or None when a value lies outside the exact-sum
    window (|y| < 2^32, a multiple of 2^-75)."""
    if not (np.all(np.isfinite(want)) and np.all(np.abs(want) < 2.0 ** 32)):
        return None
    units = np.ldexp(want, 75)
    if not np.array_equal(units, np.trunc(units)):
        return None
    return sum(int(v) for v in units)


def check(form, wg, slab, n, teams, s_i, s_f, arr, x_np):
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=slab, hbm_slab_bytes=65536, max_teams=max(8, teams))
    x = torch.from_numpy(x_np).cuda()
    y = torch.full((n,), 5.0, dtype=torch.float64, device="cuda")
    r = chain_region(ctx, "frame" if form == "batch" else form, n, teams, s_i, s_f, arr, x, y)
    stream = torch.cuda.current_stream().cuda_stream
    want = R.fma_chain(x_np, s_i, s_f, arr)
    if form == "batch":
        b = D.dsr_batch_create(ctx, [r])
        D.dsr_batch_launch(b, stream)
        st = D.dsr_batch_sync(b)
        fixed = D.dsr_batch_result(b, 0)[2]
        D.dsr_batch_free(b)
    else:
        D.dsr_launch(r, stream)
        st = D.dsr_region_sync(r)
        fixed = D.dsr_region_reduction(r, 0)[2]
    got = y.cpu().numpy()
    assert np.array_equal(got, want, equal_nan=True)
    assert np.array_equal(np.signbit(got), np.signbit(want)) or not np.all(np.isfinite(want))
    total = exact_total(want)
    assert st == (D.DSR_E_RANGE if total is None else 0)
    if total is not None:
        assert fixed == total
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("form,wg,slab", [("frame", 256, 40960), ("list", 256, 40960), ("frame", 512, 0),
                                          ("frame", 1024, 40960), ("batch", 128, 40960), ("batch", 256, 0)])
@pytest.mark.parametrize("sk", ["small", "at_bound", "over_bound", "huge", "zero"])
@pytest.mark.parametrize("xk", ["plain", "grid24", "off_grid", "denormal", "wide"])
@pytest.mark.parametrize("ni,nf,alen", [(4, 4, 0), (32, 0, 0), (2, 1, 6), (7, 3, 33), (32, 16, 1000)])
def test_steps(form, wg, slab, sk, xk, ni, nf, alen):
    rs = np.random.RandomState(ni * 100 + alen)
    s_i = scalars(sk, ni, rs)
    s_f = (rs.randint(0, 1 << 20, nf) * 2.0 ** -19 - 1.0)
    arr = rs.randint(-(1 << 16), 1 << 16, alen).astype(np.int32) if alen else None
    if alen and sk == "at_bound":
        arr[::2] = I31
    check(form, wg, slab, 4099, 2, s_i, s_f, arr, inputs(xk, 4099, rs))


@pytest.mark.parametrize("ni,nf,alen", [(8, 8, 0), (5, 2, 0), (4, 2, 10)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_inputs(ni, nf, alen, bad):
    """A chain of mixed signs over an infinity is NaN, their sum over it is not:
    the batches that hold one run every step, and the region reports RANGE."""
    rs = np.random.RandomState(5)
    s_i = scalars("small", ni, rs)
    s_i[0], s_i[1] = 3, -1
    arr = rs.randint(0, 100, alen).astype(np.int32) if alen else None
    x = inputs("plain", 3001, rs)
    x[[0, 700, 701, 2999, 3000]] = bad
    for form, wg in (("frame", 256), ("list", 256), ("batch", 128)):
        check(form, wg, 4096, 3001, 3, s_i, rs.randint(1, 9, nf).astype(np.float64), arr, x)


@pytest.mark.parametrize("n", [1, 2, 3, 127, 128, 129, 255, 511, 1023, 1024, 1025, 2047, 3071, 3073, 8191])
@pytest.mark.parametrize("ni,nf,alen", [(1, 0, 0), (16, 16, 0), (3, 2, 0), (6, 3, 14), (6, 3, 1)])
def test_ragged_sizes(n, ni, nf, alen):
    rs = np.random.RandomState(n)
    s_i = scalars("small", ni, rs)
    s_f = rs.randint(0, 1 << 53, nf) * 2.0 ** -52 - 1.0
    arr = rs.randint(0, 1 << 16, alen).astype(np.int32) if alen else None
    for form, wg, slab in (("frame", 64, 4096), ("frame", 256, 4096), ("list", 192, 0), ("batch", 128, 4096),
                           ("frame", 1024, 0)):
        check(form, wg, slab, n, 1 + n // 1500, s_i, s_f, arr, inputs("plain", n, rs))


@pytest.mark.parametrize("wg,teams,joins", [(64, 1, 1), (64, 5, 1), (256, 2, 0), (256, 3, 1), (512, 2, 0)])
@pytest.mark.parametrize("extra", [-1, 0, 1, 2, 511, 1023, 1024, 1025, 5000, 12345])
@pytest.mark.parametrize("ni,nf,alen", [(2, 2, 0), (5, 4, 0), (6, 3, 14), (6, 3, 33)])
def test_dealt_batches(wg, teams, joins, extra, ni, nf, alen):
    """Loops around the length from which their batches are dealt to all teams:
    every element once, ragged ends included; not with frames of their own."""
    waves = teams * (wg // 64 - (0 if joins else 1))
    n = 3 * 1024 * waves + extra
    rs = np.random.RandomState(n)
    s_i = scalars("small", ni, rs)
    s_f = rs.randint(0, 1 << 53, nf) * 2.0 ** -52 - 1.0
    arr = rs.randint(0, 1 << 16, alen).astype(np.int32) if alen else None
    x_np = inputs("plain", n, rs)
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=teams, master_joins=joins)
    x = torch.from_numpy(x_np).cuda()
    want = R.fma_chain(x_np, s_i, s_f, arr)
    for form in ("frame", "list"):
        y = torch.full((n + 1,), 5.0, dtype=torch.float64, device="cuda")
        r = chain_region(ctx, form, n, teams, s_i, s_f, arr, x, y)
        D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
        assert D.dsr_region_sync(r) == 0
        got = y.cpu().numpy()
        assert np.array_equal(got[:n], want) and got[n] == 5.0
        assert D.dsr_region_reduction(r, 0)[2] == exact_total(want)
        D.dsr_region_free(r)
    # a frame per team keeps team t on its own range
    img, size = D.fma_chain_frame(s_i, s_f, arr)
    stride = (size + 15) // 16 * 16
    images, parts = b"", []
    chunk = -(-n // teams)
    chunk = -(-chunk // (1024 if chunk >= 16384 else 64)) * (1024 if chunk >= 16384 else 64)
    for t in range(teams):
        images += D.fma_chain_frame(s_i + t, s_f, arr)[0].ljust(stride, b"\0")
        lo, hi = min(n, t * chunk), min(n, (t + 1) * chunk)
        parts.append(R.fma_chain(x_np[lo:hi], s_i + t, s_f, arr, i0=lo))
    y = torch.full((n,), 5.0, dtype=torch.float64, device="cuda")
    r = D.dsr_region_begin(ctx, teams)
    f = D.dsr_push(r, size, images, init_stride=stride, init_bytes=size)
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, n, inp=x.data_ptr(), out=y.data_ptr(), ni=ni, nf=nf, alen=alen)
    D.dsr_pop(r, f)
    D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
    assert D.dsr_region_sync(r) == 0
    assert np.array_equal(y.cpu().numpy(), np.concatenate(parts))
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("n", [1, 2, 6, 127, 1026])
@pytest.mark.parametrize("alen", [200, 2001])
def test_elements_past_the_end_are_not_judged(n, alen):
    """Array elements that no iteration uses would take the last x out of the
    exact-sum window; every value of the loop itself lies inside it."""
    n = min(n, alen - 50)
    x_np = np.full(n, 0.4375, np.float32)
    arr = np.full(alen, I31, np.int32)
    arr[:n] = 3
    s_i, s_f = np.full(4, I31, np.int32), np.zeros(1)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(n, dtype=torch.float64, device="cuda")
    want = R.fma_chain(x_np, s_i, s_f, arr)
    assert np.abs(want).max() < 2.0 ** 32 < 4 * 0.4375 * I31 + I31
    for wg in (256, 1024):
        ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=16384, hbm_slab_bytes=4096, max_teams=1)
        r = chain_region(ctx, "frame", n, 1, s_i, s_f, arr, x, y)
        D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
        assert D.dsr_region_sync(r) == 0
        assert np.array_equal(y.cpu().numpy(), want)
        D.dsr_region_free(r)
        D.dsr_destroy(ctx)


@pytest.mark.parametrize("alen", [0, 3, 4])
@pytest.mark.parametrize("sign", [1, -1])
def test_bins_of_a_long_stream(sign, alen):
    """The most values one lane may have, at the edge of the window: its bins
    are emptied in time, and the sum stays exact."""
    n = (1 << 21) - 3
    x_np = np.full(n, 1 - 2.0 ** -24, np.float32)
    x_np[::7] = np.float32(2.0 ** -20 + 2.0 ** -43)
    s_i = np.full(4, sign * ((1 << 30) - 1), np.int32)
    s_f = np.array([2.0 ** -52 + 2.0 ** -3])
    arr = np.array([5, -7, 11, 2][:alen], np.int32) if alen else None
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(n, dtype=torch.float64, device="cuda")
    want = R.fma_chain(x_np, s_i, s_f, arr)
    ctx = D.dsr_init(wg_size=64, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=1, master_joins=1)
    r = chain_region(ctx, "frame", n, 1, s_i, s_f, arr, x, y)
    D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
    assert D.dsr_region_sync(r) == 0
    assert np.array_equal(y.cpu().numpy(), want)
    values, counts = np.unique(want, return_counts=True)
    assert D.dsr_region_reduction(r, 0)[2] == sum(exact_total(v) * int(c) for v, c in zip(values.reshape(-1, 1), counts))
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("n", [1, 7, 64, 1026, 5000])
@pytest.mark.parametrize("alen", [0, 8])
@pytest.mark.parametrize("value,ok", [(0.0, True), (2.0 ** -23, True), (2.0 ** -75, True), (3 * 2.0 ** -75, True),
                                      (2.0 ** -76, False), (2.0 ** -60 + 2.0 ** -80, False), (1e-300, False)])
def test_grid_of_small_values(n, alen, value, ok):
    """A value between others that is on the 2^-75 grid or off it: the last
    one, or one inside."""
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=1, master_joins=1)
    arr = np.zeros(alen, np.int32) if alen else None
    for at in {0, n // 2, n - 1}:
        x_np = np.full(n, 1.0, np.float32)
        x_np[at] = 2.0 ** -20
        s_f = np.array([value * 2.0 ** 20])
        y_at = R.fma_chain(x_np, np.zeros(1, np.int32), s_f, arr)
        x = torch.from_numpy(x_np).cuda()
        y = torch.zeros(n, dtype=torch.float64, device="cuda")
        r = chain_region(ctx, "frame", n, 1, np.zeros(1, np.int32), s_f, arr, x, y)
        D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
        st = D.dsr_region_sync(r)
        on = all(float(v * 2.0 ** 75).is_integer() for v in y_at)
        assert ok <= on and st == (0 if on else D.DSR_E_RANGE)
        assert np.array_equal(y.cpu().numpy(), y_at)
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
