"""The kernel instances that hold one kind of body (fixed chains, gathers,
affine loops) against the oracle, bit for bit: programs of one publish and
of several, programs longer than the kernel arguments hold, frames buried
under others, per-team images, frames on chip and in HBM, every workgroup
class, team counts around the arrival tree's edges, ragged sizes."""
import numpy as np
import pytest

import dsr_workloads as W
from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402


def stream():
    return torch.cuda.current_stream().cuda_stream


def run_region(r):
    """Launch twice, so that counters reset by the first launch are used."""
    for _ in range(2):
        D.dsr_launch(r, stream())
        st = D.dsr_region_sync(r)
    return st


@pytest.mark.parametrize("wg", [64, 128, 256, 512, 1024])
@pytest.mark.parametrize("slab", [0, 4096])
@pytest.mark.parametrize("n,teams,publishes", [(0, 2, 1), (1, 1, 1), (1023, 5, 2), (100003, 513, 1), (65536, 512, 5)])
def test_affine(wg, slab, n, teams, publishes):
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=slab, hbm_slab_bytes=4096, max_teams=teams, master_joins=wg == 256)
    vals = [(3 + k, -17 * k, 5 - k, 1 << (20 + k)) for k in range(publishes)]
    outs = [torch.full((n + 1,), -9, dtype=torch.int32, device="cuda") for _ in vals]
    r = D.dsr_region_begin(ctx, teams)
    for v, o in zip(vals, outs):
        f = D.dsr_push(r, 24, D.affine_xor_frame(*v))
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, n, out=o.data_ptr())
        D.dsr_pop(r, f)
    assert run_region(r) == 0
    for k, (v, o) in enumerate(zip(vals, outs)):
        want, total = R.affine_xor(*v, 0, n)
        got = o.cpu().numpy()
        assert np.array_equal(got[:n], want) and got[n] == -9, (k, v)
        assert D.dsr_region_reduction(r, k)[0] == total
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("wg,joins", [(64, 1), (192, 0), (256, 1), (512, 1), (1024, 0)])
@pytest.mark.parametrize("A,length", [(1, 1), (2, 3), (3, 257), (4, 64), (5, 12), (16, 7)])
@pytest.mark.parametrize("n,chunk", [(1, 0), (4099, 514), (30011, 0), (65536, 0)])
def test_gather_shapes(wg, joins, A, length, n, chunk):
    """Flat and nested publishes of one region, the frame on chip or in HBM."""
    arrs = W.cfg3_arrays(A, length)
    frame = 4 * A * length
    teams = 6 if chunk == 0 else -(-n // chunk)
    for slab in (0, 8192):
        ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=slab, hbm_slab_bytes=8192, max_teams=teams, master_joins=joins)
        outs = [torch.full((n + 1,), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
        r = D.dsr_region_begin(ctx, teams)
        f = D.dsr_push(r, frame, D.gather_frame(arrs))
        for o, (body, depth) in zip(outs, ((D.DSR_BODY_GATHER, 0), (D.DSR_BODY_GATHER_NESTED, 2),
                                           (D.DSR_BODY_GATHER_NESTED, 3))):
            D.dsr_publish(r, f, body, n, out=o.data_ptr(), arrays=A, length=length, depth=depth, chunk=chunk)
        D.dsr_pop(r, f)
        assert run_region(r) == 0
        want = R.gather(arrs, 0, n)
        for o in outs:
            got = o.cpu().numpy()
            assert np.array_equal(got[:n], want) and got[n] == -9
        D.dsr_region_free(r)
        D.dsr_destroy(ctx)


@pytest.mark.parametrize("K", [1, 2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("slab", [0, 1024])
def test_chain_programs(K, slab):
    """Two frames of the same chain, the lower one published under the other
    and again after its pop, seven ops; then a frame of its own for each team."""
    n, teams = 5003, 7
    a, x_np = W.cfg2_inputs(K, seed=11, n=n)
    b, _ = W.cfg2_inputs(K, seed=12, n=n, with_x=False)
    x = torch.from_numpy(x_np).cuda()
    ni, nf = len(a.s_i32), len(a.s_f64)
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=slab, hbm_slab_bytes=4096, max_teams=teams)
    ys = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3)]
    r = D.dsr_region_begin(ctx, teams)
    img, size = D.fma_chain_frame(a.s_i32, a.s_f64)
    f0 = D.dsr_push(r, size + 8, img)
    f1 = D.dsr_push(r, size, D.fma_chain_frame(b.s_i32, b.s_f64)[0])
    args = {"inp": x.data_ptr(), "ni": ni, "nf": nf}
    D.dsr_publish(r, f0, D.DSR_BODY_FMA_CHAIN, n, out=ys[0].data_ptr(), **args)
    D.dsr_publish(r, f1, D.DSR_BODY_FMA_CHAIN, n, out=ys[1].data_ptr(), **args)
    D.dsr_pop(r, f1)
    D.dsr_publish(r, f0, D.DSR_BODY_FMA_CHAIN, n, out=ys[2].data_ptr(), **args)
    D.dsr_pop(r, f0)
    assert run_region(r) == 0
    wa, wb = R.fma_chain(x_np, a.s_i32, a.s_f64), R.fma_chain(x_np, b.s_i32, b.s_f64)
    for y, w in zip(ys, (wa, wb, wa)):
        assert np.array_equal(y.cpu().numpy(), w)
    # a second publish of a frame adds to the same shared sum
    ta, tb = R.fixed75_sum(wa), R.fixed75_sum(wb)
    assert [D.dsr_region_reduction(r, k)[2] for k in range(3)] == [ta, tb, 2 * ta]
    D.dsr_region_free(r)
    # per-team images
    stride = (size + 15) // 16 * 16
    chunk = 750
    images, want = b"", np.zeros(n)
    for t in range(teams):
        s_i = a.s_i32 + t
        images += D.fma_chain_frame(s_i, a.s_f64)[0].ljust(stride, b"\0")
        lo, hi = t * chunk, min(n, (t + 1) * chunk)
        want[lo:hi] = R.fma_chain(x_np[lo:hi], s_i, a.s_f64)
    r = D.dsr_region_begin(ctx, teams)
    f = D.dsr_push(r, size, images, init_stride=stride, init_bytes=size)
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, n, out=ys[0].data_ptr(), chunk=chunk, **args)
    D.dsr_pop(r, f)
    assert run_region(r) == 0
    assert np.array_equal(ys[0].cpu().numpy(), want)
    assert D.dsr_region_reduction(r, 0)[2] == R.fixed75_sum(want)
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("body", ["affine", "gather", "chain"])
def test_no_room_for_the_frame(body):
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=0, hbm_slab_bytes=0, max_teams=3)
    out = torch.zeros(256, dtype=torch.float64, device="cuda")
    x = torch.zeros(256, dtype=torch.float32, device="cuda")
    r = D.dsr_region_begin(ctx, 3)
    f = D.dsr_push(r, 64)
    if body == "affine":
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, 256, out=out.data_ptr())
    elif body == "gather":
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, 256, out=out.data_ptr(), arrays=1, length=16)
    else:
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, 256, inp=x.data_ptr(), out=out.data_ptr(), ni=1)
    D.dsr_pop(r, f)
    assert run_region(r) == D.DSR_E_NOMEM
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("depth", [0, 2, 3])
@pytest.mark.parametrize("A,length", [(1, 300), (2, 1001), (3, 4096)])
def test_gather_frames_read_in_place(depth, A, length):
    """HBM frames whose image covers them are read where the image lies: one
    image for all teams, one per team, under another frame and after its pop;
    a frame longer than its image still reads as zeros past it."""
    n, teams, chunk = 20011, 5, 4004
    arrs = W.cfg3_arrays(A, length)
    frame = 4 * A * length
    stride = (frame + 15) // 16 * 16
    body = D.DSR_BODY_GATHER_NESTED if depth else D.DSR_BODY_GATHER
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=0, hbm_slab_bytes=4 * stride, max_teams=teams, flags=D.DSR_F_TRACE)
    outs = [torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(4)]
    per_team = [[a + 7 * t for a in arrs] for t in range(teams)]
    cut = [np.concatenate([arrs[0]] + arrs[1:]).copy()]
    cut[0][A * length - length // 2:] = 0
    args = {"arrays": A, "length": length, "depth": depth, "chunk": chunk}
    r = D.dsr_region_begin(ctx, teams)
    f0 = D.dsr_push(r, frame, D.gather_frame(arrs))
    f1 = D.dsr_push(r, frame, b"".join(D.gather_frame(p).ljust(stride, b"\0") for p in per_team), init_stride=stride,
                    init_bytes=frame)
    f2 = D.dsr_push(r, frame, D.gather_frame(arrs)[:frame - 4 * (length // 2)])
    for f, o in ((f1, outs[0]), (f2, outs[1]), (f0, outs[2])):
        D.dsr_publish(r, f, body, n, out=o.data_ptr(), **args)
    D.dsr_pop(r, f2)
    D.dsr_pop(r, f1)
    D.dsr_publish(r, f0, body, n, out=outs[3].data_ptr(), **args)
    D.dsr_pop(r, f0)
    assert run_region(r) == 0
    whole = R.gather(arrs, 0, n)
    own = np.concatenate([R.gather(per_team[t], t * chunk, min(n, (t + 1) * chunk)) for t in range(teams)])
    short = R.gather([cut[0][j * length:(j + 1) * length] for j in range(A)], 0, n)
    for o, want in zip(outs, (own, short, whole, whole)):
        assert np.array_equal(o.cpu().numpy(), want)
    assert D.dsr_region_trace(r, 1)["placements"] == [("hbm", k * stride, stride) for k in range(3)]
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("wg,joins", [(64, 1), (256, 0), (256, 1), (512, 1), (1024, 0)])
@pytest.mark.parametrize("slab", [0, 16384])
@pytest.mark.parametrize("n,chunk", [(0, 0), (1, 0), (4099, 1026), (50001, 0)])
def test_programs_of_mixed_bodies(wg, joins, slab, n, chunk):
    """One program with every body: chains (fixed, with an array, through a
    list), an affine loop, flat and nested gathers, over nested frames; sums
    added to a frame from several publishes."""
    teams = 4 if chunk == 0 else -(-n // chunk)
    cf, x_np = W.cfg2_inputs(7, seed=3, n=max(n, 1))
    x_np = x_np[:n]
    x = torch.from_numpy(np.ascontiguousarray(np.resize(x_np, max(n, 1)))).cuda()
    arr = (np.arange(33) * 5 - 40).astype(np.int32)
    arrs = W.cfg3_arrays(2, 100)
    img, size = D.fma_chain_frame(cf.s_i32, cf.s_f64, arr)
    img2, size2 = D.fma_chain_frame(cf.s_i32[:2], cf.s_f64[:2])
    ni, nf = len(cf.s_i32), len(cf.s_f64)
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=slab, hbm_slab_bytes=16384, max_teams=max(teams, 1), master_joins=joins)
    ys = [torch.full((n + 1,), 9.0, dtype=torch.float64, device="cuda") for _ in range(4)]
    outs = [torch.full((n + 1,), 9, dtype=torch.int32, device="cuda") for _ in range(3)]
    r = D.dsr_region_begin(ctx, max(teams, 1))
    a = {"inp": x.data_ptr(), "chunk": chunk}
    f0 = D.dsr_push(r, size, img)
    D.dsr_publish(r, f0, D.DSR_BODY_FMA_CHAIN, n, out=ys[0].data_ptr(), ni=ni, nf=nf, alen=33, **a)
    f1 = D.dsr_push(r, 24, D.affine_xor_frame(7, -3, 11, 5))
    D.dsr_publish(r, f1, D.DSR_BODY_AFFINE_XOR, n, out=outs[0].data_ptr(), chunk=chunk)
    f2 = D.dsr_push(r, 800, D.gather_frame(arrs))
    D.dsr_publish(r, f2, D.DSR_BODY_GATHER_NESTED, n, out=outs[1].data_ptr(), arrays=2, length=100, depth=3, chunk=chunk)
    D.dsr_publish(r, f2, D.DSR_BODY_GATHER, n, out=outs[2].data_ptr(), arrays=2, length=100, chunk=chunk)
    D.dsr_pop(r, f2)
    D.dsr_pop(r, f1)
    refs = [(f0, 0)] + [(f0, 24 + 8 * nf + 4 * k) for k in range(ni)] + [(f0, 24 + 8 * k) for k in range(nf)]
    for y, deref in ((ys[1], 0), (ys[2], 1)):
        D.dsr_publish_list(r, refs, D.DSR_BODY_FMA_CHAIN_REFS, n, out=y.data_ptr(), ni=ni, nf=nf, deref=deref, **a)
    f3 = D.dsr_push(r, size2, img2)
    D.dsr_publish(r, f3, D.DSR_BODY_FMA_CHAIN, n, out=ys[3].data_ptr(), ni=2, nf=2, **a)
    D.dsr_pop(r, f3)
    D.dsr_pop(r, f0)
    assert run_region(r) == 0
    want = [R.fma_chain(x_np, cf.s_i32, cf.s_f64, arr), R.fma_chain(x_np, cf.s_i32, cf.s_f64)]
    want += [want[1], R.fma_chain(x_np, cf.s_i32[:2], cf.s_f64[:2])]
    for y, w in zip(ys, want):
        got = y.cpu().numpy()
        assert np.array_equal(got[:n], w) and got[n] == 9.0
    wa, total = R.affine_xor(7, -3, 11, 5, 0, n)
    wg_ = R.gather(arrs, 0, n)
    for o, w in zip(outs, (wa, wg_, wg_)):
        got = o.cpu().numpy()
        assert np.array_equal(got[:n], w) and got[n] == 9
    t = [R.fixed75_sum(w) for w in want]
    assert D.dsr_region_reduction(r, 1)[0] == total
    assert [D.dsr_region_reduction(r, k)[2] for k in (0, 2, 3, 4)] == [t[0], t[0] + t[1], t[0] + 2 * t[1], t[3]]
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("wg", [64, 256, 1024])
@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("image", [1, 252, 255, 256, 257, 260, 515, 2303, 8191, 8192])
def test_frames_copied_to_lds(wg, batch, image):
    """Frames on chip of sizes around whole rounds of the wave's direct
    copies, over bytes that a popped frame left there: one image for all
    teams with zeros behind it, one for each team, above one another."""
    n, teams, chunk, length = 3 * 8300, 3, 8300, 8300
    dirty = np.full(2 * length, -1, np.int32)
    vals = (np.arange(image) * 7 + 1).astype(np.int32)
    stride = (4 * image + 15) // 16 * 16
    own = [np.concatenate([vals + 100 * t, np.zeros(length - image, np.int32)]) for t in range(teams)]
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=2 * (4 * length + 16), hbm_slab_bytes=0, max_teams=teams)
    outs = [torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
    r = D.dsr_region_begin(ctx, teams)
    args = {"arrays": 1, "chunk": chunk}
    f = D.dsr_push(r, 8 * length, dirty.tobytes())
    D.dsr_publish(r, f, D.DSR_BODY_GATHER, n, out=outs[0].data_ptr(), length=2 * length, **args)
    D.dsr_pop(r, f)
    f0 = D.dsr_push(r, 4 * length, vals.tobytes())
    f1 = D.dsr_push(r, 4 * length, b"".join((vals + 100 * t).astype(np.int32).tobytes().ljust(stride, b"\0")
                                            for t in range(teams)), init_stride=stride, init_bytes=4 * image)
    D.dsr_publish(r, f1, D.DSR_BODY_GATHER, n, out=outs[1].data_ptr(), length=length, **args)
    D.dsr_pop(r, f1)
    D.dsr_publish(r, f0, D.DSR_BODY_GATHER_NESTED, n, out=outs[2].data_ptr(), length=length, depth=2, **args)
    D.dsr_pop(r, f0)
    if batch:
        b = D.dsr_batch_create(ctx, [r])
        D.dsr_batch_tune(b, wg_size=wg, lds_slab_bytes=2 * (4 * length + 16))
        for _ in range(2):
            D.dsr_batch_launch(b, stream())
            assert D.dsr_batch_sync(b) == 0
    else:
        assert run_region(r) == 0
    plain = np.concatenate([vals, np.zeros(length - image, np.int32)])
    want = [R.gather([dirty], 0, n), np.concatenate([R.gather([own[t]], t * chunk, (t + 1) * chunk) for t in range(teams)]),
            R.gather([plain], 0, n)]
    for o, w in zip(outs, want):
        assert np.array_equal(o.cpu().numpy(), w)
    if batch:
        D.dsr_batch_free(b)
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("wg,joins", [(64, 1), (192, 0), (512, 1), (1024, 0)])
@pytest.mark.parametrize("image", [127, 255, 256, 300, 1025, 8192, 30011])
@pytest.mark.parametrize("stride_pad", [0, 16])
def test_first_frame_copied_by_all_waves(wg, joins, image, stride_pad):
    """A program's first frame, an image for each team, zeros behind it."""
    teams, chunk = 4, image + 10
    length, n = image + 10, 4 * (image + 10) - 3
    stride = (4 * image + 15) // 16 * 16 + stride_pad
    own = [(np.arange(length) * 3 + 1000 * t).astype(np.int32) * (np.arange(length) < image) for t in range(teams)]
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=(4 * length + 15) // 16 * 16, hbm_slab_bytes=0, max_teams=teams,
                     master_joins=joins, flags=D.DSR_F_TRACE)
    out = torch.full((n,), -9, dtype=torch.int32, device="cuda")
    r = D.dsr_region_begin(ctx, teams)
    f = D.dsr_push(r, 4 * length, b"".join(o[:image].astype(np.int32).tobytes().ljust(stride, b"\1") for o in own),
                   init_stride=stride, init_bytes=4 * image)
    D.dsr_publish(r, f, D.DSR_BODY_GATHER, n, out=out.data_ptr(), arrays=1, length=length, chunk=chunk)
    D.dsr_pop(r, f)
    assert run_region(r) == 0
    want = np.concatenate([R.gather([own[t].astype(np.int32)], t * chunk, min(n, (t + 1) * chunk)) for t in range(teams)])
    assert np.array_equal(out.cpu().numpy(), want)
    assert D.dsr_region_trace(r, 2)["placements"] == [("lds", 0, (4 * length + 15) // 16 * 16)]
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)
