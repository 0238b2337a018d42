"""Results written straight to host memory: more regions in flight than one
pinned allocation holds, slots handed on after a free, regions that outlive
their context, relaunches, and a batch's results across relaunches and for
regions with several reductions or none."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402


def stream():
    return torch.cuda.current_stream().cuda_stream


def affine(ctx, k, out, n=300, publishes=1):
    r = D.dsr_region_begin(ctx, 2)
    f = D.dsr_push(r, 24, D.affine_xor_frame(k, 2 * k, 3, k))
    for _ in range(publishes):
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, n, out=out.data_ptr())
    D.dsr_pop(r, f)
    return r, R.affine_xor(k, 2 * k, 3, k, 0, n)[1]


def test_many_regions_in_flight_and_reused_slots():
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=2)
    out = torch.zeros(300, dtype=torch.int32, device="cuda")
    for first in (1, 50):
        regs = [affine(ctx, first + k, out, publishes=1 + k % 3) for k in range(70)]
        for r, _ in regs:
            D.dsr_launch(r, stream())
        for r, _ in regs[::2]:
            D.dsr_launch(r, stream())
        for k, (r, total) in reversed(list(enumerate(regs))):
            assert D.dsr_region_sync(r) == 0
            # later publishes of a frame add to its shared sum
            assert [D.dsr_region_reduction(r, p)[0] for p in range(1 + k % 3)] == [total * (p + 1) for p in range(1 + k % 3)]
        for r, _ in regs:
            D.dsr_region_free(r)
    kept = [affine(ctx, 7 + k, out) for k in range(3)]
    for r, _ in kept:
        D.dsr_launch(r, stream())
        assert D.dsr_region_sync(r) == 0
    D.dsr_destroy(ctx)
    for r, total in kept:
        assert D.dsr_region_reduction(r, 0)[0] == total
        D.dsr_region_free(r)


def test_batch_results_across_launches():
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=64)
    out = torch.zeros(300, dtype=torch.int32, device="cuda")
    regs, totals = [], []
    for k in range(40):
        if k % 5 == 4:                       # a region that reduces nothing
            r = D.dsr_region_begin(ctx, 1)
            f = D.dsr_push(r, 64, D.gather_frame([np.arange(16)]))
            D.dsr_publish(r, f, D.DSR_BODY_GATHER, 64, out=out.data_ptr(), arrays=1, length=16)
            D.dsr_pop(r, f)
            t = None
        else:
            r, t = affine(ctx, k, out, publishes=1 + k % 2)
        regs.append(r)
        totals.append(t)
    b = D.dsr_batch_create(ctx, regs)
    for launch in (D.dsr_batch_launch, D.dsr_batch_launch_each, D.dsr_batch_launch):
        launch(b, stream())
        with pytest.raises(D.DsrError):
            D.dsr_batch_result(b, 0)         # not collected yet
        assert D.dsr_batch_sync(b) == 0
        for k, t in enumerate(totals):
            if t is None:
                with pytest.raises(D.DsrError):
                    D.dsr_batch_result(b, k)
                continue
            for p in range(1 + k % 2):
                i64, _, _, st = D.dsr_batch_result(b, k, p)
                assert (i64, st) == (t * (p + 1), 0)
    D.dsr_batch_free(b)
    for r in regs:
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)


def static_record(region):
    rec = torch.full((D.RESULT_REC_BYTES,), 0xA5, dtype=torch.uint8, device="cuda")
    D.dsr_launch_static(region, rec.data_ptr(), stream())
    return rec


def decode(rec):
    return D.result_rec(rec.cpu().numpy().tobytes())


@pytest.mark.parametrize("wg", [64, 256, 1024])
def test_static_launches_in_a_row(wg):
    """No launch clears the workspace for the next: regions of different team
    counts (around the arrival tree's edge), bodies and lengths, one that runs
    out of memory and one out of the exact window among them, queued without a
    wait in between; every record holds its own region's results alone."""
    teams_max = 600
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=512, hbm_slab_bytes=4096, max_teams=teams_max)
    x_np = (np.arange(3000) % 97 - 48).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(3000, dtype=torch.float64, device="cuda")
    out = torch.zeros(3000, dtype=torch.int32, device="cuda")
    wide = torch.full((3000,), 1e30, dtype=torch.float32, device="cuda")
    regs, want = [], []
    for k, teams in enumerate((600, 1, 513, 512, 3, 64)):
        r = D.dsr_region_begin(ctx, teams)
        f = D.dsr_push(r, 24, D.affine_xor_frame(k, 1, 2, 3))
        for _ in range(1 + k % 3):
            D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, 3000, out=out.data_ptr())
        D.dsr_pop(r, f)
        total = R.affine_xor(k, 1, 2, 3, 0, 3000)[1]
        regs.append(r)
        want.append((0, [total * (p + 1) for p in range(1 + k % 3)], None))
        s_i = np.arange(1, 2 + k, dtype=np.int32)
        img, size = D.fma_chain_frame(s_i, [0.5])
        for src, st in ((x, 0), (wide, D.DSR_E_RANGE)):
            r = D.dsr_region_begin(ctx, teams)
            f = D.dsr_push(r, size, img)
            D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, 3000, inp=src.data_ptr(), out=y.data_ptr(), ni=1 + k, nf=1)
            D.dsr_pop(r, f)
            regs.append(r)
            want.append((st, None, R.fixed75_sum(R.fma_chain(x_np, s_i, [0.5]))))
        r = D.dsr_region_begin(ctx, min(teams, 64))
        f = D.dsr_push(r, 8192)                  # fits neither stack
        D.dsr_publish(r, f, D.DSR_BODY_GATHER if k % 2 else D.DSR_BODY_AFFINE_XOR, 3000, out=out.data_ptr(),
                      arrays=1, length=1000)
        D.dsr_pop(r, f)
        regs.append(r)
        want.append((D.DSR_E_NOMEM, None, None))
    for _ in range(2):
        recs = [static_record(r) for r in regs]
        for rec, (st, i64, fixed) in zip(recs, want):
            d = decode(rec)
            assert d["status"] == st
            if i64 is not None:
                assert d["i64"] == i64
            if st == 0 and fixed is not None:
                assert d["fixed"] == [fixed]
    for r in regs:
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)


def test_static_launch_in_a_graph():
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=64)
    x_np = (np.arange(20000) % 1013 - 500).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(20000, dtype=torch.float64, device="cuda")
    rec = torch.zeros(D.RESULT_REC_BYTES, dtype=torch.uint8, device="cuda")
    r = D.dsr_region_begin(ctx, 16)
    img, size = D.fma_chain_frame(np.array([3, -2, 7, 1], np.int32), [0.5, 0.25, 0.125, 2.0])
    f = D.dsr_push(r, size, img)
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, 20000, inp=x.data_ptr(), out=y.data_ptr(), ni=4, nf=4)
    D.dsr_pop(r, f)
    D.dsr_launch_static(r, rec.data_ptr(), stream())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        D.dsr_launch_static(r, rec.data_ptr(), stream())
    want = R.fma_chain(x_np, np.array([3, -2, 7, 1], np.int32), [0.5, 0.25, 0.125, 2.0])
    for k in range(4):
        y.zero_()
        rec.zero_()
        x.add_(0.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        d = decode(rec)
        assert np.array_equal(y.cpu().numpy(), want)
        assert d["status"] == 0 and d["fixed"] == [R.fixed75_sum(want)]
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)
