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
