"""Launches without allocation that overlapped, on two streams, spoil no launch
after them: with the workspace's first bytes (where the arrival counters and the
error word lie) holding anything, calls of a process that has used the workspace
from two streams, and graph replays, give the results and the status of their own
region."""
import ctypes as C

import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

N = 20000


def stream():
    return torch.cuda.current_stream().cuda_stream


class Words:
    """`count` 32-bit words of device memory at `ptr`, for torch.as_tensor."""

    def __init__(self, ptr, count):
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<i4", "data": (ptr, False), "version": 3}


def workspace_head():
    p = C.c_void_p()
    assert D.lib().dsr_static_workspace(torch.cuda.current_device(), C.byref(p)) == 0
    return torch.as_tensor(Words(p.value, 640), device="cuda")


LEFT = [1, 7, -1, 0x01010101]


def region(ctx, kind, teams, x, y, out):
    """A region, and (f64, i64, fixed) lists of its results."""
    r = D.dsr_region_begin(ctx, teams)
    if kind == "affine":
        f = D.dsr_push(r, 24, D.affine_xor_frame(5, 1, 2, 3))
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, N, out=out.data_ptr())
        want = {"i64": [R.affine_xor(5, 1, 2, 3, 0, N)[1]]}
    elif kind == "gather":
        f = D.dsr_push(r, 64, D.gather_frame([np.arange(16)]))
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, N, out=out.data_ptr(), arrays=1, length=16)
        want = {"i64": []}
    else:
        img, size = D.fma_chain_frame(np.array([3, -2], np.int32), [0.5])
        f = D.dsr_push(r, size, img)
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, N, inp=x.data_ptr(), out=y.data_ptr(), ni=2, nf=1,
                      schedule=D.DSR_SCHED_DYNAMIC_TAIL if kind == "tail" else D.DSR_SCHED_STATIC)
        want = {"fixed": [R.fixed75_sum(R.fma_chain(x.cpu().numpy(), [3, -2], [0.5]))]}
    D.dsr_pop(r, f)
    return r, want


def two_streams(launch):
    """One launch each on a side stream and on the current one."""
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        launch()
        torch.cuda.synchronize()
    launch()
    torch.cuda.synchronize()


def check(rec, y, out, kind, x_np, want):
    d = D.result_rec(rec.cpu().numpy().tobytes())
    assert d["status"] == 0
    for k, v in want.items():
        assert d[k] == v, k
    if kind in ("chain", "tail"):
        assert np.array_equal(y.cpu().numpy(), R.fma_chain(x_np, [3, -2], [0.5]))


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("wg", [64, 256, 1024])
@pytest.mark.parametrize("kind,teams", [("affine", 1), ("affine", 64), ("affine", 600), ("chain", 1), ("chain", 64),
                                        ("chain", 512), ("chain", 513), ("tail", 8), ("gather", 16)])
def test_any_workspace_contents(kind, teams, wg, graph):
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=4096, hbm_slab_bytes=1024, max_teams=teams)
    x_np = (np.arange(N) % 1013 - 500).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(N, dtype=torch.float64, device="cuda")
    out = torch.zeros(N, dtype=torch.int32, device="cuda")
    rec = torch.zeros(D.RESULT_REC_BYTES, dtype=torch.uint8, device="cuda")
    r, want = region(ctx, kind, teams, x, y, out)
    head = workspace_head()
    launch = lambda: D.dsr_launch_static(r, rec.data_ptr(), stream())  # noqa: E731
    two_streams(launch)
    if graph:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            launch()
        run = g.replay
    else:
        run = launch
    try:
        for left in LEFT:
            head.fill_(left)
            for _ in range(2):
                y.zero_()
                rec.fill_(0xA5)
                torch.cuda.synchronize()
                run()
                torch.cuda.synchronize()
                check(rec, y, out, kind, x_np, want)
    finally:
        head.zero_()
        torch.cuda.synchronize()
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


def test_after_launches_that_overlapped():
    """Regions of different team counts, their programs wholly in the kernel
    arguments and their frames on chip, from two streams at once; then one
    launch at a time."""
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=0, max_teams=64)
    x_np = (np.arange(N) % 1013 - 500).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    bad = torch.full((N,), 1e30, device="cuda")
    y = torch.zeros(N, dtype=torch.float64, device="cuda")
    out = torch.zeros(N, dtype=torch.int32, device="cuda")
    regs = [region(ctx, kind, teams, x, y, out) for kind, teams in (("chain", 64), ("affine", 48), ("chain", 7))]
    fails = region(ctx, "chain", 33, bad, y, out)[0]
    recs = [torch.zeros(D.RESULT_REC_BYTES, dtype=torch.uint8, device="cuda") for _ in range(5)]
    side = torch.cuda.Stream()
    for _ in range(3):
        torch.cuda.synchronize()
        for k in range(100):
            D.dsr_launch_static(regs[k % 3][0], recs[k % 3].data_ptr(), stream())
            D.dsr_launch_static(fails if k % 2 else regs[(k + 1) % 3][0], recs[3 + k % 2].data_ptr(), side.cuda_stream)
        torch.cuda.synchronize()
        for s in (stream(), side.cuda_stream, side.cuda_stream, stream()):
            for (r, want), kind in zip(regs, ("chain", "affine", "chain")):
                recs[0].fill_(0xA5)
                torch.cuda.synchronize()
                D.dsr_launch_static(r, recs[0].data_ptr(), s)
                torch.cuda.synchronize()
                check(recs[0], y, out, kind, x_np, want)
    for r in [fails] + [r for r, _ in regs]:
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
