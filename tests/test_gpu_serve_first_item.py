"""The first item of every LDS class.  A class's ring starts out cleared, and the
workgroup that waits for its item 0 may learn of it from another workgroup's
read of the published count, with a ring word in hand that it read before the
item was written: that word must not pass for the item.  The larger class's
first request has several teams and lies in a slot other than 0, so taking
the cleared word for it would run the wrong request's team."""
import time

import numpy as np
import pytest

import dsr_workloads as W
from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402


@pytest.mark.parametrize("start", range(8))
def test_first_item_of_each_class(start):
    n, teams = 4096, 16
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=32768, hbm_slab_bytes=65536, max_teams=2048)
    cf, x_np = W.cfg2_inputs(6, n=n)
    x = torch.from_numpy(x_np).cuda()
    regs, ys, want = [], [], []
    for alen in (0, 5000):                      # the small class, the large one
        arr = (np.arange(alen) % 91).astype(np.int32) if alen else None
        y = torch.zeros(n, dtype=torch.float64, device="cuda")
        regs.append(D.fma_chain_region(ctx, teams, cf.s_i32, cf.s_f64, arr, n, x.data_ptr(), y.data_ptr()))
        ys.append(y)
        want.append(R.fma_chain(x_np, cf.s_i32, cf.s_f64, arr))
    for r in regs:
        D.dsr_region_freeze(r)
    torch.cuda.current_stream().synchronize()
    srv = D.dsr_serve_start(ctx, wg_size=256, slots=4, slot_bytes=40960, max_teams=64, idle_ms=3000,
                            classes=[(4096, 0), (40960, 0)])
    got = []
    try:
        time.sleep(0.002 * start)               # from a grid still starting to one long waiting
        tickets = [D.dsr_serve_submit(srv, r) for r in regs]
        t0 = time.time()
        while len(got) < 2:
            got += D.dsr_serve_poll(srv)
            assert time.time() - t0 < 2.0, "a request did not complete"
    finally:
        D.dsr_serve_stop(srv)
    by = {d["ticket"]: d for d in got}
    for k, t in enumerate(tickets):
        assert by[t]["status"] == 0 and by[t]["fixed"] == [R.fixed75_sum(want[k])]
        assert by[t]["lds_class"] == k
        assert np.array_equal(ys[k].cpu().numpy(), want[k])
    for r in regs:
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
