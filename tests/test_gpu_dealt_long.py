"""Fma chains over loops of about 2^30 elements and more, below and above the
longest that is dealt to the waves of all teams, whose last batch is not a full one:
the elements of that batch, and the exact sum, against the oracle."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

TEAMS = 512
LONGEST = (1 << 30) + 1001
TAIL = 4001                                  # inputs that are not zero


@pytest.fixture(scope="module")
def buffers():
    x = torch.zeros(LONGEST, dtype=torch.float32, device="cuda")
    y = torch.zeros(LONGEST, dtype=torch.float64, device="cuda")
    yield x, y
    del x, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("ni,nf,alen,n", [
    (4, 4, 0, LONGEST),                      # a fixed chain, an odd length
    (3, 2, 0, LONGEST - 1),                  # run-time counts
    (2, 1, 250, LONGEST),                    # an array of even length, of odd length
    (2, 1, 251, LONGEST - 994),
    (4, 4, 0, 1 << 30),                      # the longest dealt
    (3, 2, 0, (1 << 30) - 23),
    (2, 1, 251, (1 << 30) - 500),
])
def test_last_batch_past_2_30(buffers, ni, nf, alen, n):
    x, y = buffers
    rs = np.random.RandomState(ni + alen)
    s_i = rs.randint(-1000, 1001, ni).astype(np.int32)
    s_f = rs.randint(0, 1 << 20, nf) * 2.0 ** -20
    arr = rs.randint(0, 1 << 16, alen).astype(np.int32) if alen else None
    tail = (rs.randint(1, 1 << 23, TAIL) * 2.0 ** -23).astype(np.float32)
    x.zero_()
    x[n - TAIL:n] = torch.from_numpy(tail).cuda()
    y.fill_(-1.0)
    ctx = D.dsr_init(wg_size=256, lds_slab_bytes=8192, hbm_slab_bytes=8192, max_teams=TEAMS, master_joins=1)
    img, size = D.fma_chain_frame(s_i, s_f, arr)
    r = D.dsr_region_begin(ctx, TEAMS)
    f = D.dsr_push(r, size, img)
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, n, inp=x.data_ptr(), out=y.data_ptr(), ni=ni, nf=nf, alen=alen)
    D.dsr_pop(r, f)
    D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
    assert D.dsr_region_sync(r) == 0
    want = R.fma_chain(tail, s_i, s_f, arr, n - TAIL)
    assert np.array_equal(y[n - TAIL:n].cpu().numpy(), want)
    # all elements before these have x = 0: y is the array element, or zero
    units = R.fixed75_sum(want)
    if alen:
        turns, rest = divmod(n - TAIL, alen)
        head = turns * int(arr.sum(dtype=np.int64)) + int(arr[:rest].sum(dtype=np.int64))
        units += head << 75
    assert D.dsr_region_reduction(r, 0)[2] == units
    if n < LONGEST:
        assert bool((y[n:] == -1.0).all())
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)
