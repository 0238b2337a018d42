"""Loops of one region over the same buffers: nothing orders the teams between
two loops, so each team meets the elements of its own range again, and the
region's result is that of the loops one after another.  Half of the teams
start when the others have finished: a loop whose elements went to other teams
would be overtaken by the one before it."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

TEAMS = 512                                  # one wave each, one team per CU at a time
CHUNK = 3 * 1024
N = TEAMS * CHUNK


def chain(r, s, x, y, chunk=0, per_team=False):
    imgs = [D.fma_chain_frame([s + (t if per_team else 0)], [])[0] for t in range(TEAMS if per_team else 1)]
    size = len(imgs[0])
    if per_team:
        f = D.dsr_push(r, size, b"".join(i + bytes(32 - size) for i in imgs), init_stride=32)
    else:
        f = D.dsr_push(r, size, imgs[0])
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, N, inp=x.data_ptr(), out=y.data_ptr(), ni=1, chunk=chunk)
    D.dsr_pop(r, f)


@pytest.mark.parametrize("order", ["per_team_then_shared", "chunk_then_none", "none_then_chunk", "both_none",
                                   "gather_then_chain", "chain_then_affine"])
def test_later_loop_wins(order):
    ctx = D.dsr_init(wg_size=64, lds_slab_bytes=100 << 10, hbm_slab_bytes=4096, max_teams=TEAMS)
    x_np = (np.arange(N) % 4099).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(N, dtype=torch.float64, device="cuda")
    r = D.dsr_region_begin(ctx, TEAMS)
    want_x, want_y = x_np.view(np.int32), R.fma_chain(x_np, [7], [])
    if order == "per_team_then_shared":
        chain(r, 3, x, y, per_team=True)
        chain(r, 7, x, y)
    elif order == "chunk_then_none":
        chain(r, 3, x, y, chunk=CHUNK)
        chain(r, 7, x, y)
    elif order == "none_then_chunk":
        chain(r, 3, x, y)
        chain(r, 7, x, y, chunk=CHUNK)
    elif order == "both_none":
        chain(r, 3, x, y)
        chain(r, 7, x, y)
    elif order == "gather_then_chain":
        # the bits of 1 + i * 2^-23
        f = D.dsr_push(r, 16, D.gather_frame([np.array([0x3F800000] * 4)]))
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, N, out=x.data_ptr(), arrays=1, length=4)
        D.dsr_pop(r, f)
        chain(r, 7, x, y)
        want_x = (0x3F800000 + np.arange(N)).astype(np.int32)
        want_y = R.fma_chain(want_x.view(np.float32), [7], [])
    else:
        chain(r, 7, x, y)
        f = D.dsr_push(r, 24, D.affine_xor_frame(5, 1, 2, 3))
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, N, out=x.data_ptr())
        D.dsr_pop(r, f)
        want_x = R.affine_xor(5, 1, 2, 3, 0, N)[0]
    D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
    assert D.dsr_region_sync(r) == 0
    assert np.array_equal(x.cpu().numpy().view(np.int32), want_x)
    assert np.array_equal(y.cpu().numpy(), want_y)
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)
