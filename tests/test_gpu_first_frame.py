"""Programs whose first frame is popped, and its place on chip taken by another,
before the first publish; and programs whose first frame is the published one: the
loop reads its own frame, whole, at sizes around a wave's round of loads."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

N, TEAMS = 50000, 300


@pytest.mark.parametrize("wg", [64, 256, 512])
@pytest.mark.parametrize("length", [252, 8192, 8200, 16384])
@pytest.mark.parametrize("body", ["gather", "array"])
@pytest.mark.parametrize("pops", [0, 1, 2])
def test_frame_in_a_popped_frames_place(pops, body, length, wg):
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=4 * length + 2048, hbm_slab_bytes=4096, max_teams=TEAMS)
    arr = (np.arange(length) * 7 + 1).astype(np.int32)
    other = np.full(length, 99999, np.int32)
    x_np = (np.arange(N) % 509).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    out = torch.zeros(N, dtype=torch.int32 if body == "gather" else torch.float64, device="cuda")
    r = D.dsr_region_begin(ctx, TEAMS)
    for _ in range(pops):
        f = D.dsr_push(r, 4 * length, other.tobytes())
        D.dsr_pop(r, f)
    if body == "gather":
        f = D.dsr_push(r, 4 * length, arr.tobytes())
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, N, out=out.data_ptr(), arrays=1, length=length)
        want = R.gather([arr], 0, N)
    else:
        img, size = D.fma_chain_frame([2, 3], [0.5], arr)
        f = D.dsr_push(r, size, img)
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, N, inp=x.data_ptr(), out=out.data_ptr(), ni=2, nf=1, alen=length)
        want = R.fma_chain(x_np, [2, 3], [0.5], arr)
    D.dsr_pop(r, f)
    for _ in range(2):
        out.zero_()
        D.dsr_launch(r, torch.cuda.current_stream().cuda_stream)
        assert D.dsr_region_sync(r) == 0
        assert np.array_equal(out.cpu().numpy(), want)
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)


@pytest.mark.parametrize("nbytes", [512, 1023, 1024, 1025, 1040, 2048])
def test_small_image_in_a_larger_frame(nbytes):
    """Launches without allocation, one after another, of frames around the size
    that is written from the arguments, each with an image of its own."""
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=4)
    out = torch.zeros(1000, dtype=torch.int32, device="cuda")
    rec = torch.zeros(D.RESULT_REC_BYTES, dtype=torch.uint8, device="cuda")
    for k in (1, 1000, -5):
        arr = (np.arange(100) * k).astype(np.int32)
        r = D.dsr_region_begin(ctx, 3)
        f = D.dsr_push(r, nbytes, arr.tobytes())
        whole = np.zeros(nbytes // 4, np.int32)
        whole[:100] = arr
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, 1000, out=out.data_ptr(), arrays=1, length=nbytes // 4)
        D.dsr_pop(r, f)
        D.dsr_launch_static(r, rec.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert D.result_rec(rec.cpu().numpy().tobytes())["status"] == 0
        assert np.array_equal(out.cpu().numpy(), R.gather([whole], 0, 1000))
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
