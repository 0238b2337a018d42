"""Loop buffers that lie at a multiple of one element's size and no more: views
that start one to three elements into an allocation, for every body, alone and in
a batch."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

N, TEAMS = 20003, 3


def region(ctx, body, x, out, x_np):
    r = D.dsr_region_begin(ctx, TEAMS)
    if body == "affine":
        f = D.dsr_push(r, 24, D.affine_xor_frame(3, -7, 11, 5))
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, N, out=out.data_ptr())
        want = R.affine_xor(3, -7, 11, 5, 0, N)[0]
    elif body.startswith("gather"):
        arrs = [np.arange(64) * (k + 3) for k in range(2)]
        f = D.dsr_push(r, 512, D.gather_frame(arrs))
        depth = int(body[-1])
        D.dsr_publish(r, f, D.DSR_BODY_GATHER_NESTED if depth else D.DSR_BODY_GATHER, N, out=out.data_ptr(), arrays=2,
                      length=64, depth=depth)
        want = R.gather(arrs, 0, N)
    else:
        s_i, arr = np.arange(1, 5, dtype=np.int32), np.arange(1000, dtype=np.int32) if body == "array" else None
        img, size = D.fma_chain_frame(s_i, [0.5] * 4, arr)
        f = D.dsr_push(r, size, img)
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, N, inp=x.data_ptr(), out=out.data_ptr(), ni=4, nf=4,
                      alen=0 if arr is None else len(arr))
        want = R.fma_chain(x_np, s_i, [0.5] * 4, arr)
    D.dsr_pop(r, f)
    return r, want


@pytest.mark.parametrize("wg", [128, 512, 1024])
@pytest.mark.parametrize("body", ["affine", "gather0", "gather2", "gather3", "chain", "array"])
def test_element_aligned_buffers(body, wg):
    ctx = D.dsr_init(wg_size=wg, lds_slab_bytes=8192, hbm_slab_bytes=8192, max_teams=64)
    stream = torch.cuda.current_stream().cuda_stream
    x_np = (np.arange(N) % 1013 - 500).astype(np.float32)
    wide = body in ("chain", "array")
    for at in (0, 1, 2, 3):
        x = torch.zeros(N + 8, dtype=torch.float32, device="cuda")[at:at + N]
        x.copy_(torch.from_numpy(x_np))
        whole = torch.full((N + 8,), -9, dtype=torch.float64 if wide else torch.int32, device="cuda")
        out = whole[at:at + N]
        assert out.data_ptr() % 16 == at * out.element_size() % 16 and x.data_ptr() % 16 == 4 * at
        r, want = region(ctx, body, x, out, x_np)
        b = D.dsr_batch_create(ctx, [r])
        for launch, sync, on in ((D.dsr_launch, D.dsr_region_sync, r), (D.dsr_batch_launch, D.dsr_batch_sync, b)):
            whole.fill_(-9)
            launch(on, stream)
            assert sync(on) == 0
            got = whole.cpu().numpy()
            assert np.array_equal(got[at:at + N], want)
            assert (got[:at] == -9).all() and (got[at + N:] == -9).all()
        D.dsr_batch_free(b)
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
