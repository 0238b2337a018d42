"""A serial replay that fails leaves the results of the batch's last collected
launch as they were."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402


def test_failed_replay_keeps_the_last_results():
    n = 5000
    ctx = D.dsr_init(wg_size=128, lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=8)
    x_np = (np.arange(n) % 101).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(n, dtype=torch.float64, device="cuda")
    regs = [D.fma_chain_region(ctx, 2, [3], [], None, n, x.data_ptr(), y.data_ptr()) for _ in range(2)]
    b = D.dsr_batch_create(ctx, regs)
    D.dsr_batch_launch(b, torch.cuda.current_stream().cuda_stream)
    assert D.dsr_batch_sync(b) == 0
    want = R.fixed75_sum(R.fma_chain(x_np, [3], []))
    assert D.dsr_batch_result(b, 0)[2] == want
    x.add_(1.0)
    torch.cuda.synchronize()
    with pytest.raises(D.DsrError) as e:
        D.dsr_batch_replay_serial(b, [0, 7], [0.0, 0.0])     # region 7 does not exist
    assert e.value.code == D.DSR_E_INVAL
    assert [D.dsr_batch_result(b, k)[2] for k in range(2)] == [want, want]
    D.dsr_batch_replay_serial(b, [0], [0.0])
    new = R.fixed75_sum(R.fma_chain(x_np + 1, [3], []))
    assert [D.dsr_batch_result(b, k)[2] for k in range(2)] == [new, want]
    D.dsr_batch_free(b)
    for r in regs:
        D.dsr_region_free(r)
    D.dsr_destroy(ctx)
