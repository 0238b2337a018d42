"""A team's shared sum read by a later loop of its region: the loops that leave
it and that read it run on the team's own range, [t * chunk, (t + 1) * chunk)
with chunk = ceil(n / teams) rounded up to 64, however long they are.  Also
loops of one region over the same buffers, which every team has to run in
program order on its own range."""
import numpy as np
import pytest

from oracle import ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_1711_10413_amd import dsr as D  # noqa: E402

TEAMS, N = 2, 12 * 1024                      # six 1024-element batches per one-wave team
CHUNK = N // TEAMS
S = 300000                                   # the first loop's scalar


def stream():
    return torch.cuda.current_stream().cuda_stream


def team_words(x):
    """The 32-bit words of each team's exact sum of S * x, in units of 2^-75."""
    out = []
    for t in range(TEAMS):
        units = int(x[t * CHUNK:(t + 1) * CHUNK].astype(np.int64).sum()) * S << 75
        raw = (units & ((1 << 192) - 1)).to_bytes(24, "little")
        out.append(np.frombuffer(raw, np.int32))
    return out


@pytest.mark.parametrize("slab", [0, 4096])
@pytest.mark.parametrize("reader", ["list", "list_chunk", "affine", "gather", "array"])
def test_loop_reads_an_earlier_sum(reader, slab):
    x_np = (np.arange(N) % 7 + (np.arange(N) // 1024) % 5).astype(np.float32)
    x = torch.from_numpy(x_np).cuda()
    y = torch.zeros(N, dtype=torch.float64, device="cuda")
    y2 = torch.zeros(N, dtype=torch.float64, device="cuda")
    out = torch.zeros(N, dtype=torch.int32, device="cuda")
    ctx = D.dsr_init(wg_size=64, lds_slab_bytes=slab, hbm_slab_bytes=4096, max_teams=TEAMS)
    words = team_words(x_np)
    r = D.dsr_region_begin(ctx, TEAMS)
    f = D.dsr_push(r, 28, np.array([0, 0, 0, 0, 0, 0, S], np.int32).tobytes())
    D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, N, inp=x.data_ptr(), out=y.data_ptr(), ni=1)
    pieces = [slice(t * CHUNK, (t + 1) * CHUNK) for t in range(TEAMS)]
    if reader in ("list", "list_chunk", "array"):
        g = D.dsr_push(r, 32)
        if reader == "array":                # the sum's words 3 to 5 as an array
            refs, kw = [(g, 0), (g, 24), (f, 12)], {"ni": 1, "alen": 3}
            want = np.concatenate([R.fma_chain(x_np[p], [0], [], words[t][3:6], p.start) for t, p in enumerate(pieces)])
        else:                                # word 3 as an int32 scalar
            refs, kw = [(g, 0), (f, 12)], {"ni": 1}
            if reader == "list_chunk":
                kw["chunk"] = CHUNK
            want = np.concatenate([R.fma_chain(x_np[p], [words[t][3]], []) for t, p in enumerate(pieces)])
        D.dsr_publish_list(r, refs, D.DSR_BODY_FMA_CHAIN_REFS, N, inp=x.data_ptr(), out=y2.data_ptr(), **kw)
        D.dsr_pop(r, g)
        got = y2
    elif reader == "affine":                 # a, b, c, d are the sum's words 2 to 5
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, N, out=out.data_ptr())
        want = np.concatenate([R.affine_xor(*[int(v) for v in words[t][2:6]], p.start, p.stop)[0]
                               for t, p in enumerate(pieces)])
        got = out
    else:
        D.dsr_publish(r, f, D.DSR_BODY_GATHER, N, out=out.data_ptr(), arrays=1, length=6)
        want = np.concatenate([R.gather([words[t]], p.start, p.stop) for t, p in enumerate(pieces)])
        got = out
    D.dsr_pop(r, f)
    D.dsr_launch(r, stream())
    assert D.dsr_region_sync(r) == 0
    assert np.array_equal(y.cpu().numpy(), R.fma_chain(x_np, [S], []))
    assert np.array_equal(got.cpu().numpy(), want)
    assert D.dsr_region_reduction(r, 0)[2] == R.fixed75_sum(R.fma_chain(x_np, [S], []))
    D.dsr_region_free(r)
    D.dsr_destroy(ctx)
