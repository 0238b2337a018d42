"""A team written against include/dsr_device.h alone: every call of the device
API compiles for the GPU.  A device-only compile on the CPU."""
import os
import shutil
import subprocess

import pytest

from paper_1711_10413_amd import build as B

SOURCE = r"""
#include "dsr_device.h"
using namespace dsr;

/* One region: the master shares an int64 sum and a factor, every worker lane adds
 * factor * its thread number, the master adds the waves' partials up. */
__global__ void team(uint8_t *hbm, uint32_t hbm_cap, uint32_t nw, uint32_t lds_cap, int64_t *out)
{
    extern __shared__ __align__(16) uint8_t lds[];
    team_t T = team_init(lds, nw, lds_cap, 0xFFFFFFFFu, hbm + (uint64_t)blockIdx.x * hbm_cap, hbm_cap);
    if (T.wave == nw - 1) {
        team_reset(T);
        frame_t f = push(T, 16);
        if (T.lane == 0) {
            *slot<int64_t>(T, f, 0) = 0;
            *slot<int32_t>(T, f, 8) = 3;
        }
        publish(T, f, 1, 0);
        end_parallel(T, 0, 0, 0, 0);
        int64_t sum = 0;
        for (uint32_t w = 0; w + 1 < nw; ++w) sum += (int64_t)red_slot(T, w)[0];
        if (T.lane == 0) {
            *slot<int64_t>(T, f, 0) += sum;
            out[blockIdx.x] = header(T)->bad ? -1 : *slot<int64_t>(T, f, 0);
        }
        if (!pop(T, f)) header(T)->error = -1;
        publish(T, frame_t{SPACE_NONE, 0, 0}, 0, 0);
        return;
    }
    uint32_t body, loop;
    frame_t f;
    while (await(T, &body, &f, &loop)) {
        uint64_t v = (uint64_t)*slot<int32_t>(T, f, 8) * threadIdx.x;
        for (int d = 32; d; d /= 2) v += __shfl_xor(v, d, 64);
        end_parallel(T, v, 0, 0, v > 1000000);
    }
}
"""


@pytest.mark.skipif(not shutil.which(B.HIPCC) and not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_team_on_the_device_api_compiles(tmp_path):
    src = tmp_path / "team.hip"
    src.write_text(SOURCE)
    p = subprocess.run([B.HIPCC] + B.FLAGS + ["--offload-device-only", "-c", "-o", str(tmp_path / "team.o"), str(src)],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
