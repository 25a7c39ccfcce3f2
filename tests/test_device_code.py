"""What the compiled device code has to hold that no run can show reliably (gfx950 assembly,
no GPU)."""
import os
import re
import subprocess

from paper_2207_03803_amd import build

PUBLISH = """
#include "common.h"
__global__ __launch_bounds__(512) void publish(double *part, unsigned *counter, double *out, double v)
{
    __shared__ int flag;
    part[(long)blockIdx.x * 512 + threadIdx.x] = v;
    if (arrive_last(counter, gridDim.x, &flag))
        out[threadIdx.x] = part[threadIdx.x];
}
"""


def _assembly(tmp_path, source):
    src = tmp_path / "probe.hip"
    src.write_text(source)
    out = tmp_path / "probe.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)],
                   check=True, capture_output=True, text=True)
    return out.read_text()


def test_every_wave_waits_for_its_stores_before_it_arrives(tmp_path):
    """The counter of arrive_last is raised by one wave, whose own wait covers its own stores
    only: each wave must have waited for its stores before the barrier in front of it.
    Reading side: each wave invalidates what it may hold of the others' results."""
    assert os.path.exists(build.HIPCC)
    asm = _assembly(tmp_path, PUBLISH)
    body = asm[asm.index("publish"):]
    store = body.index("global_store")
    barrier = body.index("s_barrier", store)
    atomic = body.index("global_atomic_add", barrier)
    assert re.search(r"s_waitcnt[^\n]*vmcnt\(0\)", body[store:barrier])
    last = body.index("s_barrier", atomic)
    load = body.index("global_load", last)
    assert "buffer_inv" in body[last:load]
