"""The window walk's wait for its stores orders memory for the compiler too:
compiled with the build's flags, a loop's store is made before the wait in every
turn (with the wait builtin alone the loop waits for nothing and one store
follows it)."""
import os
import re
import subprocess

import pytest

build = pytest.importorskip("paper_2609_14982_amd.build")


def _drain_source():
    src = open(os.path.join(build.CSRC, "ring.hip")).read()
    m = re.search(r"__device__ __forceinline__ void drain\(\) \{.*?\n?\}\n", src, re.S)
    assert m, "drain() of ring.hip"
    return m.group(0)


def test_stores_stay_before_the_wait(tmp_path):
    hip = tmp_path / "probe.hip"
    hip.write_text('#include <hip/hip_runtime.h>\n' + _drain_source() + '''
__global__ void probe(float* __restrict__ p, int n) {
    for (int i = 0; i < n; ++i) {
        p[0] = (float)i;
        drain();
    }
}
''')
    out = tmp_path / "probe.s"
    subprocess.check_call([build.HIPCC, *build.HIP_FLAGS, "--cuda-device-only", "-S", str(hip), "-o", str(out)])
    ops = re.findall(r"^\s*(global_store|s_waitcnt vmcnt)", out.read_text(), re.M)
    assert ops == ["global_store", "s_waitcnt vmcnt"], ops
