"""What the library launches for a call, seen from the host: its own host code runs against a stand-in for the HIP runtime
(hip_host_stub.cpp) that records every launch and refuses what the runtime would refuse.  No GPU is used."""
import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys, threading
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_records.restype = ctypes.c_char_p
import paper_1706_09453_amd as bnn
A, B, C, D, E = (0x1000000000 * i for i in range(1, 6))    # made-up device addresses, far apart
def launches():
    out = []
    for line in stub.stub_records().decode().splitlines():
        w = line.split()
        out.append(dict(kernel=w[0], grid=[int(v) for v in w[1:4]], block=int(w[4]), lds=int(w[5]), device=int(w[6]), wrong=w[7:]))
    stub.stub_clear()
    return out
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """host(code): runs `code` in a process of its own, where launches() lists what was launched; returns its `result`."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    stub = str(tmp_path_factory.mktemp("stub") / "libhip_host_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-o", stub, os.path.join(HERE, "hip_host_stub.cpp")], check=True)

    def run(code):
        src = PRELUDE.format(root=ROOT, stub=stub) + code + "\nimport json; print('RESULT ' + json.dumps(result))\n"
        res = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr[-2000:]
        return json.loads(res.stdout.split("RESULT ", 1)[1])

    return run


def test_norm_inside_the_workspace_is_written_before_the_gradient_is_scaled(host):
    """norm_out may lie in the 2048 bytes of partial sums: the launch that scales must then not be the one that stores the
    norm, since its other workgroups still read the sums."""
    got = host("""
result = []
for norm in (B, B + 4, B + 2044, B + 2048, C):
    bnn.bnn_grad_norm_clip(A, 1 << 20, 15.0, B, norm)
    result.append([l["kernel"] for l in launches()])
""")
    for kernels in got[:3]:
        assert len(kernels) == 3 and "sumsq_partial" in kernels[0] and "sumsq_final" in kernels[1] and "scale_if_above" in kernels[2], kernels
    for kernels in got[3:]:
        assert len(kernels) == 2 and "sumsq_partial" in kernels[0] and "scale_if_above" in kernels[1], kernels
