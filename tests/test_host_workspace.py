"""Workspace sizes and the tile choices they follow from, on the host: no GPU, and none asked for."""
import os
import subprocess
import sys

import paper_2409_12210_amd as m

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WIDTHS = [2816, 8448, 4224, 7040, 4928, 6336, 5632, 5632]

# a stand-in for the runtime's device queries that counts its calls and reports CUS compute units
SHIM = """
#include <hip/hip_runtime_api.h>
int device_queries = 0;
hipError_t hipGetDevice(int* dev) { ++device_queries; *dev = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int dev) {
  (void)dev; ++device_queries; p->multiProcessorCount = CUS; return hipSuccess;
}
"""
SIZES = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import paper_2409_12210_amd as m
print([m.modse_workspace_size(d, f, 2, dt, T, w) for d, f in ((2048, %r), (256, [128, 384])) for dt in ("bf16", "f32")
       for T in (1, 64, 389, 1021, 32768) for w in (m.WS_FWD, m.WS_BWD, m.WS_FWD_SAVED)],
      ctypes.c_int.in_dll(shim, "device_queries").value)
""" % WIDTHS


def test_sizes_do_not_depend_on_a_device(tmp_path):
    """modse_workspace_size is host arithmetic: it asks the runtime for nothing (a program may call it before it picks a
    device, or in a process that never has one), so its answers are the same whatever device there is."""
    src = tmp_path / "shim.c"
    src.write_text(SHIM)
    out = []
    for cus in (64, 256):
        lib = tmp_path / ("shim_%d.so" % cus)
        subprocess.run(["gcc", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DCUS=%d" % cus, "-I/opt/rocm/include", str(src),
                        "-o", str(lib)], check=True)
        r = subprocess.run([sys.executable, "-c", SIZES, str(lib)], cwd=ROOT, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        out.append(r.stdout)
    assert out[0] == out[1]
    assert out[0].split()[-1] == "0", "device queries made"


def test_a_workspace_for_a_larger_batch_serves_the_smaller_ones():
    """Sizes never fall with the token count, although the partial sums of split products are a matter of small batches: a
    program sizes once, for its largest batch."""
    for d, d_ff, k in ((2048, WIDTHS, 2), (4096, [14336] * 8, 2), (1024, [2816] * 4, 1), (96, [4128, 96, 3104, 2016], 2),
                       (32, [9600, 32], 1)):
        for dtype in ("bf16", "f32"):
            for which in (m.WS_FWD, m.WS_BWD, m.WS_FWD_SAVED):
                sizes = [m.modse_workspace_size(d, d_ff, k, dtype, T, which)
                         for T in list(range(1, 1200)) + list(range(1200, 40000, 371))]
                assert sizes == sorted(sizes), (d, dtype, which)
