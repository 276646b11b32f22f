"""Every kernel that is launched with more dynamic LDS than a kernel may have unasked (64 KB) has been asked for by then, itself and not another
variant of its tile.  Host code, checked without a GPU: tests/native/launch_recorder.c stands in for the runtime's launch path.
"""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SETUP = """
import ctypes, sys
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)          # ahead of the runtime that the library brings along
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
from paper_2604_28175_amd.binding import lib
A, F = 4096, 1e-6
def ok(status):
    assert status == 0, (status, lib.strait_last_error())
def recorded(what):
    return ctypes.c_int.in_dll(recorder, "recorded_" + what).value
"""
LDS = SETUP + """
from conv_shapes import LAYERS
for _, (n, h, w, c, k, r, stride, pad), res in LAYERS:
    ok(lib.strait_k_conv2d(None, A, n, h, w, c, A, A, k, r, r, stride, pad, 0, A if res else None, A, 0, 0))
for m, n, k in ((20000, 1024, 256), (20000, 1024, 768), (3136, 1024, 256), (3136, 1024, 1024), (1024, 3072, 768), (5000, 3072, 768), (12608, 768, 768),
                (700, 768, 3072), (1379, 768, 3072), (2758, 768, 3072), (8192, 768, 3072), (128, 768, 768)):
    for act, res in ((0, None), (3, None), (0, A), (1, A)):
        ok(lib.strait_k_gemm(None, A, A, A, m, n, k, act, res, A, 0, 0))
for m in (1, 40, 128, 300, 700, 1025, 1379, 2048, 2600, 2758, 4096, 5000, 8192, 12608, 20000):
    for n, k in ((64, 64), (768, 768), (2304, 768), (3072, 768), (768, 3072), (1024, 1024), (256, 512)):
        for act in (0, 3):
            ok(lib.strait_k_gemm_ln(None, A, A, A, None, m, n, k, act, A, A, None, None, F, A, None, 0) if k <= 1024 else 0)
        if n <= 1024:
            ok(lib.strait_k_gemm_ln(None, A, A, A, A, m, n, k, 0, None, None, None, None, F, A, A, 0))
            ok(lib.strait_k_gemm_ln(None, A, A, A, A, m, n, k, 0, A, None, A, A, F, A, A, 0))
for n, p, c, c2, k in ((128, 56, 64, 64, 256), (128, 28, 128, 256, 512), (128, 14, 256, 512, 1024), (128, 7, 512, 1024, 2048), (1, 7, 512, 1024, 2048)):
    ok(lib.strait_k_conv1x1_proj(None, A, n, p, p, c, A, 2 * p, 2 * p, c2, 2, A, A, k, 1, A, 0))
count = [recorded(what) for what in ("launches", "wide", "unasked")]
print(*count)
sys.exit(0 if count[0] > 400 and count[1] > 200 and count[2] == 0 else 1)
"""
# folded products of more tiles than compute units: the tiles of four wavefronts of which two are meant to share a unit (64 to 80 KB each)
PAIRS = SETUP + """
bad = []
for m in (1025, 1379, 2048, 2758, 4096, 5000, 8192, 12608, 16384):
    for width in (512, 640, 768, 832, 896, 960, 1024):
        for n in (width, 3 * width, 4 * width):
            for act in (0, 3):
                ok(lib.strait_k_gemm_ln(None, A, A, A, None, m, n, width, act, A, A, None, None, F, A, None, 0))
                bad.append(((m, n, width, act), [recorded("last_" + w) for w in ("grid", "block", "lds")]))
        for k in (width, 4 * width):
            ok(lib.strait_k_gemm_ln(None, A, A, A, A, m, width, k, 0, A, None, A, A, F, A, A, 0))
            bad.append(((m, width, k, "residual"), [recorded("last_" + w) for w in ("grid", "block", "lds")]))
bad = [b for b in bad if b[1][0] > 512 and b[1][1] == 256 and 80 * 1024 < b[1][2] < 96 * 1024]
print(len(bad), bad[:5])
sys.exit(1 if bad else 0)
"""


def run(program, tmp_path):
    recorder = str(tmp_path / "recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", recorder, os.path.join(ROOT, "tests", "native", "launch_recorder.c")], check=True)
    r = subprocess.run([sys.executable, "-c", program, recorder, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-1500:] + r.stderr[-1500:]


@pytest.mark.skipif(shutil.which("gcc") is None, reason="no C compiler")
def test_lds_beyond_the_default_is_asked_for_kernel_by_kernel(tmp_path):
    run(LDS, tmp_path)


@pytest.mark.skipif(shutil.which("gcc") is None, reason="no C compiler")
def test_tiles_that_are_meant_to_share_a_compute_unit_do(tmp_path):
    """The statistics of a wide LayerNorm's rows lie in the workgroup's LDS as well: with them a tile may not be chosen for sharing that it no longer does."""
    run(PAIRS, tmp_path)
