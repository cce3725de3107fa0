"""A failed call enqueues nothing: the HIP runtime's launch functions are replaced by recording ones (no
GPU), every request for dynamic LDS is refused in turn, and no kernel may have been launched by then."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2509_01085_amd import binding as B

SHIM = r"""
#include <string.h>
static int allow, grants, launches;
void shim_reset(int a) { allow = a; grants = launches = 0; }
int shim_grants(void) { return grants; }
int shim_launches(void) { return launches; }
typedef struct { unsigned x, y, z; } dim3_t;
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* f, int attr, int v) { return ++grants > allow; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st) { return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st) {
  memset(g, 0, sizeof *g); memset(b, 0, sizeof *b); *s = 0; *st = 0; return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t s, void* st) { ++launches; return 0; }
"""

CHILD = r"""
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the runtime in the lookup order
from paper_2509_01085_amd import binding as B
L, p, big = B.lib(), 4096, 1 << 60
refused = 0
# 16 blocks of 2 heads; 12 blocks; 330 of 14: both forward kernels and their combine launch, but with d = 64 and one tile a block
for H, N, d, n_keep in [(2, 16, d, k) for d in (64, 128) for k in (16, 32, 64)] + [(2, 12, d, 32) for d in (64, 128)] + [(14, 330, d, k) for d in (64, 128) for k in (16, 32, 64)]:
        s = C.byref(B.Shape(1, H, 4, 4, 4 * N, 4, 4, 4, d, B.BF16).c())
        calls = {
            "fwd": lambda: L.bsa_attn_fwd(s, p, p, p, p, p, p, n_keep, 0.1, p, p, p, big, None),
            "bwd": lambda: L.bsa_attn_bwd(s, *[p] * 11, n_keep, 0.1, p, p, p, p, big, None),
            "dense fwd": lambda: L.bsa_dense_attn_fwd(s, p, p, p, 0.1, p, p, None),
            "dense bwd": lambda: L.bsa_dense_attn_bwd(s, *[p] * 6, 0.1, p, p, p, p, big, None),
        }
        for name, call in calls.items():
            allow, st = 0, -6
            while st != 0:  # grants are kept, so every turn gets at least one further
                shim.shim_reset(allow)
                st = call()
                assert st in (0, -6), (name, st)
                if st == -6:
                    assert shim.shim_grants() == allow + 1 and shim.shim_launches() == 0, (name, d, n_keep, allow, shim.shim_launches())
                    refused += 1
                allow = 1
            assert shim.shim_launches() == 3 or not (name == "fwd" and N == 330 and (d, n_keep) in [(128, 16), (128, 32), (128, 64), (64, 64)])
            assert shim.shim_launches() > 0
print("refused", refused)
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs a C compiler")
def test_a_refused_lds_request_comes_before_any_launch(tmp_path):
    B.lib()
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-w", "-o", str(so), str(src)])
    root = os.path.dirname(os.path.dirname(os.path.abspath(B.__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(so)], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.split()[-1]) >= 18  # both forwards, dQ and dK/dV of the variants each had a request refused
