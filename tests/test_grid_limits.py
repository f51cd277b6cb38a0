"""Launches stay below the grid limit of 2^32 work-items (no GPU).

Stand-ins for the launch calls, loaded before the library, records the grids of
the Schwarz launches of every pair class for as many pairs as 13.5 million: one
launch of a workgroup of 320 lanes per pair would be 4.3e9 work-items; and of
the first and last launch of a build for batches of up to 65,535 molecules
(a grid's rows) beside one of up to 2,000 functions: a workgroup per 256
elements of the largest molecule for each would be 2.6e11.
"""
import json
import os
import subprocess
import sys

STUB = r"""
typedef struct { unsigned x, y, z; } dim3;
unsigned long long n, grids[64], lanes[64];
const void *args[64][2];
static dim3 cg, cb;
int __hipPushCallConfiguration(dim3 g, dim3 b, unsigned long m, void *t) { cg = g; cb = b; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, unsigned long *m, void **t) { *g = cg; *b = cb; *m = 0; *t = 0; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, unsigned long s, void *t) {
    grids[n] = (unsigned long long)g.x * g.y * g.z;
    lanes[n] = (unsigned long long)b.x * b.y * b.z;
    args[n][0] = *(const void **)a[0];   /* pairs, Q: first and last argument of the pair-a-workgroup kernels */
    args[n][1] = *(const void **)a[3];
    ++n;
    return 0;
}
"""

RUN = r"""
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)   # first in the search order
sys.path.insert(0, sys.argv[2])
from paper_1708_00033_amd import hfx
lib = C.CDLL(hfx._lib._name)
v = C.c_void_p
lib.hfx_launch_schwarz.argtypes = [C.c_int, v, C.c_int, v, v, v, v, v]
n = C.c_ulonglong.in_dll(stub, "n")
grids = (C.c_ulonglong * 64).in_dll(stub, "grids")
lanes = (C.c_ulonglong * 64).in_dll(stub, "lanes")
args = ((v * 2) * 64).in_dll(stub, "args")
out = []
for cid, npairs in json.loads(sys.argv[3]):
    n.value = 0
    assert lib.hfx_launch_schwarz(cid, 1 << 40, npairs, 1, 1, 1, 1 << 44, None) == 0
    out.append([(grids[i], lanes[i], args[i][0], args[i][1]) for i in range(n.value)])
print(json.dumps(out))
"""

RUN_BATCH = RUN[:RUN.index("lib.hfx_launch_schwarz.argtypes")] + r"""
i, z = C.c_int, C.c_size_t
lib.hfx_start_build.argtypes = [v, v, i, v, v, v, i, v, z, v, v]
lib.hfx_assemble.argtypes = [v, v, v, i, v, v, v, i, v, v, v]
n = C.c_ulonglong.in_dll(stub, "n")
grids = (C.c_ulonglong * 64).in_dll(stub, "grids")
lanes = (C.c_ulonglong * 64).in_dll(stub, "lanes")
bufs = (C.c_ulonglong * 16)()
out = []
for nmol, ld, nke in json.loads(sys.argv[3]):
    n.value = 0
    lib.hfx_start_build(1, 1, nmol, 1, 1, 1, ld, 1, nke, C.addressof(bufs), None)
    lib.hfx_assemble(1, 1, 1, nmol, 1, 1, 1, ld, 1, 1, None)
    out.append([(grids[k], lanes[k]) for k in range(n.value)])
print(json.dumps(out))
"""


def test_schwarz_launches(tmp_path):
    (tmp_path / "stub.c").write_text(STUB)
    stub = str(tmp_path / "stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", stub, str(tmp_path / "stub.c")], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    cases = [(cid, n) for cid in (0, 2, 5, 9, 14, 20) for n in (1, 1 << 20, (1 << 20) + 1, 13_500_000)]
    res = subprocess.run([sys.executable, "-c", RUN, stub, root, json.dumps(cases)], check=True, text=True,
                         capture_output=True).stdout
    for (cid, npairs), rows in zip(cases, json.loads(res)):
        assert rows and all(g * b < 1 << 32 for g, b, _, _ in rows), (cid, npairs)
        if cid in (14, 20):   # a workgroup per pair: each launch takes up where the last ended
            done = 0
            pair = (rows[1][2] - rows[0][2]) // rows[0][0] if len(rows) > 1 else 0
            for g, _, p, q in rows:
                assert p == (1 << 40) + pair * done and q == (1 << 44) + 8 * done
                done += g
            assert done == npairs
        else:
            assert len(rows) == 1 and rows[0][0] * rows[0][1] >= npairs


def test_build_launches_of_large_batches(tmp_path):
    (tmp_path / "stub.c").write_text(STUB)
    stub = str(tmp_path / "stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", stub, str(tmp_path / "stub.c")], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    cases = [(1, 26, 1000), (1, 9728, 10 ** 9), (256, 304, 10 ** 7), (40000, 304, 2 * 10 ** 9), (65535, 2000, 10 ** 9),
             (65535, 2, 0), (65535, 2, 10 ** 10)]
    res = subprocess.run([sys.executable, "-c", RUN_BATCH, stub, root, json.dumps(cases)], check=True, text=True,
                         capture_output=True).stdout
    for (nmol, ld, nke), rows in zip(cases, json.loads(res)):
        assert len(rows) == 2
        for g, b in rows:
            assert g * b < 1 << 32 and g % nmol == 0, (nmol, ld, nke)
        # columns for the matrices, and others for the ket elements where there are any
        assert rows[0][0] // nmol >= 1 + (nke > 0) and rows[1][0] // nmol >= 1
