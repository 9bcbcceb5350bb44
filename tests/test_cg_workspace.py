"""The CG handle's workspace holds what every later call on the handle writes:
fewer right-hand sides lay their residual partials and product partials out
otherwise, and some of these layouts are larger.  Runs the library's host code
without a GPU, on stand-ins for the HIP calls that hand out addresses, take
every launch for done, answer every read-back with ones, and hold the partial
arrays of each launch against the allocations."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
struct Dim { unsigned x, y, z; };
static std::map<uintptr_t, size_t> live;
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static uintptr_t top = 1ull << 44;
static Dim cfg[2];
static size_t lds;
static void *str;
static int bad, seen;
static void need(const char *what, const void *p, int64_t bytes)
{
    auto it = live.upper_bound((uintptr_t)p);
    ++seen;
    if (it != live.begin() && (--it, (uintptr_t)p + bytes <= it->first + it->second)) return;
    ++bad;
    printf("OUT OF BOUNDS %s: %lld bytes\n", what, (long long)bytes);
}
extern "C" {
int hipMalloc(void **p, size_t n) { *p = (void *)top; live[top] = n; top += (n + 4095) / 4096 * 4096 + 4096; return 0; }
int hipFree(void *p) { live.erase((uintptr_t)p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(n, 1); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipMemcpyAsync(void *d, const void *, size_t n, int kind, void *)
{
    if (kind == 2) for (size_t i = 0; i + 8 <= n; i += 8) ((double *)d)[i / 8] = 1.0;
    return 0;
}
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, void *) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipStreamCreateWithFlags(void **, unsigned) { return 1; }  // no capture: direct launches
int __hipPushCallConfiguration(Dim g, Dim b, size_t l, void *s) { cfg[0] = g; cfg[1] = b; lds = l; str = s; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *l, void **s) { *g = cfg[0]; *b = cfg[1]; *l = lds; *s = str; return 0; }
void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) { names()[f] = name; }
int hipLaunchKernel(const void *f, Dim g, Dim, void **a, size_t, void *)
{
    const char *k = names().at(f).c_str();
    auto i64 = [&](int i) { return *(int64_t *)a[i]; };
    auto i32 = [&](int i) { return (int64_t) * (int *)a[i]; };
    auto ptr = [&](int i) { return *(void **)a[i]; };
    if (const char *s = strstr(k, "k_resid_symILi")) {
        const int64_t nrb = (i64(2) + 63) / 64, nc = atoi(s + 14) + 1;
        need("residual row partials", ptr(8), nrb * nrb * nc * 64 * 8);
        need("residual column partials", ptr(9), nrb * i32(7) * nc * 64 * 8);
    } else if (strstr(k, "k_resid_mfma")) {
        need("residual slices", ptr(8), i32(7) * i32(5) * i64(2) * 8);
        need("residual |A| slices", ptr(9), i32(7) * i64(2) * 8);
    } else if (strstr(k, "k_cg_mv_sym")) {
        need("tile sums", ptr(5), i64(1) / 256 * i64(1) * 4);
        need("product partials (triangle)", ptr(6), (int64_t)g.x * 8);
    } else if (const char *s = strstr(k, "k_cg_mv_valuILi")) {
        need("product partials", ptr(6), i64(7) * atoi(s + 15) * 8);
    } else if (strstr(k, "k_cg_mv_ksum")) {
        need("product partials (slices)", ptr(5), i64(6) * i32(1) * 8);
    }
    return 0;
}
int stub_report(int *s) { *s = seen; return bad; }
}
"""

RUN = r"""
import ctypes as C, sys
import paper_1405_4644_amd as spd
lib, stub = spd.load(), C.CDLL(sys.argv[1])
fake = C.c_void_p(1 << 20)
o = spd.cg_default_opts(max_outer=3, max_inner=2)
for n, band in ((201, -1), (300, -1), (833, 5), (1500, -1), (2300, -1), (2500, 200), (3000, -1), (3073, -1), (3300, -1),
                (4097, -1), (6000, 16), (10000, -1)):
    for ms in ((3, 1), (3, 2), (4, 2), (5, 4, 3, 2, 1), (6, 1), (32, 1), (40, 17, 4, 2)):
        h, rep = C.c_void_p(), spd.Report()
        assert lib.spd_cg_prepare(fake, n, n, band, None, C.byref(h)) == 0
        for m in ms:
            before = C.c_int()
            stub.stub_report(C.byref(before))
            lib.spd_cg_refine(h, fake, n, fake, n, m, fake, n, C.byref(o), C.byref(rep), None)
            after = C.c_int()
            print(n, band, ms, m, "status", rep.status, flush=True)
            if stub.stub_report(C.byref(after)):
                sys.exit("a launch writes past its allocation")
            assert after.value > before.value, "nothing was looked at"
        lib.spd_cg_destroy(h)
"""


def test_a_handle_serves_fewer_right_hand_sides(tmp_path):
    import paper_1405_4644_amd as spd
    if not os.path.exists(spd.LIB_PATH):
        pytest.fail("libspd.so is not built (python -m paper_1405_4644_amd.build)")
    src, lib = tmp_path / "stub.cpp", tmp_path / "stub.so"
    src.write_text(STUB)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-o", str(lib), str(src)], check=True)
    out = subprocess.run([sys.executable, "-c", RUN, str(lib)], capture_output=True, text=True, timeout=120, cwd=ROOT,
                         env=dict(os.environ, LD_PRELOAD=str(lib)))
    assert out.returncode == 0, (out.stdout[-1500:], out.stderr[-1500:])
