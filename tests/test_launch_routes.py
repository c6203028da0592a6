"""Which kernels a call launches, without a GPU: the library's own argument checks, plans and dispatch (csrc/tp_api.cpp) compiled for the
host with launchers that write down what they are asked to launch.  Addresses are never followed."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import paper_2110_14883_amd as T
from paper_2110_14883_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = r"""
#include <cstdio>
#include <string>
#include <hip/hip_runtime_api.h>
static hipError_t some_device(int* d) { *d = 0; return hipSuccess; }
static hipError_t some_attribute(int* v) { *v = 256; return hipSuccess; }
#define hipGetDevice(d) some_device(d)
#define hipDeviceGetAttribute(v, a, d) some_attribute(v)
#define HIP_SYMBOL(x) (&(x))
#define hipGetSymbolAddress(p, s) (*(p) = (void*)(s), hipSuccess)
#undef __device__
#define __device__
#undef __align__
#define __align__(n)
#include "tp_api.cpp"
static std::string said;
namespace tpl {
static std::string product(int form, int tile, const GemmArgs& a) {
    char s[96];
    std::snprintf(s, sizeof s, "%s tile %d split %d groups %d", form == FORM_NN ? "Y" : form == FORM_NT ? "dX" : "dW", tile, a.split_k, a.n_groups > 1 ? a.n_groups : 1);
    return s;
}
static hipError_t say(const std::string& s) { said += (said.empty() ? "" : "; ") + s; return hipSuccess; }
void tile_shape(int id, int* bm, int* bn) { *bm = id == TILE_128x256 || id == TILE_128x128 ? 128 : 256; *bn = id == TILE_256x128 || id == TILE_128x128 ? 128 : 256; }
hipError_t launch_gemm(int form, int tile, const GemmArgs& a, hipStream_t) { return say(product(form, tile, a)); }
hipError_t launch_gemm_pair(int tx, const GemmArgs& x, int tw, const GemmArgs& w, hipStream_t) { return say(product(FORM_NT, tx, x) + " with " + product(FORM_TN, tw, w)); }
hipError_t launch_reduce(const ReduceArgs&, hipStream_t) { return say("fix-up"); }
hipError_t launch_dgelu(const void*, int64_t, const void*, int64_t, void*, int64_t, int64_t, int64_t, hipStream_t) { return say("dA"); }
hipError_t launch_colsum(const void*, int64_t, int64_t, int64_t, float*, float*, hipStream_t) { return say("db"); }
hipError_t launch_dgelu_colsum(const void*, int64_t, const void*, int64_t, void*, int64_t, int64_t, int64_t, float*, float*, hipStream_t) { return say("dA and db"); }
size_t colsum_ws_bytes(int64_t, int64_t) { return 0; }
hipError_t launch_bias_act(const float*, int64_t, const void*, int, void*, int64_t, int, void*, int64_t, int64_t, int64_t, hipStream_t) { return say("act"); }
}
extern "C" const char* routes(void) { static std::string s; s = said; said.clear(); return s.c_str(); }
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    assert cxx, "the extension module's compiler is missing"
    d = tmp_path_factory.mktemp("routes")
    src, lib = str(d / "routes.cpp"), str(d / "routes.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2110_14883_amd", "csrc"), src, "-o", lib], check=True, capture_output=True)
    h, typed = C.CDLL(lib), B.lib()
    for name in ("tp_linear_fwd", "tp_linear_bwd", "tp_linear_bwd_partials"):
        getattr(h, name).argtypes, getattr(h, name).restype = getattr(typed, name).argtypes, C.c_int
    h.routes.restype = C.c_char_p
    return h


WS = (0x70000000000, 1 << 34)


def _blocks(kind, items):
    return (kind * len(items))(*[kind(*i) for i in items])


def _fwd(h, m, k, n, steps=1):
    grid, dims = B._GridS(T.MODE_2D, steps, 1, 1, 0, 0, 0), B._DimsS(m * steps, k * steps, n * steps)
    st = h.tp_linear_fwd(grid, dims, steps, _blocks(B._CBlk, [(0x10000, k)] * steps), _blocks(B._CBlk, [(0x20000, n)] * steps), None, 0, B._OBlk(0x30000, n, 0),
                         B._OBlk(None, 0, 0), *WS, None)
    assert st == 0
    return h.routes().decode()


def _bwd(h, m, k, n, at, dg=None, dx_bytes=2):
    """dX [m, k] of da_row [m, n] and W [k, n], dW [k, n] of X [m, k] and da_col [m, n]; at: address of each."""
    grid, dims, none = B._GridS(T.MODE_2D, 1, 1, 1, 0, 0, 0), B._DimsS(m, k, n), B._OBlk(None, 0, 0)
    blk = lambda name, ld: _blocks(B._CBlk, [(at[name], ld)])
    st = h.tp_linear_bwd(grid, dims, 1, 1, None, None, blk("da_row", n), blk("w", n), blk("x", k), blk("da_col", n), -1, -1, C.pointer(B._CBlk(dg, k)) if dg else None,
                         B._OBlk(at["dx"], k, 0 if dx_bytes == 2 else 1), B._OBlk(at["dw"], n, 1), none, None, *WS, None)
    assert st == 0
    return h.routes().decode()


FAR = {name: (i + 1) << 32 for i, name in enumerate(("da_row", "w", "x", "da_col", "dx", "dw"))}
SMALL = [(8, 64, 40), (16, 264, 72), (40, 136, 328), (300, 136, 328)]


@pytest.mark.parametrize("m,k,n", SMALL)
def test_both_small_backward_products_share_a_launch(host, m, k, n):
    route = _bwd(host, m, k, n, FAR)
    assert " with " in route and ";" not in route, route
    assert " with " in _bwd(host, m, k, n, FAR, dg=0x900000000, dx_bytes=4)
    # blocks that touch but do not overlap
    assert " with " in _bwd(host, m, k, n, dict(FAR, dx=FAR["x"] + 2 * m * k, dw=FAR["w"] + 2 * k * n))


@pytest.mark.parametrize("m,k,n", SMALL)
@pytest.mark.parametrize("over", ["dw over w", "dw over da_row", "dw over dg", "dw over dx", "dx over x", "dx over da_col", "dx into the last row of x", "dx ends in dw"])
def test_products_that_overwrite_each_others_operands_keep_their_order(host, m, k, n, over):
    dg = 0x900000000
    at = {"dw over w": dict(FAR, dw=FAR["w"]), "dw over da_row": dict(FAR, dw=FAR["da_row"]), "dw over dg": dict(FAR, dw=dg), "dw over dx": dict(FAR, dw=FAR["dx"]),
          "dx over x": dict(FAR, dx=FAR["x"]), "dx over da_col": dict(FAR, dx=FAR["da_col"]), "dx into the last row of x": dict(FAR, dx=FAR["x"] + 2 * m * k - 16),
          "dx ends in dw": dict(FAR, dx=FAR["dw"] - 2 * m * k + 16)}[over]
    first, second = _bwd(host, m, k, n, at, dg=dg).split("; ")
    assert first.startswith("dX") and second.startswith("dW")


@pytest.mark.parametrize("over,together", [("nothing", True), ("dw over w", False), ("dx over x", False)])
def test_grouped_backward_products(host, over, together):
    m, k, n, q = 40, 136, 328, 2
    grid, dims = B._GridS(T.MODE_2D, q, 1, 1, 0, 0, 0), B._DimsS(q * m, q * k, q * n)
    w, x, dx, dw = ([(g + 1) << s for g in range(q)] for s in (32, 34, 36, 38))
    if over == "dw over w":
        dw[1] = w[0]
    if over == "dx over x":
        dx[0] = x[1] + 2 * m * k - 16
    st = host.tp_linear_bwd_partials(grid, dims, q, q, C.pointer(B._CBlk(0x1000000, n)), _blocks(B._CBlk, [(a, n) for a in w]), _blocks(B._OBlk, [(a, k, 1) for a in dx]),
                                     _blocks(B._CBlk, [(a, k) for a in x]), _blocks(B._OBlk, [(a, n, 1) for a in dw]), *WS, None)
    route = host.routes().decode()
    assert st == 0 and "groups 2" in route and (" with " in route) == together and (";" in route) == (not together), route


@pytest.mark.parametrize("m,k,n,steps,want", [
    (16, 4096, 4096, 1, "tile 13 split"), (32, 4096, 4096, 1, "tile 14 split"),       # K over workgroups
    (16, 512, 16320, 1, "tile 13 split 1"), (32, 1024, 16384, 1, "tile 14 split 1"),  # one round of strips, one and two chunks a wave
    (8, 512, 28544, 1, "tile 13 split 1"),                                            # more strips, one chunk
    (30, 2360, 16992, 1, None), (10, 1792, 18944, 1, None), (32, 1624, 10896, 3, None)])  # chains in the open
def test_forwards_of_few_rows(host, m, k, n, steps, want):
    route = _fwd(host, m, k, n, steps)
    assert (want in route) if want else ("tile 13" not in route and "tile 14" not in route), route
