"""Which kernel a call is sent to, on the host: the library's own argument checks and dispatch (bsfa_api.hip and part 0 of
bsfa_fwd.hip, compiled for the host alone), linked with launchers that note their template arguments and launch nothing."""
import atexit
import ctypes
import functools
import os
import re
import shutil
import subprocess
import tempfile
from collections import namedtuple

from paper_2512_07011_amd import binding, build

SRC = r"""
#define BSFA_PART 99
#define launch_fwd unused_launch_fwd
#define launch_scores unused_launch_scores
#include "bsfa_fwd.hip"
#undef launch_fwd
#undef launch_scores
static int noted[15];
extern "C" const int *last_launch() { return noted; }
namespace bsfa {
template <int D, int NWH, int HP, int QT, int KSP, int KR> hipError_t launch_fwd(const FwdParams &params, hipStream_t, unsigned spare)
{
    FwdParams p = params;
    const unsigned grid = decompose<HP, QT>(p);
    turned_places(p, grid, std::min(places_of(D, NWH * HP * QT, KSP), spare ? 2 : 3));
    const int now[15] = {0, D, NWH, HP, QT, KSP, KR, (int)spare, (int)grid, (int)p.turn[0], (int)p.turn[1], (int)p.turn[2], p.vt != nullptr, p.k8 != nullptr, p.counted};
    std::copy(now, now + 15, noted);
    return hipSuccess;
}
template <int D, int NWH, int HP, int QT, int KR> hipError_t launch_scores(const FwdParams &params, hipStream_t)
{
    FwdParams p = params;
    const int now[15] = {1, D, NWH, HP, QT, 1, KR, 0, (int)decompose<HP, QT>(p)};
    std::copy(now, now + 15, noted);
    return hipSuccess;
}
%s
size_t select_area_bytes(int) { return 1 << 20; }
hipError_t launch_select(const float *, long, int, int, const SelectLevels &, int, void *, float *, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_topk(const float *, int, long, long, const TopkLevels &, int, float *, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_mfma_rate_probe(const float *, float *, int, int, hipStream_t) { return hipErrorUnknown; }
}
"""

# score: the score half alone (calibration); tiles: adjacent query tiles of a workgroup; turn, counted: see FwdParams
Launch = namedtuple("Launch", "score head_dim waves heads tiles shares ring spare grid turn vt k8 counted")


@functools.lru_cache(maxsize=None)
def _lib():
    d = tempfile.mkdtemp(prefix="bsfa_dispatch_")
    atexit.register(shutil.rmtree, d, ignore_errors=True)
    parts = re.findall(r"#define (BSFA_SHAPES_\d+)\(", open(os.path.join(build.CSRC, "bsfa_fwd.hip")).read())
    stub = os.path.join(d, "stub.hip")
    with open(stub, "w") as f:
        f.write(SRC % "\n".join("%s(BSFA_DEFINE_F, BSFA_DEFINE_S)" % x for x in parts))
    common = ["-std=c++17", "-O1", "-fPIC", "-w", "-I" + build.CSRC, "-c"]
    hip = [build.HIPCC, "-x", "hip", "--offload-host-only", *common]
    # (plain C++ where a device array is defined: without device code there is nothing to register it with)
    cxx = [build.HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-D__device__=", "-D__align__(x)=", "-DHIP_SYMBOL(x)=&x", "-I/opt/rocm/include", *common]
    objs = [os.path.join(d, n) for n in ("fwd.o", "api.o", "stub.o")]
    for cmd, src, obj in ((hip + ["-DBSFA_PART=0"], os.path.join(build.CSRC, "bsfa_fwd.hip"), objs[0]),
                          (cxx, os.path.join(build.CSRC, "bsfa_api.hip"), objs[1]), (hip, stub, objs[2])):
        subprocess.run([*cmd, "-o", obj, src], check=True, capture_output=True)
    so = os.path.join(d, "dispatch.so")
    subprocess.run(["g++", "-shared", "-Wl,-z,defs", "-o", so, *objs, "-L/opt/rocm/lib", "-lamdhip64"], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    lib.last_launch.restype = ctypes.POINTER(ctypes.c_int)
    lib.bsfa_last_error.restype = ctypes.c_char_p
    return lib


def _problem(b, n, hq, hkv, d, bm, seqlens, single_head, gate_mode, qk_fp8):
    q, kv = [n * hq * d, hq * d, d], [n * hkv * d, hkv * d, d]
    p = binding.bsfa_problem(b, hq, hkv, n, d, bm, 64, *q, *kv, *kv, *q, 0)
    p.seqlens = 4096 if seqlens else None                          # (addresses that nothing on this path reads)
    p.single_head_groups, p.gate_mode, p.qk_fp8 = int(single_head), gate_mode, int(qk_fp8)
    return p


def _noted(lib, rc):
    assert rc == 0, lib.bsfa_last_error()
    x = lib.last_launch()[:15]
    return Launch(bool(x[0]), *x[1:9], tuple(x[9:12]), *map(bool, x[12:15]))


def forward(b, n, hq, hkv, d, bm, causal=True, seqlens=False, single_head=False, gate_mode=0, qk_fp8=False, workspace=False):
    lib, a = _lib(), ctypes.c_void_p(4096)
    p = _problem(b, n, hq, hkv, d, bm, seqlens, single_head, gate_mode, qk_fp8)
    if workspace or qk_fp8:
        p.workspace, p.workspace_bytes = 4096, 1 << 50
    return _noted(lib, lib.bsfa_forward(ctypes.byref(p), a, a, a, a, int(causal), a, None, None))


def scores(b, n, hq, hkv, d, bm, causal=True):
    """The score half of a calibration, through bsfa_calibrate_topk, which ends where the selection is launched."""
    lib, a = _lib(), ctypes.c_void_p(4096)
    p, k = _problem(b, n, hq, hkv, d, bm, False, False, 0, False), ctypes.c_int32(1)
    rc = lib.bsfa_calibrate_topk(ctypes.byref(p), a, a, int(causal), ctypes.byref(k), 1, 0, a, a, ctypes.c_size_t(1 << 50), None)
    assert rc == -6 and b"selection launch failed" in lib.bsfa_last_error()
    return _noted(lib, 0)


def instantiated():
    """The first seven members of a Launch, for every form that the library holds."""
    src = open(os.path.join(build.CSRC, "bsfa_fwd.hip")).read()
    lists = "".join(re.findall(r"#define BSFA_SHAPES_\d+\(F, S\)(.*)", src))
    forward_forms = {(False, *map(int, x)) for x in re.findall(r"F\((\d+), (\d), (\d), (\d), (\d), (\d)\)", lists)}
    return forward_forms | {(True, *map(int, x[:4]), 1, int(x[4])) for x in re.findall(r"S\((\d+), (\d), (\d), (\d), (\d)\)", lists)}
