"""Which kernels a call launches, with which grid and into which bytes of its workspace, as the library's host code decides it: no
GPU runs.  A process of its own loads a stand-in for the few HIP entry points that the library calls, in front of the real ones: it
reports the compute units that a test gives each device and writes down every launch."""
import json
import shutil
import subprocess
import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_2509_23202_amd" / "libfp4mr.so"
MX, NV = 0, 1
OP_GEMM, OP_SPLIT = 2, 6
NO_CODES = 4   # GEMM variant of NVFP4: picked by size, but not the kernel that dequantizes both operands in its waves

# Products of the kernel for many tokens that the tests on the device name: the tile widths of their launches with the least workspace.
NV16_HALF_ROWS = {(129, 12296, 512): [128], (192, 57344, 6656): [256], (320, 28672, 1024): [256], (577, 10248, 384): [128], (1088, 8192, 512): [256], (2100, 10240, 512): [256],
                  (449, 12288, 2048): [128], (1161, 14977, 2048): [256, 128]}
NV16_TWO_LAUNCHES = {(2048, 10240, 512): [256, 128], (1137, 14664, 512): [256, 128], (2378, 14324, 384): [256, 128], (2053, 10248, 512): [256], (4000, 10200, 512): [256]}
NV16_NARROW = {(1024, 10240, 512): [128], (1000, 10200, 512): [128], (512, 8192, 512): [128]}
NV16_ONE_ROUND = {(2048, 8192, 128): [256], (2041, 7945, 256): [256], (300, 28680, 384): [256]}
NV16_512_COLUMNS = {(2048, 8192, 6656): [512], (2041, 7945, 6784): [512], (300, 28680, 6656): [256]}
# and of those in parts along K, with all the room for them
NV16_PARTS = {(65, 400, 8320): 128, (128, 1024, 14336): 128, (200, 1000, 10368): 128, (300, 528, 16512): 128, (520, 1040, 4096): 128, (600, 520, 2048): 128}
NV16_PARTS_SHORT_K = {(134, 18560, 3840): 256, (129, 12358, 3968): 256, (642, 1368, 2048): 128}
NV16_PARTS_HALF_ROWS = {(320, 8190, 8192): 512, (192, 4200, 28672): 512, (400, 6200, 8192): 512, (160, 16384, 8192): 512, (320, 8200, 8192): 512}
NV16_PARTS_ROOM = {(128, 2056, 10240): 128, (192, 4200, 28672): 512, (300, 528, 16512): 128, (256, 528, 8320): 128}

HIP = r"""
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static const void* fn[8192]; static const char* fn_name[8192]; static int fns;
static int device, units[64], n; static char text[1 << 22]; static int at;
static dim3 g, b; static size_t lds; static void* st; static void* module;
void fake_device(int d, int cus) { device = d; units[d] = cus; }
const char* fake_launches(void) { text[at] = 0; at = n = 0; return text; }
void** __hipRegisterFatBinary(const void* d) { (void)d; return &module; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* a, char* name, int e, size_t s, int c, int gl) {}
void __hipRegisterFunction(void** m, const void* f, char* d, const char* name, unsigned t, void* ti, void* bi, void* bd, void* gd, int* ws)
{ if (fns < 8192) { fn[fns] = f; fn_name[fns++] = name; } }
int __hipPushCallConfiguration(dim3 gg, dim3 bb, size_t l, void* s) { g = gg; b = bb; lds = l; st = s; return 0; }
int __hipPopCallConfiguration(dim3* gg, dim3* bb, size_t* l, void** s) { *gg = g; *bb = b; *l = lds; *s = st; return 0; }
int hipGetDeviceCount(int* n) { *n = 64; return 0; }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = units[d]; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = (void*)s; return 0; }
int hipLaunchKernel(const void* f, dim3 gg, dim3 bb, void** args, size_t l, void* s)
{
    const char* name = "?";
    for (int i = 0; i < fns; ++i) if (fn[i] == f) name = fn_name[i];
    long long v[6] = {0};
    if (strstr(name, "splitk_reduce_kernel")) {        /* partial, parts, elements */
        v[0] = *(long long*)args[0]; v[1] = *(int*)args[1]; v[2] = *(long long*)args[2];
    } else if (strstr(name, "nv16_reduce_kernel")) {   /* Nv16Sums: partial[2], parts[2], count[2] */
        const char* a = args[0]; int parts[2];
        memcpy(v, a, 8); memcpy(v + 3, a + 8, 8); memcpy(parts, a + 16, 8); memcpy(v + 2, a + 24, 8); memcpy(v + 5, a + 32, 8);
        v[1] = parts[0]; v[4] = parts[1];
    }
    at += snprintf(text + at, sizeof text - at - 1, "%s %u %u %zu %lld %lld %lld %lld %lld %lld\n", name, gg.x, gg.y, l, v[0], v[1], v[2], v[3], v[4], v[5]);
    return 0;
}
"""

HOST = r"""
import ctypes, json, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
hip.fake_launches.restype = ctypes.c_char_p
lib.fp4_workspace_bytes.restype = ctypes.c_size_t
P, I, Z = ctypes.c_void_p, ctypes.c_int64, ctypes.c_size_t
lib.fp4_workspace_bytes.argtypes = [ctypes.c_int, I, I, I, ctypes.c_int, ctypes.c_uint32]
lib.fp4_gemm.argtypes = [P] * 6 + [I] * 3 + [ctypes.c_int, P, P, Z, ctypes.c_uint32, P]
lib.fp4_fused_linear.argtypes = lib.fp4_w4a16_linear.argtypes = [P, I, I, ctypes.c_int, P, P, I, ctypes.c_int, P, ctypes.c_uint32, P]
BUF, WS, LAYOUTS = 1 << 40, 1 << 41, 24    # addresses that nothing reads; A_LAYOUT_GEMM | W_LAYOUT_GEMM
def launches():
    out = []
    for l in hip.fake_launches().decode().split("\n")[:-1]:
        f = l.split(" ")
        out.append({"kernel": f[0], "grid": [int(f[1]), int(f[2])], "sums": [[int(v) for v in f[4:7]], [int(v) for v in f[7:10]]]})
    return out
for req in json.load(sys.stdin):
    what, a = req[0], req[1:]
    if what == "device": hip.fake_device(*a); r = None
    elif what == "variant": r = lib.fp4_set_option(0, *a)
    elif what == "bytes": r = lib.fp4_workspace_bytes(a[0], a[1], a[2], a[3], a[4], LAYOUTS)
    elif what == "gemm":
        M, N, K, fmt, room = a
        s = lib.fp4_gemm(BUF, BUF, BUF, BUF, BUF, BUF, M, N, K, fmt, BUF, WS, room, LAYOUTS, None)
        r = launches()
        assert s == 0, s
        for l in r: l["ends"] = max(p + n * c * 4 for p, n, c in l["sums"]) - WS
    else:
        M, N, K = a
        s = getattr(lib, what)(BUF, M, K, 32, BUF, BUF, N, 0, BUF, 16, None)
        r = launches()
        assert s == 0, s
    print(json.dumps(r))
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    if not LIB.exists():
        from paper_2509_23202_amd import build
        build.build(verbose=False)
    d = tmp_path_factory.mktemp("dispatch")
    (d / "hip.c").write_text(HIP)
    subprocess.run([cc, "-shared", "-fPIC", "-w", "-o", str(d / "hip.so"), str(d / "hip.c")], check=True)

    def ask(*requests):
        r = subprocess.run([sys.executable, "-c", HOST, str(d / "hip.so"), str(LIB)], input=json.dumps(requests), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [json.loads(l) for l in r.stdout.splitlines()]

    return ask


def nv16_width(kernel):
    return {"Li4ELi2E": 128, "Li4ELi4E": 256, "Li8ELi4E": 512}[kernel.split("gemm_nv16_kernelI")[1][:8]]


@pytest.mark.parametrize("shapes", [NV16_HALF_ROWS, NV16_TWO_LAUNCHES, NV16_NARROW, NV16_ONE_ROUND, NV16_512_COLUMNS], ids=["half_rows", "two_launches", "narrow", "one_round", "512_columns"])
def test_nvfp4_products_for_many_tokens_run_in_the_tiles_that_their_tests_name(host, shapes):
    for (M, N, K), widths in shapes.items():
        need = host(["bytes", OP_GEMM, M, N, K, NV])[0]
        x16, *runs = host(["device", 0, 256], ["variant", NO_CODES], ["gemm", M, N, K, NV, need])[2]
        assert "nv_x16" in x16["kernel"] and [nv16_width(r["kernel"]) for r in runs] == widths, (M, N, K)


@pytest.mark.parametrize("shapes", [NV16_PARTS, NV16_PARTS_SHORT_K, NV16_PARTS_HALF_ROWS, NV16_PARTS_ROOM], ids=["parts", "short_k", "half_rows", "room"])
def test_nvfp4_products_in_parts_run_in_the_tiles_that_their_tests_name(host, shapes):
    """With the size that promises the fastest call too, which is the one for parts where the other kernel is out of the question."""
    for (M, N, K), width in shapes.items():
        full, fastest = host(["device", 0, 256], ["variant", NO_CODES], ["bytes", OP_SPLIT, M, N, K, NV], ["bytes", 7, M, N, K, NV])[2:]
        assert full == fastest
        x16, tiles, sums = host(["device", 0, 256], ["variant", NO_CODES], ["gemm", M, N, K, NV, full])[2]
        assert "nv_x16" in x16["kernel"] and nv16_width(tiles["kernel"]) == width and "nv16_reduce" in sums["kernel"], (M, N, K)


@pytest.mark.parametrize("fmt", [MX, NV])
def test_a_plan_is_made_for_the_device_that_is_current(host, fmt):
    """A thread that goes on to a device with fewer compute units plans for that one, as a thread that starts there."""
    big, small = ["device", 0, 256], ["device", 1, 64]
    for ask in (["bytes", OP_SPLIT, 201, 4096, 14336, fmt], ["gemm", 201, 4096, 14336, fmt, 1 << 30], ["gemm", 48, 4096, 8192, fmt, 1 << 30]):
        alone = host(small, ask)[-1]
        assert host(big, ask, small, ask)[-1] == alone
        assert host(big, ask)[-1] != alone


@pytest.mark.parametrize("call", ["fp4_fused_linear", "fp4_w4a16_linear"])
@pytest.mark.parametrize("cus", [32, 255, 256, 304])
def test_few_token_linears_start_one_workgroup_per_compute_unit(host, call, cus):
    """Row-blocks of one more and of as many as there are compute units, K of one batch of fragments and of two."""
    for N in (16 * cus, 16 * cus + 8, 4096, 4104):
        for K in (4096, 4224):
            (launch,) = host(["device", 0, cus], [call, 4, N, K])[1]
            assert launch["grid"][0] == min((N + 15) // 16, cus), (N, K)


@pytest.mark.parametrize("fmt,M,N,K", [(MX, 97, 2056, 14336), (MX, 201, 4096, 14336), (NV, 128, 8192, 28672), (NV, 300, 4096, 4096), (NV, 256, 8192, 28672),
                                       (NV, 320, 8192, 8192), (NV, 129, 4104, 12288)])
def test_split_runs_have_the_parts_that_their_workspace_holds(host, fmt, M, N, K):
    """Room for every number of parts up to the best one: a run in at most as many, whose partial sums end inside the workspace; more room
    than the best run needs changes nothing."""
    start = ["device", 0, 256], ["variant", NO_CODES if fmt == NV else 0]
    base, full = host(*start, ["bytes", OP_GEMM, M, N, K, fmt], ["bytes", OP_SPLIT, M, N, K, fmt])[2:]
    base = (base + 255) // 256 * 256
    part = M * N * 4
    assert full >= base + 2 * part
    best, more = host(*start, ["gemm", M, N, K, fmt, full], ["gemm", M, N, K, fmt, full + 7 * part])[2:]
    assert best == more and best[-1]["ends"] == full
    for n in range(1, (full - base) // part + 1):
        for room in (base + n * part, base + (n + 1) * part - 1):
            run = host(*start, ["gemm", M, N, K, fmt, room])[2]
            assert ("reduce" in run[-1]["kernel"]) == (n >= 2), room
            assert max(l["ends"] for l in run) <= room


@pytest.mark.parametrize("M,K", [(1, 235520), (2, 117760), (3, 77824), (4, 58368)])
def test_fused_linear_takes_the_one_shot_kernel_where_lds_does_not_hold_the_codes(host, M, K):
    held, over = (host(["device", 0, 256], ["fp4_fused_linear", M, 24, k])[1] for k in (K, K + 128))
    assert "gemm_few_stream_kernel" in held[0]["kernel"] and "gemm_fused_decode_kernel" in over[0]["kernel"]


@pytest.mark.parametrize("M,N,K,kernel", [(1, 512, 1152, "gemm_skinny_kernel"), (16, 2048, 1536, "gemm_skinny_kernel"), (7, 1024, 2048, "Li1ELi1ELi1E"),
                                          (5, 16384, 1280, "gemm_skinny_kernel"), (16, 4096, 1536, "Li1ELi1ELi1E"), (16, 2048, 2048, "Li1ELi1ELi1E"),
                                          (8, 6144, 2048, "Li1ELi1ELi2E"), (8, 40960, 1152, "Li1ELi1ELi3E"), (55, 42752, 2560, "Li4ELi1ELi3E"),
                                          (20, 57344, 3072, "Li2ELi1ELi2E"), (12, 24576, 1536, "Li1ELi1ELi3E"), (1, 28672, 4096, "Li1ELi1ELi2E"),
                                          (16, 4096, 14336, "Li1ELi4ELi2E"), (16, 14336, 14336, "Li1ELi4ELi3E"), (2, 10240, 5120, "Li1ELi2ELi3E"),
                                          (20, 14336, 14336, "Li2ELi4ELi2E")])
def test_mxfp4_few_tokens_take_the_buffers_that_suit_their_walk(host, M, N, K, kernel):
    """One-shot kernel, or token blocks, batches per row-block and buffers of the persistent one."""
    (launch,) = host(["device", 0, 256], ["gemm", M, N, K, MX, 0])[1]
    assert kernel in launch["kernel"], launch


@pytest.mark.parametrize("M,N,K,buffers", [(4, 4096, 4096, 1), (1, 4104, 4096, 2), (3, 768, 4224, 2), (4, 2048, 6144, 2), (2, 7168, 8192, 2), (2, 7176, 8192, 3), (4, 8192, 8192, 3), (1, 8192, 8192, 3), (1, 28672, 8192, 2),
                                           (4, 57344, 7168, 2), (2, 8200, 8192, 3), (4, 28672, 7296, 3), (4, 57344, 8320, 2)])
def test_fused_linear_takes_the_buffers_that_suit_its_walk(host, M, N, K, buffers):
    (launch,) = host(["device", 0, 256], ["fp4_fused_linear", M, N, K])[1]
    assert f"gemm_few_stream_kernelILb1ELb0ELi{buffers}E" in launch["kernel"], launch


@pytest.mark.parametrize("M,N,K,tile,parts", [(119, 8320, 24576, (128, 128), 3), (108, 8570, 27136, (128, 128), 3), (230, 6248, 26752, (256, 128), 4),
                                               (201, 8190, 28672, (256, 128), 4), (220, 17152, 28416, (256, 256), 3), (201, 4096, 14336, (64, 128), 2), (201, 6144, 4096, (64, 128), 1)])
def test_mxfp4_tiles_and_parts_of_long_and_narrow_layers(host, M, N, K, tile, parts):
    runs = host(["device", 0, 256], ["gemm", M, N, K, MX, 1 << 30])[1]
    assert f"gemm_mx_kernelILi{tile[0]}ELi{tile[1]}E" in runs[0]["kernel"] and runs[0]["grid"][1] == parts and len(runs) == (2 if parts > 1 else 1), runs


@pytest.mark.parametrize("M,N,K,last", [(134, 18560, 3840, 6), (161, 18432, 3840, 33), (642, 1368, 2048, 2), (129, 12352, 3968, 1), (320, 8192, 8192, 64), (520, 1368, 2048, 0), (520, 1368, 3072, 0)])
def test_nvfp4_parts_with_their_half_tiles_last(host, M, N, K, last):
    """Split runs hand out the tiles of a last row of at most 64 tokens last, as half tiles: from K = 4096 on, and below it where all whole
    tiles' parts are a workgroup for every compute unit or less, and the half ones' come on top."""
    full = host(["bytes", OP_SPLIT, M, N, K, NV])[0]
    runs = host(["device", 0, 256], ["variant", NO_CODES], ["gemm", M, N, K, NV, full])[2]
    assert "nv16_reduce" in runs[-1]["kernel"] and runs[-1]["sums"][1][2] == last * N


@pytest.mark.parametrize("M,N,K,blocks", [(57, 56400, 1024, 2), (41, 28456, 1280, 2), (57, 59008, 1024, 4), (41, 28456, 2176, 4), (33, 14344, 128, 4), (64, 13824, 8320, 2), (32, 16384, 8320, 2)])
def test_nvfp4_33_to_64_tokens_row_blocks_per_workgroup(host, M, N, K, blocks):
    (launch,) = host(["device", 0, 256], ["gemm", M, N, K, NV, 0])[1]
    assert f"gemm_skinny_nt_kernelILi1ELi{blocks}E" in launch["kernel"], launch
