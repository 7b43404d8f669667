"""What the host code decides, without a GPU: a small program links the built library, takes the place of the HIP
runtime's calls and of the launches it looks at, and prints what these were given."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2602_08007_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include <dlfcn.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "gemm.h"
#include "small.h"
#include "tsr.h"
static char *ws, *ws_end;
static int device = 0;
static const char* name_of(const void* symbol) {
    Dl_info at{};
    return dladdr(symbol, &at) && at.dli_sname ? at.dli_sname : "?";
}
extern "C" {
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s) {
    *g = *b = dim3(1); *n = 0; *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t, hipStream_t) {
    printf("launch %s\n", name_of(kernel));
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* kernel, hipFuncAttribute, int) {
    printf("lds %p %d\n", kernel, device);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
}
namespace tsr {
hipError_t launch_gram64(const Gram64Block* table, const Gram64Block* single, int blocks, int, int max_splits, hipStream_t) {
    for (int i = 0; i < blocks; ++i) {
        const Gram64Block& b = table ? table[i] : *single;
        const size_t bytes = b.splits > 1 ? (size_t)b.k * b.k * b.splits * sizeof(double) : 0;
        const bool inside = !bytes || ((char*)b.part >= ws && (char*)b.part + bytes <= ws_end);
        printf("gram64 %d %d %d %d %d\n", b.rows, b.k, b.splits, b.chunk, inside && b.splits <= max_splits);
    }
    return hipSuccess;
}
hipError_t launch_project_one(const ProjectOne&, int, int, int, hipStream_t) { printf("project_one\n"); return hipSuccess; }
hipError_t launch_lift_one(const LiftOne&, int, int, hipStream_t) { printf("lift_one\n"); return hipSuccess; }
}
static int call(int m, int n, int r) {                         // the projection and the lift of one matrix
    float* a = (float*)0x10000;
    const size_t bytes = tsr_project_workspace_bytes(m, n, r), lift = tsr_backproject_workspace_bytes(m, n, r);
    if (tsr_project_core(a, 0, m, n, n, a, a, r, 1.0f, 0, a, 0, (void*)0x100000, bytes, nullptr) != TSR_OK) return 3;
    return tsr_backproject_apply(a, m, n, n, a, a, a, r, 1.0f, 0.0f, 1.0f, 0, (void*)0x100000, lift, nullptr) == TSR_OK ? 0 : 4;
}
// a plan of fp32 blocks m n r, its workspace in bytes and the launches of a step
static int step(int workers, int count, char** dims) {
    std::vector<tsr_matrix_desc> d(count);
    float* a = (float*)0x10000;
    for (int i = 0; i < count; ++i) {
        d[i] = tsr_matrix_desc{};
        d[i].m = atoi(dims[3 * i]); d[i].n = atoi(dims[3 * i + 1]); d[i].r = atoi(dims[3 * i + 2]);
        d[i].G = a; d[i].ldg = d[i].ldw = d[i].n; d[i].g_stride = (long long)d[i].m * d[i].n;
        d[i].W = d[i].U = d[i].V = d[i].M = d[i].Vm = d[i].C = d[i].D = a;
    }
    const size_t bytes = tsr_plan_workspace_bytes(d.data(), count, workers, 0, 0, 0);
    printf("bytes %zu\n", bytes);
    tsr_plan* plan = nullptr;
    if (tsr_plan_create(d.data(), count, workers, 0, 0, 0, aligned_alloc(256, bytes), bytes, nullptr, &plan) != TSR_OK) return 5;
    const tsr_hyper h{1e-3f, 0.0f, 0.9f, 0.999f, 1e-8f, 1.0f};
    return tsr_step_batched(plan, 1, &h, nullptr) == TSR_OK ? 0 : 6;
}
// refreshes of one matrix on two devices in turn
static int devices(int m, int n, int r) {
    float* a = (float*)0x10000;
    const size_t bytes = tsr_refresh_workspace_bytes(m, n, r, 0);
    for (int d : {0, 1, 0, 1}) {
        device = d;
        if (tsr_refresh_rsvd(a, 0, m, n, n, a, r, 0, 1, a, a, a, (void*)0x100000, bytes, nullptr) != TSR_OK) return 7;
    }
    return 0;
}
// "devices" m n r; "call" m n r; "step" workers, then m n r per block; or the refresh of a plan: g_dtype r p, then m n per block
int main(int argc, char** argv) {
    if (!strcmp(argv[1], "call")) return call(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
    if (!strcmp(argv[1], "devices")) return devices(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
    if (!strcmp(argv[1], "step")) return step(atoi(argv[2]), (argc - 3) / 3, argv + 3);
    const int g = atoi(argv[1]), r = atoi(argv[2]), p = atoi(argv[3]), count = (argc - 4) / 2;
    std::vector<tsr_matrix_desc> d(count);
    float* a = (float*)0x10000;
    for (int i = 0; i < count; ++i) {
        d[i] = tsr_matrix_desc{};
        d[i].m = atoi(argv[4 + 2 * i]); d[i].n = atoi(argv[5 + 2 * i]); d[i].r = r;
        d[i].G = a; d[i].g_dtype = g; d[i].ldg = (d[i].n + 7) / 8 * 8; d[i].ldw = d[i].n;
        d[i].W = d[i].U = d[i].V = d[i].M = d[i].Vm = d[i].C = d[i].D = a;
    }
    const size_t bytes = tsr_plan_workspace_bytes(d.data(), count, 1, g, 1, p);
    ws = (char*)aligned_alloc(256, bytes);                     // (nothing but tables is written to it)
    ws_end = ws + bytes;
    tsr_plan* plan = nullptr;
    if (tsr_plan_create(d.data(), count, 1, g, 1, p, ws, bytes, nullptr, &plan) != TSR_OK) return 1;
    std::vector<const float*> omegas(count, a);
    if (tsr_refresh_batched(plan, omegas.data(), 1, nullptr) != TSR_OK) return 2;
    tsr_plan_destroy(plan);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    import paper_2602_08007_amd as tsr  # noqa: F401  (builds the library if it is not there)
    where = tmp_path_factory.mktemp("host")
    src, exe = where / "program.cpp", where / "program"
    src.write_text(PROGRAM)
    build = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                            "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe),
                            "-rdynamic", os.path.join(PKG, "libtsr.so"), "-Wl,-rpath," + PKG,
                            "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-ldl", "-Wl,-rpath," + os.path.join(ROCM, "lib")],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True)
        assert out.returncode == 0, (out.returncode, out.stderr)
        return [ln.split() for ln in out.stdout.splitlines()]
    return run


@pytest.mark.parametrize("g", [0, 1])
@pytest.mark.parametrize("r,dims", [(16, [(32000, 2048)] * 2), (128, [(32000, 2048)] * 2), (24, [(32000, 1024)]),
                                    (16, [(2048, 2048)] * 4 + [(2048, 5461)] * 2 + [(5461, 2048)])])
def test_gram_matrices_are_cut_into_row_pieces(program, g, r, dims):
    """The fp64 Gram matrices of a few tall blocks: about 200 waves a launch and more, no wave with more than
    2048 rows (some 60 us), the partial matrices inside the workspace.  Blocks with bf16 gradients as well, whose other
    Gram matrices are computed elsewhere."""
    rows = [tuple(map(int, ln[1:])) for ln in program(g, r, 8, *[x for d in dims for x in d]) if ln[0] == "gram64"]
    assert len(rows) % len(dims) == 0 and len(rows) >= 2 * len(dims)
    for at in range(0, len(rows), len(dims)):
        launch = rows[at:at + len(dims)]
        waves = 0
        for n, k, splits, chunk, inside in launch:
            assert inside and k == r + 8 and splits * chunk >= n
            assert -(-n // splits) <= 2048, (n, k, splits)
            tiles = -(-k // 32)
            waves += splits * tiles * (tiles + 1) // 2
        if max(n for n, *_ in launch) >= 32000:
            assert waves >= 190, launch


# (the sizes of the comment at the rule: with more than 128 units the general kernels are up to a quarter faster
# there, as they are for the projection of square and wide matrices above r = 96)
@pytest.mark.parametrize("m,n,r,project,lift", [
    (512, 1376, 64, True, True), (8000, 512, 64, True, True), (2000, 1000, 128, True, True), (1000, 2000, 96, True, True),
    (512, 512, 128, True, True), (4000, 512, 128, True, True), (512, 8000, 72, False, True), (3000, 1024, 72, False, False),
    (3000, 1000, 128, False, False), (1024, 1024, 128, False, True), (512, 4000, 128, False, True), (4096, 4096, 64, False, False),
    (300, 300, 129, False, False)])
def test_kernels_of_one_small_matrix(program, m, n, r, project, lift):
    taken = [ln[0] for ln in program("call", m, n, r) if ln[0] != "launch"]
    assert taken == ["project_one"] * project + ["lift_one"] * lift


# partials of G V (m x r outputs): 8, 16, 56 of few outputs, none; of U^T P: 8, 4, 2, 56
@pytest.mark.parametrize("m,n,r,shared", [(1024, 1024, 130, [False, False]), (512, 2048, 200, [False, False]),
                                          (130, 9000, 130, [True, False]), (8000, 130, 130, [True])])
def test_reductions_that_share_the_partials(program, m, n, r, shared):
    reductions = [ln[1] for ln in program("call", m, n, r) if ln[0] == "launch" and "splitk_reduce" in ln[1]]
    assert ["wide" in x for x in reductions] == shared, reductions


# plans of blocks at least four times as high as wide beside others: earlier sizes of their workspaces, which programs
# may hold, and the products of their lift (one more where the tall blocks' intermediate lies on their columns' side)
@pytest.mark.parametrize("dims,workers,earlier,products", [
    ([(2172, 2975, 450), (1044, 854, 2), (610, 45, 24)], 2, 58298368, 2), ([(35, 214, 3), (1009, 90, 1)], 1, 18944, 2),
    ([(209, 86, 1), (193, 30, 10)], 2, 32768, 2), ([(2048, 512, 64)] * 3, 1, 11032320, 2),
    ([(32000, 512, 128)] * 2 + [(512, 512, 128)] * 4, 1, 80789760, 3)])
def test_plans_with_tall_blocks(program, dims, workers, earlier, products):
    out = program("step", workers, *[x for d in dims for x in d])
    assert int(out[0][1]) <= earlier
    # behind Adam: the lift
    names = [ln[1] for ln in out if ln[0] == "launch"]
    at = max(i for i, x in enumerate(names) if "adam" in x)
    lift = [x for x in names[at + 1:] if "gemm" in x]
    assert len(lift) == products, names


@pytest.mark.parametrize("r,kernels", [(72, 1), (136, 1), (500, 3)])
def test_large_lds_is_allowed_on_each_device(program, r, kernels):
    """Kernels with more than 64 KB of dynamic LDS: the attribute is set once per kernel and device."""
    lds = [tuple(ln[1:]) for ln in program("devices", 1000, 1000, r) if ln[0] == "lds"]
    assert len(lds) == len(set(lds)), lds
    assert {k for k, d in lds if d == "0"} == {k for k, d in lds if d == "1"}
    assert len({k for k, _ in lds}) >= kernels
