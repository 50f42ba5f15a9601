// Products whose panel table cannot be had: memory has run out, or the call is being captured on a stream that was warmed up with
// a smaller matrix.  No GPU: the runtime calls on the way are answered and written down here.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "../include/fuse.h"
#include <hip/hip_runtime.h>

static std::string calls;                // of the current step: l load, a allocation, p m r the three kernels of a plan
static size_t room = (size_t)1 << 40, largest = 0;
static bool capturing = false;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    if (capturing || n > room)
        return hipErrorOutOfMemory;
    calls += 'a';
    largest = n > largest ? n : largest;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipModuleLoadData(hipModule_t *m, const void *)
{
    calls += 'l';
    *m = nullptr;
    return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipModuleGetFunction(hipFunction_t *f, hipModule_t, const char *name)
{
    const char *k = !std::strcmp(name, "fuse_outer_prep") ? "p" : !std::strcmp(name, "fuse_outer_rows") ? "r" : !std::strncmp(name, "fuse_outer_", 11) ? "m" : "k";
    *f = (hipFunction_t)k;
    return hipSuccess;
}
hipError_t hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(int *n, hipFunction_t, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, hipStream_t, void **, void **)
{
    calls += *(const char *)f;
    return hipSuccess;
}
}

static int step(const char *what, int64_t rows, int64_t cols, int64_t nnz, int agg, size_t stream, const char *want)
{
    static const fuse_tok tok[] = {{FUSE_OP_MAIN, 0, 0.0}, {FUSE_OP_UVDOT, 0, 0.0}, {FUSE_OP_MUL, 0, 0.0}};
    fuse_expr e = {};
    e.toks = tok;
    e.ntoks = 3;
    void *at = (void *)0x10000;
    fuse_csr x = {};
    x.rowptr = at, x.colidx = (const int32_t *)at, x.vals = (const double *)at, x.rows = rows, x.cols = cols, x.nnz = nnz;
    fuse_dense u = {}, v = {};
    u.data = v.data = (double *)at, u.rows = rows, v.rows = cols, u.cols = v.cols = u.ld = v.ld = 100;
    calls.clear();
    const int rc = fuse_outer(&e, &x, &u, &v, nullptr, 0, agg, (double *)at, (void *)stream);
    const bool ok = rc == 0 && calls == want;
    std::printf("%-40s %d %s%s%s\n", what, rc, calls.c_str(), ok ? "" : "   expected ", ok ? "" : want);
    return !ok;
}

int main()
{
    int bad = 0;
    const int R = FUSE_AGG_RIGHT_MM, L = FUSE_AGG_LEFT_MM;
    bad += step("small", 1000, 1000, 20000, R, 64, "laam");                    // (arrival counters and workspace)
    bad += step("large", 100000, 40000, 4000000, R, 64, "lapmr");
    capturing = true;
    bad += step("large, captured, all there", 100000, 40000, 4000000, R, 64, "pmr");
    bad += step("larger table, captured", 400000, 40000, 16000000, R, 64, "m");
    capturing = false;
    bad += step("small, another stream", 1000, 1000, 20000, R, 128, "aam");
    capturing = true;
    bad += step("large, captured after a small one", 100000, 40000, 4000000, R, 128, "m");
    capturing = false;
    room = 1 << 20;
    bad += step("large, no room", 100000, 40000, 4000000, R, 192, "aam");
    bad += step("large, no room, captured", 100000, 40000, 4000000, R, 192, "m");
    room = (size_t)1 << 40;
    setenv("FUSE_OUTER_RUNS", "0", 1);
    bad += step("left_mm, row mapping", 40000, 100000, 4000000, L, 256, "laam");
    unsetenv("FUSE_OUTER_RUNS");
    room = largest;                                                           // for the transposed matrix and nothing beside it
    bad += step("left_mm, no room for the table", 40000, 100000, 4000000, L, 320, "laam");
    room = (size_t)1 << 40;
    bad += step("left_mm, within the workspace's slack", 40000, 100000, 4000000, L, 320, "pmr");
    return bad;
}
