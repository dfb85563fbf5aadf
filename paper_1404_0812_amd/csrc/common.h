// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <string>

#include "rbffd.h"

// Device memory of the context's last destroyed operator, kept for the next one
// of a similar size (the slab and the state workspace, SPARE_MAX bytes in all).
// Given back when the context is destroyed and whenever an allocation of the
// library fails.  Shared by the context and its operators, which may be
// destroyed later and by other threads.
struct SpareMemory {
    struct Block {
        void* p = nullptr;
        size_t bytes = 0;
    };
    std::mutex mu;
    int owners = 1;
    int device = 0;
    bool open = true;  // the context is alive
    Block block[2];
};
constexpr size_t SPARE_MAX = (size_t)2 << 30;

struct rbffd_ctx_s {
    hipStream_t stream = nullptr;
    int device = 0;
    char err[512] = {0};
    // growable scratch owned by the context
    void* scratch = nullptr;
    size_t scratch_bytes = 0;
    SpareMemory* spare = nullptr;
    // work list of the batched weights launch (kept apart from scratch, which kNN uses)
    void* batch = nullptr;
    size_t batch_bytes = 0;
};

// One slice of the operator: 64 consecutive internal rows of one surface.
struct OpSlice {
    int64_t off32;  // element offset of the slice in the off-diagonal arrays (n - 1 slots)
    int32_t n;      // stencil size of the slice's rows
    int32_t rows;   // rows in use (64 except at a surface's end)
    int32_t halo;   // distinct neighbour rows of the slice (<= OP_HALO_MAX), -1: too many
    int32_t pad;
};

// Largest slice neighbourhood staged in LDS by the stage kernels.
constexpr int OP_HALO_MAX = 640;

struct rbffd_op_s {
    rbffd_ctx ctx = nullptr;
    int64_t N = 0;        // rows in caller order (sum over surfaces)
    int64_t P = 0;        // internal rows, each surface padded to a multiple of 64
    int32_t n = 0;        // largest stencil size
    int32_t nsurf = 0;
    int64_t nslices = 0;
    int64_t slots = 0;    // off-diagonal slots of all slices
    OpSlice* slices = nullptr;    // device, nslices
    double* wd64 = nullptr;       // FP64 diagonal weight of every internal row (P)
    int32_t* idx32 = nullptr;     // off-diagonal slots 1..n-1 of row (slice, r) at off32 + slot_pos(k-1, n-1, r)
    double* w64 = nullptr;        // FP64 weights of those slots
    float* w32 = nullptr;         // FP32 weights of those slots (difference form)
    uint16_t* lidx = nullptr;     // slot entries as positions in the slice's halo list
    int32_t* halo = nullptr;      // OP_HALO_MAX sorted distinct neighbour rows per slice
    int32_t* perm = nullptr;      // internal row -> caller row (-1 for padding), P entries
    SpareMemory::Block slab;      // the one device allocation that holds the arrays above and the counters
    SpareMemory::Block work;      // state workspace (internal order), allocated on first use
    SpareMemory* spare = nullptr; // of the context that built it
    // vectors of the implicit (BDF) stepper, allocated on first use
    void* impl = nullptr;
    size_t impl_bytes = 0;
    // captured graph cache
    hipGraphExec_t graph = nullptr;
    // graph of KRYLOV_BATCH implicit-solver iterations, valid while its
    // vectors sit where they were when it was captured (kgraph_key)
    hipGraphExec_t kgraph = nullptr;
    const void* kgraph_key = nullptr;
    int graph_key_species = -1, graph_key_prec = -1, graph_key_react = -1, graph_key_steps = -1;
    double graph_key_dt = 0.0;
    double graph_key_D[2] = {0, 0};
    double graph_key_params[5] = {0, 0, 0, 0, 0};
    int graph_key_forced = 0;
    double graph_key_t0 = 0.0, graph_key_lam = 0.0;
    // device: int64 steps done by the forced stages, then int non-finite flag
    void* counters = nullptr;
    int* nonfinite_host = nullptr;  // pinned host copy of the flag
};

int set_error(rbffd_ctx ctx, int code, const char* fmt, ...);
// Look up the device address of the allocation-free call's array on `device`
// (current); once per device, at context creation.
int noalloc_scratch_setup(rbffd_ctx ctx, int device);
// Ensure ctx->scratch holds at least `bytes`; returns 0 or an error code.
int ensure_scratch(rbffd_ctx ctx, size_t bytes);
// hipMalloc; when it fails, once more without the spare memory.
hipError_t device_alloc(SpareMemory* spare, void** p, size_t bytes);
// A spare block of bytes .. 4 bytes, or a new one; false: out of memory.
bool spare_take(SpareMemory* spare, size_t bytes, SpareMemory::Block& out);
// The blocks of a destroyed operator, idle on the device, in place of those
// kept so far; freed instead with `keep` false or the context gone.
void spare_give(SpareMemory* spare, const SpareMemory::Block (&blocks)[2], bool keep);
// One owner less; the last deletes it.
void spare_leave(SpareMemory* spare, bool context);

#define HIP_TRY(ctx, call)                                                                   \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return set_error((ctx), RBFFD_E_HIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

// Internal entry points of the translation units.
int knn_internal(rbffd_ctx ctx, int64_t N, const double* xyz, int32_t n, int32_t* idx,
                 int32_t* perm);
