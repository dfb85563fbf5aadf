// Context lifetime, errors and scratch.
#include "common.h"

#include <cstdlib>
#include <cstring>
#include <new>
#include <utility>

int set_error(rbffd_ctx ctx, int code, const char* fmt, ...) {
    if (ctx) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(ctx->err, sizeof(ctx->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

namespace {
void free_blocks(SpareMemory::Block (&b)[2]) {
    for (SpareMemory::Block& q : b) {
        if (q.p) (void)hipFree(q.p);
        q = SpareMemory::Block{};
    }
}
}  // namespace

hipError_t device_alloc(SpareMemory* spare, void** p, size_t bytes) {
    for (;;) {
        *p = nullptr;
        const hipError_t e = hipMalloc(p, bytes);
        if (e == hipSuccess) return e;
        *p = nullptr;
        (void)hipGetLastError();  // not for the next call to find
        std::lock_guard<std::mutex> lock(spare->mu);
        if (!spare->block[0].p && !spare->block[1].p) return e;
        free_blocks(spare->block);
    }
}

bool spare_take(SpareMemory* spare, size_t bytes, SpareMemory::Block& out) {
    {
        std::lock_guard<std::mutex> lock(spare->mu);
        SpareMemory::Block* best = nullptr;
        for (SpareMemory::Block& b : spare->block)
            if (b.p && b.bytes >= bytes && b.bytes / 4 <= bytes && (!best || b.bytes < best->bytes)) best = &b;
        if (best) {
            out = *best;
            *best = SpareMemory::Block{};
            return true;
        }
    }
    out.bytes = bytes;
    return device_alloc(spare, &out.p, bytes) == hipSuccess;
}

void spare_give(SpareMemory* spare, const SpareMemory::Block (&blocks)[2], bool keep) {
    SpareMemory::Block drop[2] = {blocks[0], blocks[1]};
    if (!drop[0].p) return;  // an operator that got no memory
    if (keep && blocks[0].bytes + blocks[1].bytes <= SPARE_MAX) {
        std::lock_guard<std::mutex> lock(spare->mu);
        if (spare->open)
            for (int q = 0; q < 2; ++q) std::swap(spare->block[q], drop[q]);
    }
    free_blocks(drop);
}

void spare_leave(SpareMemory* spare, bool context) {
    bool last;
    {
        std::lock_guard<std::mutex> lock(spare->mu);
        if (context) {
            spare->open = false;
            free_blocks(spare->block);
        }
        last = --spare->owners == 0;
    }
    if (last) delete spare;
}

int ensure_scratch(rbffd_ctx ctx, size_t bytes) {
    if (bytes <= ctx->scratch_bytes) return RBFFD_OK;
    if (ctx->scratch) {
        // work already enqueued may still read the old buffer
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        HIP_TRY(ctx, hipFree(ctx->scratch));
        ctx->scratch = nullptr;
        ctx->scratch_bytes = 0;
    }
    size_t want = bytes + bytes / 4 + (1u << 20);
    if (device_alloc(ctx->spare, &ctx->scratch, want) != hipSuccess) {
        return set_error(ctx, RBFFD_E_NOMEM, "cannot allocate %zu bytes of scratch", want);
    }
    ctx->scratch_bytes = want;
    return RBFFD_OK;
}

extern "C" void rbffd_default_opts(rbffd_weight_opts* o) {
    if (!o) return;
    std::memset(o, 0, sizeof(*o));
    o->n = 31;
    o->kernel = RBFFD_KERNEL_MQ;
    o->poly_degree = 2;
    o->eps_mode = RBFFD_EPS_FIXED;
    o->eps_fixed = 2.0;
    o->kappa_target = 1e12;
    o->eps_tol = 1e-4;
    o->bracket_lo = 0.05;
    o->bracket_hi = 20.0;
    o->band_lo = 1e11;
    o->band_hi = 1e13;
    o->rank_tol = 1e-10;
    o->band_stop = 0;
    o->max_expand = 8;
}

extern "C" int rbffd_create(rbffd_ctx* out, void* stream) {
    if (!out) return RBFFD_E_ARG;
    rbffd_ctx c = new (std::nothrow) rbffd_ctx_s();
    if (!c) return RBFFD_E_NOMEM;
    c->stream = reinterpret_cast<hipStream_t>(stream);
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return RBFFD_E_HIP;
    }
    if (noalloc_scratch_setup(c, c->device) != RBFFD_OK) {
        delete c;
        return RBFFD_E_HIP;
    }
    c->spare = new (std::nothrow) SpareMemory();
    if (!c->spare) {
        delete c;
        return RBFFD_E_NOMEM;
    }
    c->spare->device = c->device;
    *out = c;
    return RBFFD_OK;
}

extern "C" int rbffd_destroy(rbffd_ctx ctx) {
    if (!ctx) return RBFFD_E_ARG;
    if (ctx->scratch) {
        (void)hipStreamSynchronize(ctx->stream);
        (void)hipFree(ctx->scratch);
    }
    if (ctx->batch) {
        (void)hipStreamSynchronize(ctx->stream);
        (void)hipFree(ctx->batch);
    }
    spare_leave(ctx->spare, true);
    delete ctx;
    return RBFFD_OK;
}

extern "C" const char* rbffd_last_error(rbffd_ctx ctx) { return ctx ? ctx->err : "null context"; }
