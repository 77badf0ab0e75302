// A copy to the host that fails after others were queued: the call reports
// it, and no earlier copy is still in flight into the caller's memory when
// it returns.  The HIP calls that the library makes on the way are defined
// here, so nothing reaches a device: launches do nothing, a copy is noted as
// in flight until the stream is waited for, and one chosen copy fails.
// Run by tests/test_abi_copy_failure.py on the CPU; prints "copy failure ok".
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <vector>

#include "../include/mtp.h"

static int to_host = 0;          // copies to the host asked for
static int in_flight = 0;        // of them, queued and not waited for
static int fail_at = -1;         // the one that fails

extern "C" {
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind kind, hipStream_t) {
    if (kind != hipMemcpyDeviceToHost) return hipSuccess;
    if (to_host++ == fail_at) return hipErrorOutOfMemory;
    ++in_flight;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    in_flight = 0;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s) {
    *g = *b = dim3(1);
    *n = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
}

static int failures = 0;
#define CHECK(cond)                                                        \
    do {                                                                   \
        if (!(cond)) {                                                     \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
            ++failures;                                                    \
        }                                                                  \
    } while (0)

static void* fake(uintptr_t k) { return reinterpret_cast<void*>(k << 20); }

// Fails each copy of a call in turn, then none.
template <class F>
static void every_copy(int copies, F call) {
    for (int i = 0; i < copies; ++i) {
        to_host = 0;
        fail_at = i;
        CHECK(call() == MTP_EHIP);
        CHECK(to_host == i + 1);
        CHECK(in_flight == 0);
    }
    to_host = 0;
    fail_at = -1;
    CHECK(call() == MTP_OK);
    CHECK(to_host == copies && in_flight == 0);
}

static mtp_config config() {
    mtp_config c{};
    c.n_layers = 2; c.d_model = 256; c.n_heads = 4; c.d_ff = 256; c.vocab = 1025; c.eos_id = 1024; c.n_phone = 512;
    c.max_pos = 256; c.k_heads = 2; c.topk_max = 4; c.max_batch = 3; c.max_prompt = 64; c.max_new = 8; c.eos_min = 8;
    c.page_size = 16; c.dtype = MTP_DTYPE_F32; c.flags = MTP_FLAG_NO_GRAPH;
    return c;
}

int main() {
    const mtp_buffers b{fake(1), static_cast<const float*>(fake(2)), fake(3), fake(4)};
    {   // NAR: three utterances, whose target rows are three runs of rows
        mtp_config c = config();
        c.flags |= MTP_FLAG_NAR;
        mtp_ctx* ctx = nullptr;
        CHECK(mtp_create(&c, &b, nullptr, &ctx) == MTP_OK);
        const std::vector<int32_t> ids(600, 1);
        const int32_t pl[3] = {5, 6, 7}, ql[3] = {4, 3, 2}, tl[3] = {20, 30, 25};
        CHECK(mtp_nar_prepare(ctx, 3, ids.data(), pl, ids.data(), ql, ids.data(), tl) == MTP_OK);
        CHECK(mtp_nar_run(ctx) == MTP_OK);
        std::vector<float> logits(75 * 1024);
        every_copy(3, [&] { return mtp_nar_get_logits(ctx, 1, logits.data()); });
        mtp_destroy(ctx);
    }
    {   // decode step and lattices
        mtp_config c = config();
        mtp_ctx* ctx = nullptr;
        CHECK(mtp_create(&c, &b, nullptr, &ctx) == MTP_OK);
        const std::vector<int32_t> ids(200, 1);
        const int32_t pl[3] = {5, 6, 7}, al[3] = {10, 11, 12};
        int32_t tok[6], cnt[3];
        std::vector<float> f(3 * 8 * 64);
        std::vector<int32_t> i(3 * 8 * 64);
        CHECK(mtp_prefill(ctx, 3, ids.data(), pl, ids.data(), al) == MTP_OK);
        every_copy(2, [&] { return mtp_decode_step(ctx, 2, 3, tok, cnt); });
        every_copy(5, [&] { return mtp_get_lattice(ctx, i.data(), f.data(), f.data(), i.data(), i.data()); });
        CHECK(mtp_set_selection(ctx, MTP_LATTICE_UNION, 0) == MTP_OK);
        CHECK(mtp_decode_step(ctx, 2, 3, tok, cnt) == MTP_OK);
        every_copy(6, [&] {
            return mtp_get_union_lattice(ctx, i.data(), i.data(), f.data(), f.data(), i.data(), i.data());
        });
        mtp_destroy(ctx);
    }
    if (failures) {
        std::fprintf(stderr, "%d checks failed\n", failures);
        return 1;
    }
    std::printf("copy failure ok\n");
    return 0;
}
