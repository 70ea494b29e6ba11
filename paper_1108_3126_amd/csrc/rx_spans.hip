// The span kernels of rx_match, rx_match_first and their fixed-length forms
// (see rx_spans.h): a searched program over equal spans of the strings' bytes.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "rx_internal.h"
#include "rx_spans.h"

namespace rx {

namespace {

struct SpanArgs {
    SpanProg prog;
    SpanText text;
    SpanOut out;
    const int64_t* skip;   // rx_match's layout slot (see taken_by_sliced)
    int64_t skip_id;
};

// The results before any span runs (a kernel, not a memset: it may be captured).
template <class V>
__global__ __launch_bounds__(256) void k_fill(V* __restrict__ out, int64_t n, V v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = v;
}

// (as many wavefronts per SIMD as the LDS of narrow sets lets in)
template <int W, int T, bool FIRST>
__global__ __launch_bounds__(T, W <= 2 ? 6 : W <= 4 ? 5 : 1) void k_spans(SpanArgs a) {
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr int WP = span_row_words(W);
    if (a.skip && __hip_atomic_load(a.skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2 * a.skip_id) return;
    const int64_t o0 = a.text.offsets ? a.text.offsets[0] : 0;
    const int64_t oN = a.text.offsets ? a.text.offsets[a.text.n] : a.text.n * a.text.stride;
    const int64_t total = oN - o0 + 15;
    if (oN <= o0) return;
    const int B = span_bytes(total, (int64_t)gridDim.x * T);
    const int64_t regions = (total + T * B - 1) / (T * B);
    const int64_t per = (regions + gridDim.x - 1) / gridDim.x, r0 = blockIdx.x * per;
    const int64_t r1 = r0 + per < regions ? r0 + per : regions;
    if (r0 >= r1) return;
    uint32_t* M = lds;
    uint32_t* N = M + 256 * WP;
    uint32_t* F = N + 257 * WP;
    span_tables<W, T>(a.prog, M, N, F);
    span_regions<W, T, FIRST>(a.prog, a.text, a.out, o0, oN, B, r0, r1, M, N, F, F + a.prog.L * WP);
}

template <int W, bool FIRST>
int launch_spans_w(const LaunchArgs& a, const SpanArgs& k, int cus) {
    constexpr int T = span_threads(W);
    const int lds = 4 * span_lds_words(W, a.L, T);
    if (lds > 64 * 1024)   // (the widest program's size: another thread's call must not lower it before the launch)
        if (hipError_t e = hipFuncSetAttribute((const void*)k_spans<W, T, FIRST>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               4 * span_lds_words(W, 32 * W, T)))
            return (int)e;
    int per_cu = (160 * 1024) / (lds + 256);
    if (per_cu > 2048 / T) per_cu = 2048 / T;
    if (per_cu < 1) per_cu = 1;
    hipLaunchKernelGGL((k_spans<W, T, FIRST>), dim3((unsigned)(cus * per_cu)), dim3(T), (size_t)lds,
                       (hipStream_t)a.stream, k);
    return (int)hipGetLastError();
}

}  // namespace

int launch_spans_fill(const LaunchArgs& a) {
    const int64_t blocks = (a.n + 255) / 256;
    const dim3 grid((unsigned)(blocks < 4096 ? blocks : 4096));
    if (a.first_pos)
        hipLaunchKernelGGL((k_fill<int64_t>), grid, dim3(256), 0, (hipStream_t)a.stream, a.first_pos, a.n, (int64_t)-1);
    else
        hipLaunchKernelGGL((k_fill<uint8_t>), grid, dim3(256), 0, (hipStream_t)a.stream, a.out, a.n, (uint8_t)0);
    return (int)hipGetLastError();
}

namespace {
__global__ void k_span_long_begin(int64_t* slot, int64_t id, uint8_t* out, int64_t* first) {
    __hip_atomic_store(slot, 2 * id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (first) *first = -1;
    else *out = 0;
}
}  // namespace

int launch_span_long_begin(const LongGate& gate, uint8_t* out, int64_t* first, void* stream) {
    hipLaunchKernelGGL(k_span_long_begin, dim3(1), dim3(1), 0, (hipStream_t)stream, const_cast<int64_t*>(gate.slot),
                       gate.id, out, first);
    return (int)hipGetLastError();
}

int launch_spans(const LaunchArgs& a) {
    SpanArgs k;
    k.prog = {a.first, a.follow, a.bytemask, a.L, a.prefix};
    k.text = {a.bytes, a.offsets, a.stride, a.n};
    k.out = {a.out, a.first_pos, a.undone, kSpanLongLimit};
    k.skip = a.skip;
    k.skip_id = a.skip_id;
    int cus = 0;
    if (hip_cu_count(&cus) || cus <= 0) cus = 256;
    switch (a.W) {
#define RX_SPAN_CASE(w) \
    case w: return a.first_pos ? launch_spans_w<w, true>(a, k, cus) : launch_spans_w<w, false>(a, k, cus);
        RX_SPAN_CASE(1) RX_SPAN_CASE(2) RX_SPAN_CASE(3) RX_SPAN_CASE(4) RX_SPAN_CASE(5) RX_SPAN_CASE(6)
        RX_SPAN_CASE(7) RX_SPAN_CASE(8) RX_SPAN_CASE(9) RX_SPAN_CASE(10) RX_SPAN_CASE(11) RX_SPAN_CASE(12)
        RX_SPAN_CASE(13) RX_SPAN_CASE(14) RX_SPAN_CASE(15) RX_SPAN_CASE(16)
#undef RX_SPAN_CASE
    default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace rx
