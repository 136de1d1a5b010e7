// sg_topk: exact budgeted top-k per unit row by a range-adaptive count
// (select_common.h).
//
// One workgroup of 1024 threads owns one (request, layer, KV head) row (or, for
// block selection, one request's row of L * M block importances) and holds it
// in registers, ITEMS keys per thread (up to 80); a row shorter than the
// call's longest uses only the items it needs, spread over all wavefronts.
// ITEMS = 32 is compiled for 64 VGPRs, so two workgroups share a CU, and one
// fits beside a score workgroup (208 VGPRs, two wavefronts per SIMD) when the
// select region runs a request pair's top-k beside the next pair's score.
//
// Against four fixed 8-bit digit passes with consecutive keys per thread (512
// threads for many long rows): 256 rows of 8K keys 14.5 -> 8.6 us, 1,024 rows
// of 2K to 32K keys 179 -> 41 us, one row of 32K block importances 41.7 ->
// 16.2 us (5.5 us of it its loads: what one CU draws from beyond its L2).
#include "select_common.h"

namespace sg {

// Wavefronts per SIMD: two workgroups per CU (64 VGPRs) while the row fits.
constexpr int topk_waves(int items) { return items <= 32 ? 8 : 4; }

template <int ITEMS>
__global__ __launch_bounds__(TOPK_THREADS) __attribute__((amdgpu_waves_per_eu(topk_waves(ITEMS)))) void topk_kernel(
    int B, const int32_t *__restrict__ cu_seqlens, int64_t T, const int32_t *__restrict__ cu_k, int64_t K_total,
    const float *__restrict__ scores, int32_t *__restrict__ idx) {
    __shared__ SelectSmem sm;
    const int b = blockIdx.x % B;
    const int64_t lh = blockIdx.x / B;
    const int tid = threadIdx.x;
    const int64_t c0 = cu_k[b], c1 = cu_k[b + 1];
    const int64_t s0 = cu_seqlens[b], s1 = cu_seqlens[b + 1];
    if (c0 < 0 || c1 < c0 || c1 > K_total) return;  // no writable segment
    int32_t *out = idx + lh * K_total + c0;
    const int64_t kk = c1 - c0;
    const int64_t N = s1 - s0;
    if (s0 < 0 || s1 < s0 || s1 > T || kk > N || N > (int64_t)ITEMS * TOPK_THREADS) {
        for (int64_t i = tid; i < kk; i += TOPK_THREADS) out[i] = -1;
        return;
    }
    if (kk == 0) return;
    if (kk == N) {  // everything is selected
        for (int64_t i = tid; i < kk; i += TOPK_THREADS) out[i] = (int32_t)i;
        return;
    }
    const float *row = scores + lh * T + s0;
    const int n = (int)N, it = select_items(n);
    const int entry0 = select_entry(it);
    // every load issued before the first key is made (an entry past the row reads its last one)
    float x[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i < it) x[i] = row[min(entry0 + i * 64, n - 1)];       // uniform
    uint32_t key[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) key[i] = i < it && entry0 + i * 64 < n ? order_key(x[i]) : 0u;
    select_top<ITEMS>(key, it, (int)kk, out, sm);
}

}  // namespace sg

using namespace sg;

extern "C" int sg_topk(void *stream, int B, int L, int Hkv, const int32_t *cu_seqlens, int64_t T, int max_seqlen,
                       const int32_t *cu_k, int64_t K_total, const float *scores, int32_t *idx) {
    SG_REQUIRE(B >= 1 && L >= 1 && Hkv >= 1, SG_EINVAL, "sg_topk: B, L, Hkv must be >= 1");
    SG_REQUIRE(T >= 0 && K_total >= 0 && max_seqlen >= 0, SG_EINVAL, "sg_topk: negative size");
    SG_REQUIRE(max_seqlen <= 80 * TOPK_THREADS, SG_EUNSUPPORTED, "sg_topk: max_seqlen %d above %d", max_seqlen,
               80 * TOPK_THREADS);
    if (K_total == 0) return SG_OK;
    SG_REQUIRE(cu_seqlens && cu_k && scores && idx, SG_EINVAL, "sg_topk: null pointer");
    const int64_t blocks = (int64_t)B * L * Hkv;
    SG_REQUIRE(blocks <= 0x7fffffff, SG_EINVAL, "sg_topk: too many rows");
    hipStream_t s = as_stream(stream);
    const unsigned grid = (unsigned)blocks;
    const int items = (int)ceil_div(std::max(max_seqlen, 1), TOPK_THREADS);
#define SG_TOPK(I) topk_kernel<I><<<grid, TOPK_THREADS, 0, s>>>(B, cu_seqlens, T, cu_k, K_total, scores, idx)
    if (items <= 2) SG_TOPK(2);
    else if (items <= 4) SG_TOPK(4);
    else if (items <= 8) SG_TOPK(8);
    else if (items <= 16) SG_TOPK(16);
    else if (items <= 32) SG_TOPK(32);
    else if (items <= 64) SG_TOPK(64);
    else SG_TOPK(80);    // block rows of up to 80 layers x 1024 blocks
#undef SG_TOPK
    return launch_status("sg_topk");
}
