// sg_split: Algorithm 1 (KV index splitting and reordering), one wavefront
// per row of the KV index, or one workgroup where the rows are few and long.
//
// The row is walked in 64-entry chunks.  Each lane gathers the mask value of
// its entry (operator 1); three ballots give, for every lane, how many earlier
// lanes carry each mask value, so the stable partitions (operators 2, 3) and
// the stable descending sort by mask value (operators 4, 5) are all prefix
// popcounts plus a running per-value count.  For a reordered row a first pass
// counts the remote and local entries, which fixes where the local and pad
// blocks start; without reordering the row is read once (the 64-request
// decode step's split: 37.3 M entries, 0.34 ms with both passes).  Each pass
// takes four chunks at a time, issuing all their loads together.
#include "sg_internal.h"

namespace sg {

constexpr int SPLIT_WAVES = 4;
constexpr int SPLIT_GROUP = 4;     // 64-entry chunks whose loads are issued together

__global__ __launch_bounds__(64 * SPLIT_WAVES) void split_kernel(
    int rows, const int32_t *__restrict__ row_off, int64_t total, const int32_t *__restrict__ kv_index,
    const int8_t *__restrict__ mask, int64_t mask_bytes, const int64_t *__restrict__ mask_off,
    const int32_t *__restrict__ mask_len, int reorder, int32_t *__restrict__ out_index,
    int32_t *__restrict__ local, int32_t *__restrict__ remote, int32_t *__restrict__ n_local,
    int32_t *__restrict__ n_remote, int32_t *__restrict__ n_kept) {
    const int r = blockIdx.x * SPLIT_WAVES + threadIdx.x / 64;
    if (r >= rows) return;
    const int lane = threadIdx.x % 64;
    int64_t o = row_off[r], e = row_off[r + 1];
    if (o < 0 || e < o || e > total) {  // bad device metadata: empty row
        if (lane == 0) {
            n_local[r] = 0;
            n_remote[r] = 0;
            if (n_kept) n_kept[r] = 0;
        }
        return;
    }
    const int64_t n = e - o;
    const int64_t moff = mask_off[r];
    const int32_t mlen = moff >= 0 ? mask_len[r] : 0;   // a negative offset makes every entry a pad
    const uint64_t lt = lanemask_lt();

    // The loads of SPLIT_GROUP chunks are issued together (indices, then mask
    // values at clamped addresses), so a group costs two memory round trips.
    const bool has_mask = mask_bytes > 0;
    auto load_group = [&](int64_t c, int32_t (&t)[SPLIT_GROUP], int (&m)[SPLIT_GROUP]) {
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) t[u] = kv_index[o + min<int64_t>(c + u * 64 + lane, n - 1)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            const bool ok = has_mask && t[u] >= 0 && t[u] < mlen && moff + t[u] < mask_bytes;
            const int x = has_mask ? mask[ok ? moff + t[u] : 0] : 0;
            m[u] = ok && (x == 1 || x == 2) ? x : 0;
        }
    };
    // pass 1 (reordered rows only): count remote and local entries, which fix
    // where the local and pad blocks start in the reordered row
    int64_t n2 = 0, n1 = 0;
    for (int64_t c = 0; reorder && c < n; c += 64 * SPLIT_GROUP) {
        int32_t t[SPLIT_GROUP];
        int m[SPLIT_GROUP];
        load_group(c, t, m);
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            const bool in = c + u * 64 + lane < n;
            n2 += __popcll(__ballot(in && m[u] == 2));
            n1 += __popcll(__ballot(in && m[u] == 1));
        }
    }
    // pass 2: write the partitions
    int64_t c2 = 0, c1 = 0, c0 = 0;
    for (int64_t c = 0; c < n; c += 64 * SPLIT_GROUP) {
        int32_t tt[SPLIT_GROUP];
        int mm[SPLIT_GROUP];
        load_group(c, tt, mm);
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            const int64_t i = c + u * 64 + lane;
            const int32_t t = tt[u];
            const int m = mm[u];
            const uint64_t b2 = __ballot(i < n && m == 2);
            const uint64_t b1 = __ballot(i < n && m == 1);
            const uint64_t b0 = __ballot(i < n && m == 0);
            if (i < n) {
                if (m == 2) {
                    const int64_t p = c2 + __popcll(b2 & lt);
                    remote[o + p] = t;
                    if (reorder) out_index[o + p] = t;
                } else if (m == 1) {
                    const int64_t p = c1 + __popcll(b1 & lt);
                    local[o + p] = t;
                    if (reorder) out_index[o + n2 + p] = t;
                } else if (reorder) {
                    out_index[o + n2 + n1 + c0 + __popcll(b0 & lt)] = t;
                }
            }
            c2 += __popcll(b2);
            c1 += __popcll(b1);
            c0 += __popcll(b0);
        }
    }
    // the running counts are the totals (equal to pass 1's when it ran)
    n1 = c1;
    n2 = c2;
    // unused tails of the compacted outputs
    for (int64_t i = n1 + lane; i < n; i += 64) local[o + i] = -1;
    for (int64_t i = n2 + lane; i < n; i += 64) remote[o + i] = -1;
    if (lane == 0) {
        n_local[r] = (int32_t)n1;
        n_remote[r] = (int32_t)n2;
        if (n_kept) n_kept[r] = (int32_t)(n1 + n2);
    }
}

// One workgroup per row, for few long rows (a single request's step): every
// wavefront takes SPLIT_GROUP chunks of a sweep of WG_SWEEP entries, the counts
// of the wavefronts meet in LDS, and each then knows its places.  A row of one
// sweep is read once, also when it is reordered; a longer reordered row is
// counted in a first pass.
constexpr int SPLIT_WG_WAVES = 16;
constexpr int WG_SWEEP = SPLIT_WG_WAVES * SPLIT_GROUP * 64;

__global__ __launch_bounds__(64 * SPLIT_WG_WAVES) void split_wg_kernel(
    const int32_t *__restrict__ row_off, int64_t total, const int32_t *__restrict__ kv_index,
    const int8_t *__restrict__ mask, int64_t mask_bytes, const int64_t *__restrict__ mask_off,
    const int32_t *__restrict__ mask_len, int reorder, int32_t *__restrict__ out_index,
    int32_t *__restrict__ local, int32_t *__restrict__ remote, int32_t *__restrict__ n_local,
    int32_t *__restrict__ n_remote, int32_t *__restrict__ n_kept) {
    __shared__ int cnt[2][3][SPLIT_WG_WAVES];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int64_t o = row_off[r], e = row_off[r + 1];
    if (o < 0 || e < o || e > total) {  // bad device metadata: empty row
        if (tid == 0) {
            n_local[r] = 0;
            n_remote[r] = 0;
            if (n_kept) n_kept[r] = 0;
        }
        return;
    }
    const int64_t n = e - o;
    const int64_t moff = mask_off[r];
    const int32_t mlen = moff >= 0 ? mask_len[r] : 0;   // a negative offset makes every entry a pad
    const bool has_mask = mask_bytes > 0;
    int32_t t[SPLIT_GROUP];
    int m[SPLIT_GROUP];                                 // mask value, -1 past the row
    uint64_t b2[SPLIT_GROUP], b1[SPLIT_GROUP], b0[SPLIT_GROUP];
    int sweep = 0;
    // loads the sweep at c and counts it: before2 / before1 / before0 entries
    // of each value in earlier wavefronts, all2 / all1 / all0 in the sweep
    int before2, before1, before0, all2, all1, all0;
    auto take = [&](int64_t c) {
        const int64_t w0 = c + wave * (SPLIT_GROUP * 64) + lane;
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) t[u] = kv_index[o + min<int64_t>(w0 + u * 64, n - 1)];
        __builtin_amdgcn_sched_barrier(0);
        int n2 = 0, n1 = 0, n0 = 0;
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            const bool ok = has_mask && t[u] >= 0 && t[u] < mlen && moff + t[u] < mask_bytes;
            const int x = has_mask ? mask[ok ? moff + t[u] : 0] : 0;
            m[u] = w0 + u * 64 >= n ? -1 : ok && (x == 1 || x == 2) ? x : 0;
        }
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            b2[u] = __ballot(m[u] == 2);
            b1[u] = __ballot(m[u] == 1);
            b0[u] = __ballot(m[u] == 0);
            n2 += __popcll(b2[u]);
            n1 += __popcll(b1[u]);
            n0 += __popcll(b0[u]);
        }
        int (*cs)[SPLIT_WG_WAVES] = cnt[sweep++ & 1];   // two sets: one barrier per sweep is enough
        if (lane == 0) {
            cs[0][wave] = n0;
            cs[1][wave] = n1;
            cs[2][wave] = n2;
        }
        __syncthreads();
        before2 = before1 = before0 = all2 = all1 = all0 = 0;
#pragma unroll
        for (int w = 0; w < SPLIT_WG_WAVES; ++w) {
            const int x0 = cs[0][w], x1 = cs[1][w], x2 = cs[2][w];
            before0 += w < wave ? x0 : 0;
            before1 += w < wave ? x1 : 0;
            before2 += w < wave ? x2 : 0;
            all0 += x0;
            all1 += x1;
            all2 += x2;
        }
    };
    int64_t n2 = 0, n1 = 0;
    if (reorder && n > WG_SWEEP)
        for (int64_t c = 0; c < n; c += WG_SWEEP) {     // uniform
            take(c);
            n2 += all2;
            n1 += all1;
        }
    const uint64_t lt = lanemask_lt();
    int64_t c2 = 0, c1 = 0, c0 = 0;
    for (int64_t c = 0; c < n; c += WG_SWEEP) {
        take(c);
        if (n <= WG_SWEEP) {
            n2 = all2;
            n1 = all1;
        }
        int64_t p2 = c2 + before2, p1 = c1 + before1, p0 = c0 + before0;
#pragma unroll
        for (int u = 0; u < SPLIT_GROUP; ++u) {
            if (m[u] == 2) {
                const int64_t p = p2 + __popcll(b2[u] & lt);
                remote[o + p] = t[u];
                if (reorder) out_index[o + p] = t[u];
            } else if (m[u] == 1) {
                const int64_t p = p1 + __popcll(b1[u] & lt);
                local[o + p] = t[u];
                if (reorder) out_index[o + n2 + p] = t[u];
            } else if (m[u] == 0 && reorder) {
                out_index[o + n2 + n1 + p0 + __popcll(b0[u] & lt)] = t[u];
            }
            p2 += __popcll(b2[u]);
            p1 += __popcll(b1[u]);
            p0 += __popcll(b0[u]);
        }
        c2 += all2;
        c1 += all1;
        c0 += all0;
    }
    // unused tails of the compacted outputs
    for (int64_t i = c1 + tid; i < n; i += 64 * SPLIT_WG_WAVES) local[o + i] = -1;
    for (int64_t i = c2 + tid; i < n; i += 64 * SPLIT_WG_WAVES) remote[o + i] = -1;
    if (tid == 0) {
        n_local[r] = (int32_t)c1;
        n_remote[r] = (int32_t)c2;
        if (n_kept) n_kept[r] = (int32_t)(c1 + c2);
    }
}

}  // namespace sg

using namespace sg;

extern "C" int sg_split(void *stream, int rows, const int32_t *row_off, int64_t total,
                        const int32_t *kv_index, const int8_t *mask, int64_t mask_bytes,
                        const int64_t *mask_off, const int32_t *mask_len, int reorder, int32_t *out_index, int32_t *local,
                        int32_t *remote, int32_t *n_local, int32_t *n_remote, int32_t *n_kept) {
    SG_REQUIRE(rows >= 0 && total >= 0 && mask_bytes >= 0, SG_EINVAL, "sg_split: negative size");
    if (rows == 0) return SG_OK;
    SG_REQUIRE(row_off && n_local && n_remote && mask_off && mask_len, SG_EINVAL, "sg_split: null pointer");
    SG_REQUIRE(total == 0 || (kv_index && mask && local && remote), SG_EINVAL, "sg_split: null pointer");
    SG_REQUIRE(!reorder || total == 0 || out_index, SG_EINVAL, "sg_split: reorder needs out_index");
    // Few rows (fewer than two per CU) of at least 256 entries on average leave
    // a wavefront per row walking alone, two memory round trips per 256
    // entries: a workgroup takes a row (64 rows of 2,293 entries, reordered:
    // 30.7 -> 6.2 us).
    if (rows < 2 * device_cus() && total >= (int64_t)rows * 256) {
        split_wg_kernel<<<rows, 64 * SPLIT_WG_WAVES, 0, as_stream(stream)>>>(
            row_off, total, kv_index, mask, mask_bytes, mask_off, mask_len, reorder ? 1 : 0, out_index, local, remote,
            n_local, n_remote, n_kept);
        return launch_status("sg_split");
    }
    const int blocks = (int)ceil_div(rows, SPLIT_WAVES);
    split_kernel<<<blocks, 64 * SPLIT_WAVES, 0, as_stream(stream)>>>(
        rows, row_off, total, kv_index, mask, mask_bytes, mask_off, mask_len, reorder ? 1 : 0, out_index, local, remote,
        n_local, n_remote, n_kept);
    return launch_status("sg_split");
}
