// Exact top-k of a row held in registers by one workgroup of 1024 threads,
// shared by sg_topk and the decode-time selection.
//
// Scores are mapped to 32-bit keys of the same order (NaN -> 1, the lowest key
// of an entry; -0 -> +0; 0 stands for a slot past the row's end).  The k-th
// largest key is found in the row's own key range: the keys between the row's
// largest and smallest are counted in 2048 equal bins from the top (LDS
// atomics), and the bin that holds the k-th is searched again, at most three
// times in all.  A bin whose entries are all taken ends the search; one of at
// most SEL_LIST entries is gathered into LDS and ranked by comparing all with
// all.  (Bins of the fixed top 11 bits would give four bins per power of two;
// over a row's own range of a few dozen powers a bin is 10 to 40 times finer,
// and one count is nearly always enough.)
//
// Layout: wavefront w holds the row's consecutive entries [w, w + 1) * 64 * it
// (it = the row's entries per thread), entry i * 64 + lane of them in its
// lane's key[i]: loads are whole 256-byte pieces whatever the row's alignment.
// The kept entries of 64 consecutive ones are one ballot, whose halves go to
// lanes 2i and 2i + 1; each lane then knows its place from one scan and writes
// its own ids, so ids come out ascending with ties resolved to the lower index.
//
// Bound by instruction issue and barriers of one CU, not by the row's bytes:
// scalar work per entry (ballots, their counts) costs as much as ten vector
// instructions, so the loops over a thread's entries keep to vector
// instructions.  Figures: topk.hip.
#pragma once

#include <utility>

#include "sg_internal.h"

namespace sg {

constexpr int TOPK_THREADS = 1024;
constexpr int TOPK_WAVES = TOPK_THREADS / 64;
constexpr int SEL_BITS = 11;
constexpr int SEL_BINS = 1 << SEL_BITS;
constexpr int SEL_LIST = 256;                 // entries ranked by comparing all with all
static_assert(SEL_BINS == 2 * TOPK_THREADS, "a thread scans two bins");

__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 1u;  // NaN: below every number (-inf is 0x007fffff)
    if (u == 0x80000000u) u = 0u;                     // -0 ranks as +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// DPP lane moves of a wavefront scan: row shifts by 1, 2, 4, 8, then the last
// lane of a row to the next rows.
#define SG_SCAN_STEPS(STEP) STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)

// inclusive sum over the 64 lanes
__device__ __forceinline__ int wave_scan_incl(int x) {
#define SG_STEP(C, R) x += __builtin_amdgcn_update_dpp(0, x, C, R, 0xf, false);
    SG_SCAN_STEPS(SG_STEP)
#undef SG_STEP
    return x;
}
// largest / smallest over the 64 lanes, in lane 63
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
#define SG_STEP(C, R) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, C, R, 0xf, false));
    SG_SCAN_STEPS(SG_STEP)
#undef SG_STEP
    return x;
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
#define SG_STEP(C, R) x = min(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, C, R, 0xf, false));
    SG_SCAN_STEPS(SG_STEP)
#undef SG_STEP
    return x;
}

// x with lane `lane` replaced by the wavefront-uniform value v: the intrinsic
// by its own name (there is no builtin for it; through inline assembly the
// compiler would not place the wait states between the compare that makes v
// and this read of it)
__device__ int writelane(int v, int lane, int x) __asm("llvm.amdgcn.writelane.i32");
template <int L>
__device__ __forceinline__ uint32_t set_lane(uint32_t x, uint32_t v) {
    return (uint32_t)writelane((int)v, L, (int)x);
}

struct SelectSmem {
    uint32_t hist[SEL_BINS];
    uint32_t list[SEL_LIST];          // 16-byte reads
    uint32_t wmax[TOPK_WAVES], wmin[TOPK_WAVES];
    int wsum[TOPK_WAVES], weq[TOPK_WAVES];
    uint32_t digit, thr;
    int rem, in_bin, nlist;
};

// Entries per thread of a row of n.
__device__ __forceinline__ int select_items(int n) { return (n + TOPK_THREADS - 1) / TOPK_THREADS; }

// Index of the entry in key[0] of this thread (key[i]: 64 i further).
__device__ __forceinline__ int select_entry(int it) {
    return (int)(threadIdx.x / 64) * 64 * it + (int)(threadIdx.x % 64);
}

// f(key[i], i) for the thread's items, STEP at a time up to the row's `it`.
template <int ITEMS, int STEP, int I0, typename F, int... J>
__device__ __forceinline__ void select_step(const uint32_t (&key)[ITEMS], F &f, std::integer_sequence<int, J...>) {
    (f(key[I0 + J], std::integral_constant<int, I0 + J>{}), ...);
}
template <int ITEMS, int STEP, int I0, typename F>
__device__ __forceinline__ void select_each(const uint32_t (&key)[ITEMS], int it, F &f) {
    if constexpr (I0 < ITEMS) {
        if (I0 >= it) return;          // uniform
        select_step<ITEMS, STEP, I0>(key, f, std::make_integer_sequence<int, STEP>{});
        select_each<ITEMS, STEP, I0 + STEP>(key, it, f);
    }
}

// Writes the ids of the kk largest keys (ties: lower id), ascending, to
// out[0 .. kk).  0 < kk <= number of entries; keys of slots past the row are
// 0.  Every thread of the workgroup must call it.
template <int ITEMS>
__device__ __forceinline__ void select_top(const uint32_t (&key)[ITEMS], int it, int kk, int32_t *out,
                                           SelectSmem &sm) {
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // loops over the thread's keys stop at the row's own items, four at a time
    // (slots past them hold key 0, which changes nothing below)
    constexpr int STEP = ITEMS < 4 ? ITEMS : 4;
    static_assert(ITEMS % STEP == 0, "whole steps");
    auto each = [&](auto &&f) { select_each<ITEMS, STEP, 0>(key, it, f); };

    // the row's key range (key - 1: an empty slot does not count for the smallest)
    uint32_t mx = 0u, mn = 0xffffffffu;
    each([&](uint32_t k, auto) {
        mx = max(mx, k);
        mn = min(mn, k - 1u);
    });
    mx = wave_max_u32(mx);
    mn = wave_min_u32(mn);
    if (lane == 63) {
        sm.wmax[wave] = mx;
        sm.wmin[wave] = mn;
    }
    reinterpret_cast<uint2 *>(sm.hist)[tid] = make_uint2(0u, 0u);
    if (tid < SEL_LIST) sm.list[tid] = 0u;
    if (tid == 0) sm.nlist = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < TOPK_WAVES; ++w) {
        mx = max(mx, sm.wmax[w]);
        mn = min(mn, sm.wmin[w]);
    }
    // Keys at or below `hi` and above hi - width are searched; bin d holds those
    // with (hi - key) >> shift == d.  (Empty slots, key 0, are below them all.)
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)mx);
    uint32_t width = hi - (uint32_t)__builtin_amdgcn_readfirstlane((int)mn);     // largest - smallest + 1
    int shift = max(0, 32 - __builtin_clz((width - 1u) | 1u) - SEL_BITS);
    int rem = kk;
    uint32_t thr;
    bool all;                          // every key >= thr is taken; else `rem` of those equal to it
    for (;;) {
        // Lanes of one bin wait for one another in an atomic.  Where more than a
        // few of the wavefront's first entries share the bin of the first or the
        // last of them, that bin is counted in a register.  (Equal keys, not
        // equal bins, were looked for, and empty slots were counted as one bin:
        // 1,024 rows of 20K keys, all but one value within 1% of another 120 ->
        // 56 us, of spread keys 34 -> 33; 4,096 rows of 9,000 keys 112 -> 76.)
        const uint32_t o0 = hi - key[0], d0 = o0 >> shift;
        const uint64_t act = __ballot(o0 < width);
        uint32_t crowd = 0u;           // the crowded bin
        int shared = 0;                // lanes in it
        if (act != 0) {                // uniform
            const uint32_t da = (uint32_t)__builtin_amdgcn_readlane((int)d0, __ffsll((unsigned long long)act) - 1);
            const uint32_t dz = (uint32_t)__builtin_amdgcn_readlane((int)d0, 63 - __clzll((long long)act));
            const int na = __popcll(__ballot(o0 < width && d0 == da)), nz = __popcll(__ballot(o0 < width && d0 == dz));
            crowd = na >= nz ? da : dz;
            shared = max(na, nz);
        }
        if (shared > 8) {
            int mine = 0;
            each([&](uint32_t k, auto) {
                const uint32_t o = hi - k, d = o >> shift;
                if (o < width) {
                    if (d == crowd) ++mine;
                    else atomicAdd(&sm.hist[d], 1u);
                }
            });
            mine = wave_scan_incl(mine);
            if (lane == 63) atomicAdd(&sm.hist[crowd], (uint32_t)mine);
        } else {
            each([&](uint32_t k, auto) {
                const uint32_t o = hi - k;
                if (o < width) atomicAdd(&sm.hist[o >> shift], 1u);
            });
        }
        __syncthreads();
        // thread t owns bins 2t and 2t + 1, from the top
        const uint2 c = reinterpret_cast<const uint2 *>(sm.hist)[tid];
        const int sum = (int)(c.x + c.y);
        const int scan = wave_scan_incl(sum);
        if (lane == 63) sm.wsum[wave] = scan;
        __syncthreads();
        int before = 0;
#pragma unroll
        for (int w = 0; w < TOPK_WAVES; ++w) before += w < wave ? sm.wsum[w] : 0;
        const int excl = before + scan - sum;
        if (excl < rem && rem <= excl + sum) {
            const bool first = rem <= excl + (int)c.x;
            sm.digit = (uint32_t)(2 * tid) + (first ? 0u : 1u);
            sm.rem = rem - excl - (first ? 0 : (int)c.x);
            sm.in_bin = (int)(first ? c.x : c.y);
        }
        reinterpret_cast<uint2 *>(sm.hist)[tid] = make_uint2(0u, 0u);    // for another pass
        __syncthreads();
        const uint32_t d = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.digit);
        const int in_bin = __builtin_amdgcn_readfirstlane(sm.in_bin);
        rem = __builtin_amdgcn_readfirstlane(sm.rem);
        hi -= d << shift;
        width = min(1u << shift, hi);      // the bin's keys: (hi - width, hi], above 0
        if (in_bin == rem) {
            thr = hi - width + 1u;
            all = true;
            break;
        }
        if (shift == 0) {              // a bin is one key
            thr = hi;
            all = false;
            break;
        }
        if (in_bin <= SEL_LIST) {
            each([&](uint32_t k, auto) {
                if (hi - k < width) {
                    const int p = atomicAdd(&sm.nlist, 1);
                    if (p < SEL_LIST) sm.list[p] = k;
                }
            });
            __syncthreads();
            if (tid < in_bin) {
                const uint32_t mine = sm.list[tid];
                int above = 0, atleast = 0;
                for (int j = 0; j < in_bin; j += 4) {      // entries past in_bin are 0
                    const uint4 x = *reinterpret_cast<const uint4 *>(&sm.list[j]);
                    above += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
                    atleast += (x.x >= mine) + (x.y >= mine) + (x.z >= mine) + (x.w >= mine);
                }
                if (above < rem && rem <= atleast) {       // equal entries write the same values
                    sm.thr = mine;
                    sm.rem = rem - above;
                    sm.in_bin = atleast - above;
                }
            }
            __syncthreads();
            thr = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.thr);
            rem = __builtin_amdgcn_readfirstlane(sm.rem);
            all = __builtin_amdgcn_readfirstlane(sm.in_bin) == rem;
            break;
        }
        shift = max(0, 32 - __builtin_clz((width - 1u) | 1u) - SEL_BITS);
    }

    // Kept entries: lanes 2i and 2i + 1 take the halves of item i's ballot (32
    // items at a time).
    constexpr int HALVES = 32;
    constexpr int ROUNDS = (ITEMS + HALVES - 1) / HALVES;
    const uint32_t thr1 = all ? thr : thr + 1u;
    uint32_t take[ROUNDS], ties[ROUNDS];
    int mine = 0, eqs = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) take[r] = ties[r] = 0u;
    each([&](uint32_t k, auto i) {
        const uint64_t m = __ballot(k >= thr1);
        constexpr int I = decltype(i)::value, r = I / HALVES, l = 2 * (I % HALVES);
        take[r] = set_lane<l>(take[r], (uint32_t)m);
        take[r] = set_lane<l + 1>(take[r], (uint32_t)(m >> 32));
    });
    if (!all)
        each([&](uint32_t k, auto i) {
            const uint64_t m = __ballot(k == thr);
            constexpr int I = decltype(i)::value, r = I / HALVES, l = 2 * (I % HALVES);
            ties[r] = set_lane<l>(ties[r], (uint32_t)m);
            ties[r] = set_lane<l + 1>(ties[r], (uint32_t)(m >> 32));
        });
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        mine += __popc(take[r]);
        eqs += __popc(ties[r]);
    }
    mine = wave_scan_incl(mine);
    eqs = wave_scan_incl(eqs);
    if (lane == 63) {
        sm.wmax[wave] = (uint32_t)mine;
        sm.weq[wave] = eqs;
    }
    __syncthreads();
    int pos = 0, seen = 0;             // taken above the threshold and tied, in the wavefronts before
#pragma unroll
    for (int w = 0; w < TOPK_WAVES; ++w) {
        pos += w < wave ? (int)sm.wmax[w] : 0;
        seen += w < wave ? sm.weq[w] : 0;
    }
    pos += min(seen, rem);             // (no ties are listed when all are taken)
    const int base = wave * 64 * it;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        uint32_t m = take[r];
        const uint32_t e = ties[r];
        // the ties taken are the first `rem` of the row
        const int sc_eq = wave_scan_incl(__popc(e));
        int quota = rem - (seen + sc_eq - __popc(e));
        seen += __builtin_amdgcn_readlane(sc_eq, 63);
        if (!all) {
            uint32_t left = e;
            while (left != 0u && quota > 0) {
                m |= left & (0u - left);
                left &= left - 1u;
                --quota;
            }
        }
        const int n = __popc(m), sc = wave_scan_incl(n);
        int p = pos + sc - n;
        pos += __builtin_amdgcn_readlane(sc, 63);
        const int first = base + (r * HALVES + lane / 2) * 64 + (lane % 2) * 32;
        while (m != 0u) {
            out[p++] = first + __builtin_ctz(m);
            m &= m - 1u;
        }
    }
}

}  // namespace sg
