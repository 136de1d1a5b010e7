// sg_score_topshare: selection-frequency importance when every window row
// picks a fixed share of the keys it sees.
//
// Row w of q head g (prompt position p = N - W + w) sees the n = p + 1 keys
// j <= p and picks those whose logit z_j = q . k_j / sqrt(d) is at or above
// its k-th largest, k = floor(n * ratio_bp / 10000) clamped to [1, n]; keys
// tied with the k-th largest are all picked.  counts[j] is the number of
// (q head, window row) pairs of the unit that pick key j.
//
// The k-th largest logit of every row is found exactly, in three passes over
// the logits (recomputed by the MFMA engine of sg_score each time) and a small
// sample:
//
//   sample : the logits of 512 to 2048 keys spread over the prompt (held in
//            registers) give each row an interval [a, b) that holds its k-th
//            largest logit with near certainty: the sample's quantiles 4.75
//            standard deviations around the wanted rank, or open ends with
//            a quarter of the sample's range to spare;
//   hist   : every logit of the row goes to one of 64 equal bins of [a, b), or
//            below or above it (LDS atomics, bins x rows); the chunk's bins go
//            into the unit's global histogram with integer atomics;
//   digit  : one thread per row finds the bin of the k-th largest (the keys
//            above or below the interval are one too, if few) and the smallest
//            and largest float in it;
//   again  : units with a row that the sample misjudged or whose bin holds more
//            than TS_CMAX keys take hist and digit once more, over the next
//            interval or that bin (every other unit returns at once);
//   gather : the values inside a row's bin (a few tens at most) are appended
//            to the row's list, in LDS, then in the workspace; of a bin that
//            still holds more (ties) the smallest and largest are kept;
//   pick   : the exact k-th largest among them is the row's threshold, or the
//            one value of a bin of ties;
//   radix  : rows still unresolved (different ties side by side, NaN) take an
//            exact radix select over the logits' bit patterns, one workgroup
//            per 32 rows with such a row (every other one returns at once);
//   count  : each key's picks, counted against the rows' thresholds.
//
// Against a radix select in 6-bit digits for all rows (three histogram passes,
// gather and count, one workgroup per CU in each): 32 layers x 8 heads of 8K
// keys, 256 rows each, at 20%: 1.14 -> 0.60-0.65 ms (sample 62, hist 187, digit
// 13, gather 195, pick 25, count 139 us, the three idle launches 15 us).  Rows of
// ties take hist again and the careful loop of gather.  8 layers of 8K keys,
// every logit zero / one of a few values / repeating every 64 keys: 0.29 / 0.30
// / 0.48 ms; with the radix select in gather's place 1.13 / 1.00 / 0.81, with one
// for all rows 0.63.
//
// A logit's bits are the same in every pass: the same MFMA operands in the
// same contraction order (C = K Q^T in hist and gather, Q K^T in count).  The
// passes work on the raw products q . k_j: the positive scale 1/sqrt(d) keeps
// their order.  Bins are a monotone function of the logit, so the bin's
// bounds are exact floats.  Values order as their bit patterns do: a NaN with
// the sign bit set below -inf, any other above +inf; -0 and +0 are equal
// floats and picked together.
#include <algorithm>

#include "score_tiles.h"

namespace sg {

constexpr int TS_BINS = 64;        // bins of a row's interval
constexpr int TS_CMAX = 92;        // keys a row may gather
constexpr int TS_ROW_WORDS = 99;   // workspace words per row: six below, the rest bins, then lists
constexpr int TS_UNIT_WORDS = 9;
static_assert(6 + TS_CMAX <= TS_ROW_WORDS && TS_BINS <= TS_CMAX, "the row lists take the bins' place");

// The call's workspace.
struct TsWork {
    float *xa, *xb;        // [rows] interval scale and offset, then the bounds of the row's bin
    uint32_t *need;        // [rows] rank inside the bin | keys in the bin << 16; 0: settled; TS_AGAIN; TS_TIED; TS_RADIX
    uint32_t *above;       // [rows] keys above the interval
    uint32_t *gcount;      // [rows] keys gathered
    float *thr;            // [rows] threshold
    uint32_t *hist;        // [units][TS_BINS][R] bins
    uint32_t *list;        // [rows][TS_CMAX] gathered values (in the bins' place)
    uint32_t *fail;        // [units] bit per 32 rows: a row needs the radix select
    uint32_t *again;       // [units] a row of the unit needs another histogram; TS_TIED_UNIT: one was left tied
};
constexpr uint32_t TS_TIED_UNIT = 2u;
constexpr uint32_t TS_AGAIN = 0xffffffffu;      // need: another histogram over the interval in xa, xb
constexpr uint32_t TS_RADIX = 0xfffffffeu;      // need: the radix select, between xa and xb (NaN: anywhere)
// need: more keys in the bin than a row may gather, in a bin that is narrow by
// now, so most likely equal: gather takes their smallest and largest order key
// (in the words of thr and gcount) instead of a list
constexpr uint32_t TS_TIED = 0xfffffffdu;
constexpr uint32_t TS_TIED_LANE = 0x80000000u;  // gather's count of a lane of such a row

__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t x = __float_as_uint(f);
    return x ^ ((uint32_t)((int32_t)x >> 31) | 0x80000000u);
}

__device__ __forceinline__ float key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// The float threshold of a row whose picks are the keys >= key.
__device__ __forceinline__ float threshold_value(uint32_t key) {
    constexpr uint32_t NEG_INF_KEY = 0x007fffffu;         // order_key(-inf); keys below it are NaN patterns
    return key < NEG_INF_KEY ? -INFINITY : key_value(key);
}

// The bin of logit x: with t = x * scale + offset, t in [1, 2) over the row's
// interval, the exponent and the top six mantissa bits of t count up through
// the interval's 64 bins (TS_LOW + 1 .. TS_LOW + 64); below it (negative t
// too) TS_LOW, above it TS_LOW + 65.  Signed compares put every bit pattern,
// NaN included, where its order is.
constexpr int TS_LOW = (0x3f800000 >> 17) - 1;
__device__ __forceinline__ int ts_bin(float x, float scale, float off) {
    const int b = (int)__float_as_uint(fmaf(x, scale, off)) >> 17;
    return min(max(b, TS_LOW), TS_LOW + TS_BINS + 1);
}

// The number of low bits that hold every set bit of the lanes' x.
__device__ __forceinline__ int wave_max_bits(uint32_t x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x |= (uint32_t)__shfl_xor((int)x, o, 64);
    return 32 - __builtin_clz(x | 1u) - (x == 0u ? 1 : 0);
}

// The rank (from the top) of the wanted key among the n a row sees.
__device__ __forceinline__ int64_t ts_rank(int64_t n, int ratio_bp) {
    return min(max(n, (int64_t)1), max((int64_t)1, n * ratio_bp / 10000));
}

// ---------------------------------------------------------------- sample

// One workgroup of NWV wavefronts per (unit, ROWS rows): wavefront w holds the
// logits of SPW sampled keys for those rows in registers, C = K Q^T, keys and
// queries straight from memory; a row leaves out the samples past its causal
// limit.  The rows' intervals are narrowed by counting the sample in 128 bins
// of the current interval (first [min, max]) and moving its ends to the bins of
// the bounding ranks, again (up to four times) while some row's interval holds
// many more samples than the ranks ask for (far outliers; the larger sample
// always twice).  Also clears the unit's counters.
template <typename T, int D, int NWV, int ROWS>
__global__ __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(2))) void ts_sample_kernel(
    int B, int L, int Hq, int Hkv, int W, const int32_t *__restrict__ cu_seqlens, int64_t T_,
    const T *__restrict__ q_win, const T *__restrict__ k, int64_t k_layer_rows, int ratio_bp, int64_t u0, TsWork ws) {
    using M = MT<T, D>;
    constexpr int NRB = ROWS / M::BM, SPW = 8192 / ROWS, NKB = SPW / M::BM, NS = SPW * NWV;
    constexpr int SB = 128, QB = SB / 4;       // bins of the sample; a quarter of them
    __shared__ uint32_t bins[SB + 1][ROWS];
    __shared__ float smin[NWV][ROWS], smax[NWV][ROWS], ra[ROWS], rs[ROWS];
    __shared__ int qsum[4][ROWS], found[4][ROWS];  // found: the bins of the two ranks and the samples above them
    const int R = (Hq / Hkv) * W, ngrp = (int)ceil_div(R, ROWS);
    const int64_t u = u0 + blockIdx.x / ngrp;
    const int grp = blockIdx.x % ngrp;
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int N = (int)g.N, tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // the rows' counters
    for (int i = tid; i < TS_BINS * ROWS; i += 64 * NWV) {
        const int row = grp * ROWS + i % ROWS;
        if (row < R) ws.hist[(u * TS_BINS + i / ROWS) * R + row] = 0u;
    }
    const int myrow = grp * ROWS + tid;        // threads 0 .. ROWS - 1: a row each
    const bool owner = tid < ROWS && myrow < R;
    if (owner) {
        ws.above[u * R + myrow] = 0u;
        ws.gcount[u * R + myrow] = 0u;
        if (myrow == 0) ws.fail[u] = ws.again[u] = 0u;
    }
    if (N < W) return;                         // uniform: the count pass writes zeros
    const T *qunit = q_win + (((int64_t)g.b * L + g.l) * Hq + (int64_t)g.h * (Hq / Hkv)) * W * D;
    const T *kunit = k + ((int64_t)g.l * k_layer_rows + (int64_t)g.h * T_ + g.s0) * D;
    // ns of the keys (one in eight, at least 512: a short prompt beside long
    // ones leaves wavefronts without keys, which only keep the barriers).  The
    // window's own keys are among them, for the rows that see them: where they
    // are the largest, in short prompts of rising logits, a sample of the keys
    // that every row sees misjudges them all (200 keys, a window of 64: 8 layers
    // 136 us against 83; 700 keys, a window of 512: 244 against 99).
    const int seen = N - W + 1, ns = min(N, max(512, min(NS, N / 8 / SPW * SPW)));
    const bool busy = wave * SPW < ns;         // uniform across the wavefront
    TA<T, D> qf[NRB][M::KS];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        const T *p = qunit + (int64_t)min(grp * ROWS + rb * M::BM + lane % M::BM, R - 1) * D;
#pragma unroll
        for (int ks = 0; ks < M::KS; ++ks) qf[rb][ks] = M::load_global(p, ks, lane);
    }
    TC<T, D> val[NKB][NRB];
    if (busy) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            const int i = wave * SPW + kb * M::BM + lane % M::BM;
            const T *p = kunit + (int64_t)sample_key(min(i, ns - 1), ns, N) * D;
            TA<T, D> kf[M::KS];
#pragma unroll
            for (int ks = 0; ks < M::KS; ++ks) kf[ks] = M::load_global(p, ks, lane);
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) val[kb][rb] = block_mma<T, D, true>(kf, qf[rb]);
        }
    }
    // values past a row's causal limit or past the sample (a short prompt)
    // become NaN, which every compare and minimum below leaves out; samples
    // below `early` have keys that every row sees
    const float per = (float)ns / (float)N;
    const int early = (int)((float)seen * per) - 1;
    if (busy && (wave + 1) * SPW > early) {    // uniform
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            const int i0 = wave * SPW + kb * M::BM, i = i0 + lane % M::BM;
            if (i0 + M::BM <= early) continue;
            const int key = i < ns ? sample_key(i, ns, N) : N;
#pragma unroll
            for (int v = 0; v < M::NV; ++v) {
                const int kv = __shfl(key, M::crow(v, lane), 64);
#pragma unroll
                for (int rb = 0; rb < NRB; ++rb) {
                    const int last = N - W + (grp * ROWS + rb * M::BM + lane % M::BM) % W;
                    val[kb][rb][v] = kv <= last ? val[kb][rb][v] : __builtin_nanf("");
                }
            }
        }
    }
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        float mn = INFINITY, mx = -INFINITY;
        if (busy) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int v = 0; v < M::NV; ++v) {
                    mn = fminf(mn, val[kb][rb][v]);
                    mx = fmaxf(mx, val[kb][rb][v]);
                }
        }
#pragma unroll
        for (int off = M::BM; off < 64; off <<= 1) {
            mn = fminf(mn, __shfl_xor(mn, off, 64));
            mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        }
        if (lane < M::BM) {
            smin[wave][rb * M::BM + lane] = mn;
            smax[wave][rb * M::BM + lane] = mx;
        }
    }
    __syncthreads();
    // a row's interval [a, b] and the sample ranks (from the top) that bound it
    // (thread t: row t % ROWS)
    const int col = tid % ROWS, quarter = tid / ROWS % 4;
    const bool scans = tid < 4 * ROWS;
    float a = smin[0][col], b = smax[0][col];
    for (int w = 1; w < NWV; ++w) {
        a = fminf(a, smin[w][col]);
        b = fmaxf(b, smax[w][col]);
    }
    const float top = b, quarter_range = 0.25f * (b - a);
    // the row's keys and, of them, the sampled ones: those of whole stretches
    // and, by its place, the one of the stretch that its last key is in
    const int nrow = seen + (grp * ROWS + col) % W, whole = min((int)((float)nrow * per), ns);
    const int srow = whole + (whole < ns && sample_key(whole, ns, N) < nrow ? 1 : 0);
    const int64_t kk = ts_rank(nrow, ratio_bp);
    const float p = (float)kk / (float)nrow, r = p * srow;
    // five standard deviations less a little; near the ends the wanted key lies inside the
    // sample's extremes unless all `r` expected samples beyond it are missing
    // (e^-11 from r = 11 on), else the interval is open there (r_hi < 0, r_lo > srow)
    const float spread = 4.75f * sqrtf(r * (1.f - p)) + 1.f;
    const int r_hi = max((int)floorf(r - spread), r >= 11.f ? 0 : -1);
    const int r_lo = min((int)ceilf(r + spread), (float)srow - r >= 11.f ? srow : srow + 1);
    for (int round = 0; round < 4; ++round) {
        const float sc = b > a ? (float)SB / (b - a) : 0.f;
        if (tid < ROWS) {
            ra[tid] = a;
            rs[tid] = sc;
            found[0][tid] = SB - 1;                    // ranks above or below every bin: keep that end
            found[1][tid] = 0;
            found[2][tid] = found[3][tid] = 0;
        }
        for (int i = tid; i < (SB + 1) * ROWS; i += 64 * NWV) (&bins[0][0])[i] = 0u;
        __syncthreads();
        if (busy) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                const int row = rb * M::BM + lane % M::BM;
                const float lo = ra[row], rsc = rs[row];
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int v = 0; v < M::NV; ++v) {
                        const float x = val[kb][rb][v];
                        // bin SB: above the interval (its upper end too, after the first round)
                        const int d = min((int)((x - lo) * rsc), round == 0 ? SB - 1 : SB);
                        if (x >= lo) atomicAdd(&bins[max(d, 0)][row], 1u);
                    }
            }
        }
        __syncthreads();
        // four threads per row scan a quarter of its bins each, from the top
        uint32_t c[QB];
        int sum = 0;
        if (scans) {
#pragma unroll
            for (int j = 0; j < QB; ++j) {
                c[j] = bins[(4 - quarter) * QB - 1 - j][col];
                sum += (int)c[j];
            }
            qsum[quarter][col] = sum;
        }
        __syncthreads();
        if (scans) {
            int cum = (int)bins[SB][col];
            for (int w = 0; w < quarter; ++w) cum += qsum[w][col];
#pragma unroll
            for (int j = 0; j < QB; ++j) {
                const int d = (4 - quarter) * QB - 1 - j, next = cum + (int)c[j];
                if (cum <= r_hi && next > r_hi) {      // the first sample past the upper rank
                    found[0][col] = d;
                    found[2][col] = cum;
                }
                if (cum < r_lo && (next >= r_lo || d == 0)) {      // down to the bin of the lower rank
                    found[1][col] = d;
                    found[3][col] = next;
                }
                cum = next;
            }
        }
        __syncthreads();
        const int hi_bin = found[0][col], lo_bin = found[1][col];
        const float step = (b - a) / (float)SB;
        const float na = a + lo_bin * step, nb = hi_bin == SB - 1 ? b : a + (hi_bin + 1) * step;
        if (nb > na) {
            a = na;
            b = nb;
        }
        const int want = min(r_lo, srow) - max(r_hi, 0);
        // (ties are not told apart, and an interval much narrower than its ends
        // are large could not place its values)
        const int wide = grp * ROWS + col < R && kk < nrow && b - a > 0x1p-11f * fmaxf(fabsf(a), fabsf(b)) &&
                         found[3][col] - found[2][col] > want + want / 2 + 8;
        if (__syncthreads_or(wide) == 0 && round >= (NS > 512 ? 1 : 0)) break;     // uniform
    }
    if (owner) {
        // open ends: room beyond the sample's extremes, where a few tens of
        // keys lie; those past the room are gathered as if it were a bin
        // (digit).  With an interval meant to cover them all, ranks at the
        // ends took hist again and the radix select (4 layers of 16K keys, the
        // largest or all but the smallest of each row: 832 and 1,135 us, now
        // 209 and 211)
        if (r_hi < 0) b = top + fmaxf(top - a, quarter_range);
        else if (b >= top) b = top + 1e-3f * (top - a);
        if (r_lo > srow) a -= fmaxf(b - a, quarter_range);
        // ties, a constant sample: no narrower than places every value to a
        // fraction of a bin with an offset in fp32 (ties fell outside: 4 layers
        // of 64K keys, logits of a few values, 3.03 ms, 0.86 now)
        const float tight = fmaxf(0x1p-12f * fmaxf(fabsf(a), fabsf(b)), 2e-20f);
        if (!(b - a >= tight)) {
            a -= 0.5f * tight;
            b += 0.5f * tight;
        }
        const float edge = 1e-3f * (b - a);    // (a tied value at an end stays inside)
        a -= edge;
        b += edge;
        const float scale = 1.f / (b - a), off = 1.f - a * scale;
        const bool ok = b > a && scale < INFINITY && scale > 0.f && fabsf(off) < INFINITY;
        ws.xa[u * R + myrow] = ok ? scale : 0.f;           // 0, 0: every logit below the interval
        ws.xb[u * R + myrow] = ok ? off : 0.f;
    }
}

// ---------------------------------------------------------------- hist

// Keys per LDS tile of the hist and gather passes: beside the bins or the
// lists, 64-key tiles leave room for two workgroups per CU at rows of 256 bytes
// a key up to four wavefronts and at 128 bytes always (fp32 at d = 128, and
// eight wavefronts at 256 bytes: one).
constexpr int TS_TILE_KEYS = 64;

// One block of the histogram pass.  A word of the bins holds two rows' counts
// (row blocks 2 i and 2 i + 1 of the wavefront, one after the other in a lane,
// so they never meet in one instruction); a chunk's counts stay below 2^16.
// No branch per value (it would split the block and undo the MFMA / vector
// interleave): values outside the interval go to the end bins.
template <typename T, int D, int NW, bool MASK>
struct HistStep {
    using M = MT<T, D>;
    static constexpr int NRB = QFrags<T, D>::NRB, WORDS = 32 * NW;
    uint32_t *hist;                 // LDS [TS_BINS + 2][WORDS]
    const float (&scale)[NRB], (&off)[NRB];
    const int (&pos)[NRB];          // window position of the lane's row (-1: padded row)
    int lane, wave, key0;
    __device__ __forceinline__ void operator()(TC<T, D> &acc, int kb, int rb) const {
        uint32_t *h = hist + wave * 32 + (rb / 2) * M::BM + lane % M::BM - TS_LOW * WORDS;
        const uint32_t one = rb % 2 ? 0x10000u : 1u;
#pragma unroll
        for (int v = 0; v < M::NV; ++v) {
            int t = ts_bin(acc[v], scale[rb], off[rb]);
            if (MASK) t = key0 + kb * M::BM + M::crow(v, lane) <= pos[rb] ? t : TS_LOW;
            __hip_atomic_fetch_add(h + t * WORDS, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
};

template <typename T, int D, int NW, bool AGAIN>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void ts_hist_kernel(
    int B, int L, int Hq, int Hkv, int W, const int32_t *__restrict__ cu_seqlens, int64_t T_,
    const T *__restrict__ q_win, const T *__restrict__ k, int64_t k_layer_rows, int nchunk, int chunk_keys,
    TsWork ws) {
    using M = MT<T, D>;
    constexpr int TKEYS = TS_TILE_KEYS;
    using KT = KTile<T, D, TKEYS>;
    constexpr int NRB = QFrags<T, D>::NRB, WORDS = 32 * NW;
    __shared__ __attribute__((aligned(16))) char kbA[KT::BYTES];
    __shared__ __attribute__((aligned(16))) char kbB[KT::BYTES];
    __shared__ __attribute__((aligned(16))) uint32_t hist[(TS_BINS + 2) * WORDS];
    int64_t u;
    int chunk;
    unit_chunk((int64_t)L * Hkv * B, nchunk, u, chunk);
    if (AGAIN && ws.again[u] == 0u) return;
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int G = Hq / Hkv, R = G * W;
    const int N = (int)g.N;
    const int key_begin = chunk * chunk_keys;
    if (N < W || key_begin >= N) return;
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const T *qunit = q_win + (((int64_t)g.b * L + g.l) * Hq + (int64_t)g.h * G) * W * D;
    const T *kunit = k + ((int64_t)g.l * k_layer_rows + (int64_t)g.h * T_ + g.s0) * D;
    const int key_end = min(N, key_begin + chunk_keys);
    const int ntile = (int)ceil_div(key_end - key_begin, KT::TK);
    KT::template load<NW>(kbA, kunit, key_begin, N, wave, lane);
    QFrags<T, D> q;
    q.load(qunit, R, wave, lane);
    for (int i = threadIdx.x; i < (TS_BINS + 2) * WORDS / 4; i += 64 * NW)
        reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
    float scale[NRB], off[NRB];
    int pos[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        const int row = wave * 64 + rb * M::BM + lane % M::BM;
        pos[rb] = row < R ? N - W + row % W : -1;
        const bool on = row < R && (!AGAIN || ws.need[u * R + row] == TS_AGAIN);
        scale[rb] = on ? ws.xa[u * R + row] : 0.f;         // 0, 0: every logit below the interval
        off[rb] = on ? ws.xb[u * R + row] : 0.f;
    }
    TC<T, D> zero[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) zero[rb] = M::zero();
    auto step = [&](int t, char *cur, char *nxt, auto mask) {
        constexpr bool MASK = decltype(mask)::value;
        barrier_after_loads();      // tile t landed (and the bins are clear); tile t - 1 done everywhere
        const int key0 = key_begin + t * KT::TK;
        if (t + 1 < ntile) KT::template load<NW>(nxt, kunit, key0 + KT::TK, N, wave, lane);
        const HistStep<T, D, NW, MASK> f{hist, scale, off, pos, lane, wave, key0};
        if (MASK) tile_sweep_plain<T, D, true, TKEYS>(cur, q, zero, lane, f);
        else tile_sweep<T, D, true, TKEYS>(cur, q, zero, lane, f);
    };
    const int nfull = full_tiles(key_begin, ntile, KT::TK, N, W);
    int t = 0;
    for (; t + 1 < nfull; t += 2) {
        step(t, kbA, kbB, std::false_type{});
        step(t + 1, kbB, kbA, std::false_type{});
    }
    for (; t < ntile; ++t) {
        if (t & 1) step(t, kbB, kbA, std::true_type{});
        else step(t, kbA, kbB, std::true_type{});
    }
    barrier_after_loads();      // every bin final, no load in flight
    // the interval's bins and the keys above it; those below are not needed
    for (int i = threadIdx.x; i < (TS_BINS + 1) * WORDS; i += 64 * NW) {
        const uint32_t both = hist[i + WORDS];
        const int d = i / WORDS, x = i % WORDS;            // word x: wavefront x / 32
        const int row0 = x / 32 * 64 + x % 32 / M::BM * 2 * M::BM + x % M::BM;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int row = row0 + half * M::BM;
            const uint32_t v = half ? both >> 16 : both & 0xffffu;
            uint32_t *dst = d < TS_BINS ? ws.hist + (u * TS_BINS + d) * R + row : ws.above + u * R + row;
            if (row < R && v != 0u) __hip_atomic_fetch_add(dst, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

constexpr int TS_DIGIT_THREADS = 64;

// The order keys of the smallest float (in bit-pattern order) that falls into
// bin `d` of the interval or above it, and into bin d + 1 or above.
__device__ __forceinline__ void ts_bounds(int d, float scale, float off, uint32_t &k0, uint32_t &k1) {
    constexpr uint32_t FIRST = 0x007fffffu, LAST = 0xff800000u;    // order keys of -inf and +inf; +inf is above
    uint32_t lo0 = FIRST, hi0 = LAST, lo1 = FIRST, hi1 = LAST;
    while (lo0 < hi0 || lo1 < hi1) {
        const uint32_t m0 = lo0 + (hi0 - lo0) / 2u, m1 = lo1 + (hi1 - lo1) / 2u;
        const bool at0 = ts_bin(key_value(m0), scale, off) >= d, at1 = ts_bin(key_value(m1), scale, off) > d;
        hi0 = at0 ? m0 : hi0;
        lo0 = at0 ? lo0 : min(m0 + 1u, hi0);
        hi1 = at1 ? m1 : hi1;
        lo1 = at1 ? lo1 : min(m1 + 1u, hi1);
    }
    k0 = lo0;
    k1 = lo1;
}

// One thread per row, one workgroup per unit: the bin of the row's k-th
// largest logit.  The bins of a row are R words apart, so a wavefront's 64 rows
// read each bin as one contiguous run; 32 bins are read before any is used.
template <bool AGAIN>
__global__ __launch_bounds__(TS_DIGIT_THREADS) void ts_digit_kernel(int R, int W, int B, int Hkv,
                                                                     const int32_t *__restrict__ cu_seqlens,
                                                                     int64_t T_, int ratio_bp, TsWork ws) {
    const int64_t u = blockIdx.x;
    if (AGAIN && ws.again[u] == 0u) return;
    const int r = (int)blockIdx.y * TS_DIGIT_THREADS + (int)threadIdx.x;
    if (r >= R) return;
    const int64_t i = u * R + r;
    if (AGAIN && ws.need[i] != TS_AGAIN) return;
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int64_t n = g.N - W + r % W + 1;                 // keys the row sees
    uint32_t need = 0u;
    float xa = INFINITY, xb = INFINITY, thr = INFINITY;    // nothing to gather
    const int64_t kk = ts_rank(n, ratio_bp);
    if (g.N >= W && kk == n) {
        thr = -INFINITY;                                   // every key the row sees
    } else if (g.N >= W) {
        uint32_t *h = ws.hist + u * TS_BINS * (int64_t)R + r;
        const float scale = ws.xa[i], off = ws.xb[i];
        int64_t above = ws.above[i], rest = 0;
        int bin = -1;
        uint32_t in_bin = 0u;
        const bool inside = above < kk;
        const int64_t above_in = above;
        for (int b0 = TS_BINS - 1; b0 >= 0; b0 -= 32) {
            uint32_t c[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) c[j] = h[(int64_t)(b0 - j) * R];
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                if (inside && bin < 0 && above + c[j] >= kk) {
                    bin = b0 - j;
                    rest = kk - above;
                    in_bin = c[j];
                }
                above += c[j];
            }
        }
        const int64_t below = n - above;       // keys below the interval
        if (bin < 0 && scale > 0.f && !inside && above_in <= TS_CMAX) {
            // few keys above the interval, the wanted one among them: a bin
            bin = TS_BINS;
            rest = kk;
            in_bin = (uint32_t)above_in;
        }
        bool found = bin >= 0;
        if (!found && scale > 0.f && inside && below <= TS_CMAX) {      // or below it (bin -1)
            found = true;
            rest = kk - above;
            in_bin = (uint32_t)below;
        }
        if (found) {                           // (both searches at once: their steps overlap)
            uint32_t k0, k1;
            ts_bounds(TS_LOW + 1 + bin, scale, off, k0, k1);
            xa = key_value(k0);
            xb = bin < TS_BINS ? key_value(k1 - 1u) : INFINITY;
        }
        if (found && bin < TS_BINS && xa == xb) {          // one value: nothing to gather
            thr = xb;
            xa = xb = INFINITY;
        } else if (found && in_bin <= (uint32_t)TS_CMAX) {
            need = (uint32_t)rest | in_bin << 16;
        } else {
            // another interval: the bin, or (the sample misjudged the row) the
            // stretch above or below the last one, far where few keys lie
            const float a = (1.f - off) / scale, w = 1.f / scale;
            const float up = above_in <= 4 * TS_CMAX ? 16.f * w : w;
            const float down = below <= 4 * TS_CMAX ? 16.f * w : w;
            // (the margins cover the rounding of the offset: a tied value at the
            // first interval's end had fallen outside of both)
            const float wide = fmaxf(xb - xa, 0x1p-18f * fmaxf(fabsf(xa), fabsf(xb)));
            const float na = found ? xa - 0.02f * wide : inside ? a - down : a + 0.98f * w;
            const float nb = found ? xb + 0.02f * wide : inside ? a + 0.02f * w : a + w + up;
            const float ns = 1.f / (nb - na), no = 1.f - na * ns;
            if (!AGAIN && nb > na && ns > 0.f && ns < INFINITY && fabsf(no) < INFINITY) {
                need = TS_AGAIN;
                xa = ns;
                xb = no;
                ws.above[i] = 0u;
                for (int d = 0; d < TS_BINS; ++d) h[(int64_t)d * R] = 0u;
                atomicMax(ws.again + u, 1u);
            } else if (found) {
                need = TS_TIED;
                atomicMax(ws.again + u, TS_TIED_UNIT);
                thr = __uint_as_float(0xffffffffu);
                ws.gcount[i] = 0u;
            } else {
                need = TS_RADIX;
                xa = xb = __builtin_nanf("");
                atomicOr(ws.fail + u, 1u << (r / 32));
            }
        }
    }
    ws.need[i] = need;
    ws.xa[i] = xa;
    ws.xb[i] = xb;
    ws.thr[i] = thr;
}

// ---------------------------------------------------------------- gather

// The entries of a row's list in LDS, shared evenly by its lanes: 40 where that
// takes no workgroup off a CU (256 rows of 256 bytes a key), else 32.  A list
// that runs over takes its workgroup's chunk once more: with 32 entries random
// logits of 256 units did so now and then, 290 us for the pass instead of 200.
// (At 64 and 128 rows, three workgroups per CU instead of four: 154 -> 168 us.)
template <typename T, int D, int NW>
constexpr int ts_list() { return D * (int)sizeof(T) == 256 && NW == 4 ? 40 : 32; }

// One block of the gather pass: the values of a row that lie in [xa, xb] are
// appended to the lane's list in LDS (a row's values sit in the lanes of equal
// lane % BM; each keeps its own).  Vector instructions only: the median of
// (value, xa, xb) equals the value inside the interval; the lane keeps its
// last match and a bit per value, and appends the match after the block.  A
// lane with several matches in one block (one block in twenty has one) takes
// them one by one.  (Masks per value, joined and tested in scalar registers,
// took 254 us for the pass at 8K keys; a list entry turns up in nearly every
// block.)
// CARE: for units with rows that want only the smallest and largest value of
// their bin (kept in the first two words of the lane's list) and for chunks in
// which a list ran over: a list that would run over first moves to the workspace.
template <typename T, int D, int NW, bool MASK, bool CARE = false>
struct GatherStep {
    using M = MT<T, D>;
    static constexpr int NRB = QFrags<T, D>::NRB, CAP = ts_list<T, D, NW>() * M::BM / 64;   // entries per lane and row block
    uint32_t *mylist;               // LDS, this lane's: [NRB][CAP], words 64 apart
    uint32_t (&cnt)[NRB];           // values gathered so far
    const float (&xa)[NRB], (&xb)[NRB];
    const int (&pos)[NRB];
    int lane, wave, key0, R;
    uint32_t *gcount, *glist, *gmin;        // the unit's counts, lists and tied rows' smallest keys in the workspace
    // a lane's values go after those the row already has (their order does not
    // matter: the pick below ranks them)
    __device__ __forceinline__ void flush(int rb) const {
        int ln = lane;
        asm volatile("" : "+v"(ln));    // addresses made here, not held in registers across the caller's loop
        const uint32_t row = wave * 64 + rb * M::BM + ln % M::BM, n = min(cnt[rb], (uint32_t)CAP);
        if (row >= (uint32_t)R || n == 0u) return;
        if (cnt[rb] >= TS_TIED_LANE) {
            atomicMin(gmin + row, mylist[rb * CAP * 64]);
            atomicMax(gcount + row, mylist[(rb * CAP + 1) * 64]);
            return;
        }
        cnt[rb] = 0u;
        const uint32_t base = __hip_atomic_fetch_add(gcount + row, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (uint32_t j = 0; j < n && base + j < (uint32_t)TS_CMAX; ++j)
            glist[row * TS_CMAX + base + j] = mylist[(rb * CAP + j) * 64];
    }
    __device__ __forceinline__ void operator()(TC<T, D> &acc, int kb, int rb) const {
        uint32_t hits = 0u;
        float last = 0.f;
#pragma unroll
        for (int v = 0; v < M::NV; ++v) {
            bool h = __builtin_amdgcn_fmed3f(acc[v], xa[rb], xb[rb]) == acc[v];
            if (MASK) h = h && key0 + kb * M::BM + M::crow(v, lane) <= pos[rb];
            last = h ? acc[v] : last;
            hits = hits + hits + (h ? 1u : 0u);
        }
        if (CARE && __any(hits != 0u && cnt[rb] >= TS_TIED_LANE)) {
            float lo = INFINITY, hi = -INFINITY;
#pragma unroll
            for (int v = 0; v < M::NV; ++v) {
                const bool h = (hits >> (M::NV - 1 - v)) & 1u;
                lo = fminf(lo, h ? acc[v] : lo);
                hi = fmaxf(hi, h ? acc[v] : hi);
            }
            if (hits != 0u && cnt[rb] >= TS_TIED_LANE) {
                uint32_t *l = mylist + rb * CAP * 64;
                l[0] = min(l[0], order_key(lo));
                l[64] = max(l[64], order_key(hi));
                hits = 0u;
            }
        }
        static_assert(M::NV <= CAP, "an empty list holds a block's values");
        if (CARE && __any(cnt[rb] < TS_TIED_LANE && cnt[rb] + (uint32_t)__popc(hits) > (uint32_t)CAP)) flush(rb);
        auto add = [&](float x) {
            if (cnt[rb] < (uint32_t)CAP) mylist[(rb * CAP + cnt[rb]) * 64] = __float_as_uint(x);
            ++cnt[rb];
        };
        if (__any((hits & (hits - 1u)) != 0u)) {
#pragma unroll
            for (int v = 0; v < M::NV; ++v)
                if ((hits >> (M::NV - 1 - v)) & 1u) add(acc[v]);
        } else if (hits != 0u) {
            add(last);
        }
    }
};

template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(sizeof(T) * D * 8 / NW <= 128 ? 4 : 2))) void ts_gather_kernel(
    int B, int L, int Hq, int Hkv, int W, const int32_t *__restrict__ cu_seqlens, int64_t T_,
    const T *__restrict__ q_win, const T *__restrict__ k, int64_t k_layer_rows, int nchunk, int chunk_keys,
    TsWork ws) {
    using M = MT<T, D>;
    constexpr int TKEYS = TS_TILE_KEYS;
    using KT = KTile<T, D, TKEYS>;
    constexpr int NRB = QFrags<T, D>::NRB;
    __shared__ __attribute__((aligned(16))) char kbA[KT::BYTES];
    __shared__ __attribute__((aligned(16))) char kbB[KT::BYTES];
    constexpr int CAP = GatherStep<T, D, NW, false>::CAP;
    __shared__ uint32_t lists[NW * NRB * CAP * 64];
    int64_t u;
    int chunk;
    unit_chunk((int64_t)L * Hkv * B, nchunk, u, chunk);
    const bool tied = ws.again[u] == TS_TIED_UNIT;     // uniform
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int G = Hq / Hkv, R = G * W;
    const int N = (int)g.N;
    const int key_begin = chunk * chunk_keys;
    if (N < W || key_begin >= N) return;
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const T *qunit = q_win + (((int64_t)g.b * L + g.l) * Hq + (int64_t)g.h * G) * W * D;
    const T *kunit = k + ((int64_t)g.l * k_layer_rows + (int64_t)g.h * T_ + g.s0) * D;
    const int key_end = min(N, key_begin + chunk_keys);
    const int ntile = (int)ceil_div(key_end - key_begin, KT::TK);
    KT::template load<NW>(kbA, kunit, key_begin, N, wave, lane);
    QFrags<T, D> q;
    q.load(qunit, R, wave, lane);
    uint32_t cnt[NRB];
    float xa[NRB], xb[NRB];
    int pos[NRB];
    uint32_t *mylist = lists + wave * (NRB * CAP * 64) + lane;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        const int row = wave * 64 + rb * M::BM + lane % M::BM;
        pos[rb] = row < R ? N - W + row % W : -1;
        const uint32_t need = row < R ? ws.need[u * R + row] : TS_RADIX;
        xa[rb] = need != TS_RADIX ? ws.xa[u * R + row] : INFINITY;
        xb[rb] = need != TS_RADIX ? ws.xb[u * R + row] : INFINITY;
        cnt[rb] = need == TS_TIED ? TS_TIED_LANE : 0u;
        if (need == TS_TIED) {
            mylist[rb * CAP * 64] = 0xffffffffu;
            mylist[(rb * CAP + 1) * 64] = 0u;
        }
    }
    TC<T, D> zero[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) zero[rb] = M::zero();
    uint32_t *gcount = ws.gcount + u * R, *glist = ws.list + u * R * TS_CMAX;
    uint32_t *gmin = reinterpret_cast<uint32_t *>(ws.thr) + u * R;
    auto step = [&](int t, char *cur, char *nxt, auto mask, auto care) {
        constexpr bool MASK = decltype(mask)::value, CARE = decltype(care)::value;
        barrier_after_loads();      // tile t landed; tile t - 1 done everywhere
        const int key0 = key_begin + t * KT::TK;
        if (t + 1 < ntile) KT::template load<NW>(nxt, kunit, key0 + KT::TK, N, wave, lane);
        const GatherStep<T, D, NW, MASK, CARE> f{mylist, cnt, xa, xb, pos, lane, wave, key0, R, gcount, glist, gmin};
        if (MASK) tile_sweep_plain<T, D, true, TKEYS>(cur, q, zero, lane, f);
        else tile_sweep<T, D, true, TKEYS>(cur, q, zero, lane, f);
    };
    bool care = tied;
    if (!care) {
        const int nfull = full_tiles(key_begin, ntile, KT::TK, N, W);
        int t = 0;
        for (; t + 1 < nfull; t += 2) {
            step(t, kbA, kbB, std::false_type{}, std::false_type{});
            step(t + 1, kbB, kbA, std::false_type{}, std::false_type{});
        }
        for (; t < ntile; ++t) {
            if (t & 1) step(t, kbB, kbA, std::true_type{}, std::false_type{});
            else step(t, kbA, kbB, std::true_type{}, std::false_type{});
        }
        barrier_after_loads();      // the tiles are done with, no load in flight
        // a list that ran over anywhere in the workgroup (logits that follow the
        // position put most of a row's bin into one chunk): the chunk again, with
        // care.  32 layers of 8K keys, rising logits: 0.94 ms; 1.36 with the radix
        // select for such rows; 0.68 with full lists moved between tiles, which
        // took every call 8 to 10 of the pass's 190 us.
        bool over = false;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) over |= cnt[rb] > (uint32_t)CAP;
        int *flags = reinterpret_cast<int *>(kbA);
        if (lane == 0) flags[wave] = 0;
        if (over) flags[wave] = 1;
        __syncthreads();
        int any = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) any |= flags[w];
        care = __builtin_amdgcn_readfirstlane(any) != 0;
        if (care) {                 // uniform across the workgroup
            __syncthreads();        // every flag read
            KT::template load<NW>(kbA, kunit, key_begin, N, wave, lane);
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) cnt[rb] = 0u;
        }
    }
    if (care) {
        for (int t = 0; t < ntile; ++t) {
            if (t & 1) step(t, kbB, kbA, std::true_type{}, std::true_type{});
            else step(t, kbA, kbB, std::true_type{}, std::true_type{});
        }
        barrier_after_loads();      // no load in flight
    }
    const GatherStep<T, D, NW, true, true> rest{mylist, cnt, xa, xb, pos, lane, wave, 0, R, gcount, glist, gmin};
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) rest.flush(rb);
}

// The exact value of rank `need` (from the top) among a row's gathered ones: a
// wavefront takes PICK_ROWS rows, all their loads issued first, a value (or
// two) per lane, and finds every row's key bit by bit below the bits that the
// bin's two ends share: the largest key that at least `rank` values reach.  A
// list that does not hold what the histogram counted in its bin (it never is
// so for numbers) sends the row to the radix select.
constexpr int PICK_ROWS = 8;
__global__ __launch_bounds__(256) void ts_pick_kernel(int64_t nrows, int R, int64_t group0, TsWork ws) {
    const int lane = threadIdx.x % 64;
    const int64_t wave = (group0 + blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t i0 = wave * PICK_ROWS;
    if (i0 >= nrows) return;
    const int64_t mine = min(i0 + lane % PICK_ROWS, nrows - 1);
    uint32_t need = i0 + lane % PICK_ROWS < nrows ? ws.need[mine] : 0u;
    const uint32_t got = ws.gcount[mine];
    const uint32_t ka = order_key(ws.xa[mine]), kb = order_key(ws.xb[mine]);
    uint32_t v0[PICK_ROWS], v1[PICK_ROWS];
#pragma unroll
    for (int j = 0; j < PICK_ROWS; ++j) {
        const uint32_t *l = ws.list + min(i0 + j, nrows - 1) * TS_CMAX;
        v0[j] = l[lane];
        v1[j] = l[min(64 + lane, TS_CMAX - 1)];
    }
    // lane j: row i0 + j
    if (need == TS_RADIX) need = 0u;
    if (need == TS_TIED) {             // one value (-0 and +0 are equal) is the threshold
        const uint32_t lo = reinterpret_cast<const uint32_t *>(ws.thr)[mine];
        const float x = key_value(lo), y = key_value(got);
        if (lane < PICK_ROWS) {
            ws.thr[mine] = y;
            ws.xa[mine] = x == 0.f ? -0.f : x;         // else: the radix select between them
            ws.xb[mine] = y == 0.f ? 0.f : y;
        }
        if (x == y) need = 0u;
    }
    if (need != 0u && got != need >> 16) {
        const int64_t u = mine / R;
        if (lane < PICK_ROWS) {
            ws.need[mine] = TS_RADIX;
            atomicOr(ws.fail + u, 1u << ((int)(mine % R) / 32));
        }
        need = 0u;
    }
    if (!__any(need != 0u)) return;
    int rank[PICK_ROWS];
    uint32_t cur[PICK_ROWS];
    const int top = wave_max_bits(need != 0u ? ka ^ kb : 0u);      // bits to decide, of every row
    bool two = false;                                   // some row has more than 64 values
#pragma unroll
    for (int j = 0; j < PICK_ROWS; ++j) {
        const uint32_t nd = (uint32_t)__builtin_amdgcn_readlane((int)need, j);
        const int n = (int)(nd >> 16);
        rank[j] = (int)(nd & 0xffffu);
        cur[j] = (uint32_t)__builtin_amdgcn_readlane((int)kb, j) & (top >= 32 ? 0u : ~0u << top);
        v0[j] = lane < n ? order_key(__uint_as_float(v0[j])) : 0u;
        v1[j] = 64 + lane < n ? order_key(__uint_as_float(v1[j])) : 0u;
        two |= n > 64;
    }
    for (int bit = top - 1; bit >= 0; --bit) {
#pragma unroll
        for (int j = 0; j < PICK_ROWS; ++j) {
            const uint32_t t = cur[j] | 1u << bit;
            int c = (int)__popcll(__ballot(v0[j] >= t));
            if (two) c += (int)__popcll(__ballot(v1[j] >= t));
            cur[j] = c >= rank[j] ? t : cur[j];
        }
    }
    float thr = 0.f;
#pragma unroll
    for (int j = 0; j < PICK_ROWS; ++j) thr = lane == j ? threshold_value(cur[j]) : thr;
    if (lane < PICK_ROWS && need != 0u) ws.thr[mine] = thr;
}

// ---------------------------------------------------------------- radix

// The exact thresholds of the rows that the passes above did not resolve, 32
// rows of a unit per workgroup: 6-bit digits of the logits' order keys, most
// significant first, below the bits that the ends of every such row's bin
// share (a bin of ties is narrow by now: two or three digits), over all the
// keys.
constexpr int TS_RADIX_WAVES = 8, TS_RADIX_COPIES = 2;
template <typename T, int D>
__global__ __launch_bounds__(64 * TS_RADIX_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void ts_radix_kernel(
    int B, int L, int Hq, int Hkv, int W, const int32_t *__restrict__ cu_seqlens, int64_t T_,
    const T *__restrict__ q_win, const T *__restrict__ k, int64_t k_layer_rows, int ratio_bp, int64_t u0, TsWork ws) {
    using M = MT<T, D>;
    constexpr int NB32 = 32 / M::BM;                   // row blocks
    using KT = KTile<T, D, M::BM>;                     // one key block
    __shared__ __attribute__((aligned(16))) char bufs[TS_RADIX_WAVES * 2 * KT::BYTES];
    // two copies (with ties, wavefronts queue for one word); the last bin takes
    // the keys that do not match the prefix
    __shared__ uint32_t hist[TS_RADIX_COPIES][TS_BINS + 1][32];
    __shared__ int over[32];                           // keys above the row's bin
    __shared__ uint32_t prefix[32];
    __shared__ int64_t rank[32];
    __shared__ int bits;
    const int R = (Hq / Hkv) * W, ngrp = (int)ceil_div(R, 32);
    const int64_t u = u0 + blockIdx.x / ngrp;
    const int grp = blockIdx.x % ngrp;
    if (((ws.fail[u] >> grp) & 1u) == 0u) return;
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int N = (int)g.N, tid = threadIdx.x, lane = tid % 64;
    if (N < W) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const T *qunit = q_win + (((int64_t)g.b * L + g.l) * Hq + (int64_t)g.h * (Hq / Hkv)) * W * D;
    const T *kunit = k + ((int64_t)g.l * k_layer_rows + (int64_t)g.h * T_ + g.s0) * D;
    TA<T, D> qf[NB32][M::KS];
    int pos[NB32];
#pragma unroll
    for (int rb = 0; rb < NB32; ++rb) {
        const int row = grp * 32 + rb * M::BM + lane % M::BM;
        pos[rb] = row < R ? N - W + row % W : -1;
        const T *p = qunit + (int64_t)min(row, R - 1) * D;
#pragma unroll
        for (int ks = 0; ks < M::KS; ++ks) qf[rb][ks] = M::load_global(p, ks, lane);
    }
    const int64_t myrow = u * R + grp * 32 + tid;
    const bool mine = tid < 32 && grp * 32 + tid < R && ws.need[myrow] == TS_RADIX;
    if (tid < 64) {
        uint32_t ka = 0u, diff = 0u;
        if (mine) {
            const float xa = ws.xa[myrow], xb = ws.xb[myrow];
            ka = order_key(xa);
            diff = xa <= xb ? ka ^ order_key(xb) : ~0u;        // NaN: nothing known
        }
        const int nbits = wave_max_bits(diff);
        if (tid < 32) {
            prefix[tid] = nbits < 32 ? ka >> nbits << nbits : 0u;
            over[tid] = 0;
            rank[tid] = ts_rank(N - W + (grp * 32 + tid) % W + 1, ratio_bp);
        }
        if (tid == 0) bits = nbits;
    }
    __syncthreads();
    const int hi0 = __builtin_amdgcn_readfirstlane(bits);
    char *mybuf = bufs + wave * (2 * KT::BYTES);
    for (int hi = hi0; hi > 0;) {
        const int sh = max(0, hi - 6);
        for (int i = tid; i < TS_RADIX_COPIES * (TS_BINS + 1) * 32; i += 64 * TS_RADIX_WAVES) (&hist[0][0][0])[i] = 0u;
        __syncthreads();
        // no branch per value: one whose key does not match the row's prefix
        // adds to the last bin.  For a prefix that holds the sign bit, the
        // value's bits ^ flip = its key ^ prefix.
        const uint32_t lim = 1u << (hi - sh);
        uint32_t flip[NB32], end[NB32];
        int above[NB32];
#pragma unroll
        for (int rb = 0; rb < NB32; ++rb) {
            const uint32_t p = prefix[rb * M::BM + lane % M::BM];
            flip[rb] = p ^ ((p & 0x80000000u) ? 0x80000000u : 0xffffffffu);
            end[rb] = hi < 32 ? p | ((1u << hi) - 1u) : ~0u;
            above[rb] = 0;
        }
        // every wavefront streams its own key blocks through two LDS buffers,
        // the next one's loads in flight (straight from memory each lane would
        // read pieces of its own key's row, and the rows of several wavefronts
        // do not fit the L1)
        if (wave * M::BM < N) KT::template load<1>(mybuf, kunit, wave * M::BM, N, 0, lane);
        for (int key0 = wave * M::BM, t = 0; key0 < N; key0 += TS_RADIX_WAVES * M::BM, ++t) {      // uniform per wavefront
            const char *cur = mybuf + (t & 1) * KT::BYTES;
            KT::template load<1>(mybuf + (~t & 1) * KT::BYTES, kunit, min(key0 + TS_RADIX_WAVES * M::BM, N - 1), N, 0, lane);
            wait_vmem<KT::BYTES / 1024>();
            {
                TA<T, D> kf[M::KS];
#pragma unroll
                for (int ks = 0; ks < M::KS; ++ks) kf[ks] = KT::frag(cur, 0, ks, lane);
#pragma unroll
                for (int rb = 0; rb < NB32; ++rb) {
                    const TC<T, D> acc = block_mma<T, D, true>(kf, qf[rb]);
#pragma unroll
                    for (int v = 0; v < M::NV; ++v) {
                        const bool sees = key0 + M::crow(v, lane) <= pos[rb];
                        const uint32_t y = hi == 32 ? order_key(acc[v]) : __float_as_uint(acc[v]) ^ flip[rb];
                        const uint32_t d = sees ? min(y >> sh, lim) : lim;
                        if (hi == hi0) above[rb] += sees && order_key(acc[v]) > end[rb] ? 1 : 0;
                        __hip_atomic_fetch_add(&hist[wave % TS_RADIX_COPIES][d][rb * M::BM + lane % M::BM], 1u, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
        }
        wait_vmem<0>();
        if (hi == hi0)
#pragma unroll
            for (int rb = 0; rb < NB32; ++rb) atomicAdd(&over[rb * M::BM + lane % M::BM], above[rb]);
        __syncthreads();
        if (tid < 32) {
            int64_t above = hi == hi0 ? over[tid] : 0;
            const int64_t want = rank[tid];
            for (int d = (1 << (hi - sh)) - 1; d >= 0; --d) {
                int64_t c = 0;
#pragma unroll
                for (int w = 0; w < TS_RADIX_COPIES; ++w) c += hist[w][d][tid];
                if (above < want && want <= above + c) {
                    prefix[tid] |= (uint32_t)d << sh;
                    rank[tid] = want - above;
                }
                above += c;
            }
        }
        __syncthreads();
        hi = sh;
    }
    if (mine) ws.thr[myrow] = threshold_value(prefix[tid]);
}

// ---------------------------------------------------------------- count

// Keys per LDS tile of the count pass.
template <typename T>
constexpr int ts_count_tile_keys() { return sizeof(T) == 2 ? 128 : 64; }

// One block of the count pass, C = Q K^T: a lane's values belong to one key,
// and a key's picks are added up in the lane.
template <typename T, int D, bool MASK>
struct TsCountStep {
    static constexpr int NRB = QFrags<T, D>::NRB;
    int (&cs)[KTile<T, D, ts_count_tile_keys<T>()>::NKB];
    const TC<T, D> (&thr)[NRB];            // the thresholds of the lane's rows (+inf: padded row)
    const int *poss;                       // window position of every row of the unit (-1: padded), LDS
    int lane, wave, key0;
    __device__ __forceinline__ void operator()(TC<T, D> &acc, int kb, int rb) const {
        using M = MT<T, D>;
        const int key = key0 + kb * M::BM + lane % M::BM;
        int n[2] = {0, 0};
#pragma unroll
        for (int g4 = 0; g4 < M::NV / 4; ++g4) {
            int4 pos = make_int4(0, 0, 0, 0);
            if (MASK) pos = *reinterpret_cast<const int4 *>(poss + wave * 64 + rb * M::BM + M::crow(4 * g4, lane));
            const int ps[4] = {pos.x, pos.y, pos.z, pos.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bool pick = acc[4 * g4 + i] >= thr[rb][4 * g4 + i];
                if (MASK) pick = pick && key <= ps[i];
                n[i % 2] += pick ? 1 : 0;
            }
        }
        cs[kb] += n[0] + n[1];
    }
};

template <typename T, int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void ts_count_kernel(
    int B, int L, int Hq, int Hkv, int W, const int32_t *__restrict__ cu_seqlens, int64_t T_,
    const T *__restrict__ q_win, const T *__restrict__ k, int64_t k_layer_rows, int nchunk, int chunk_keys,
    const float *__restrict__ thr_rows, float *__restrict__ counts) {
    using M = MT<T, D>;
    constexpr int TKEYS = ts_count_tile_keys<T>();
    using KT = KTile<T, D, TKEYS>;
    constexpr int NRB = QFrags<T, D>::NRB, NKB = KT::NKB;
    __shared__ __attribute__((aligned(16))) char kbA[KT::BYTES];
    __shared__ __attribute__((aligned(16))) char kbB[KT::BYTES];
    __shared__ int csum[2][NW][KT::TK];
    __shared__ __attribute__((aligned(16))) float thr_s[NW * 64];
    __shared__ __attribute__((aligned(16))) int poss[NW * 64];
    int64_t u;
    int chunk;
    unit_chunk((int64_t)L * Hkv * B, nchunk, u, chunk);
    const UnitGeom g = unit_geom(u, B, Hkv, cu_seqlens, T_);
    const int G = Hq / Hkv, R = G * W;
    const int N = (int)g.N;
    const int key_begin = chunk * chunk_keys;
    const int key_end = min(N, key_begin + chunk_keys);
    float *orow = counts + ((int64_t)g.l * Hkv + g.h) * T_ + g.s0;
    if (N < W) {  // documented fallback: zero counts
        for (int j = key_begin + (int)threadIdx.x; j < key_end; j += blockDim.x) orow[j] = 0.f;
        return;
    }
    if (key_begin >= N) return;
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const T *qunit = q_win + (((int64_t)g.b * L + g.l) * Hq + (int64_t)g.h * G) * W * D;
    const T *kunit = k + ((int64_t)g.l * k_layer_rows + (int64_t)g.h * T_ + g.s0) * D;
    const int ntile = (int)ceil_div(key_end - key_begin, KT::TK);
    KT::template load<NW>(kbA, kunit, key_begin, N, wave, lane);
    QFrags<T, D> q;
    q.load(qunit, R, wave, lane);
    for (int r = threadIdx.x; r < NW * 64; r += 64 * NW) {
        thr_s[r] = r < R ? thr_rows[u * R + r] : INFINITY;
        poss[r] = r < R ? N - W + r % W : -1;
    }
    __syncthreads();
    TC<T, D> zero[NRB], thr[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        zero[rb] = M::zero();
#pragma unroll
        for (int v = 0; v < M::NV; ++v) thr[rb][v] = thr_s[wave * 64 + rb * M::BM + M::crow(v, lane)];
    }
    // the wavefronts' picks of tile t sit in csum[t & 1]; they are added and
    // stored after the next barrier
    auto flush = [&](int t) {
        const int key0 = key_begin + t * KT::TK;
        for (int j = threadIdx.x; j < KT::TK; j += 64 * NW) {
            int v = 0;
            for (int w = 0; w < NW; ++w) v += csum[t & 1][w][j];
            if (key0 + j < N) orow[key0 + j] = (float)v;
        }
    };
    auto step = [&](int t, char *cur, char *nxt, auto mask) {
        constexpr bool MASK = decltype(mask)::value;
        barrier_after_loads();      // tile t landed; tile t - 1 finished everywhere
        if (t > 0) flush(t - 1);
        const int key0 = key_begin + t * KT::TK;
        if (t + 1 < ntile) KT::template load<NW>(nxt, kunit, key0 + KT::TK, N, wave, lane);
        int cs[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) cs[kb] = 0;
        const TsCountStep<T, D, MASK> f{cs, thr, poss, lane, wave, key0};
        if (MASK) tile_sweep_plain<T, D, false, TKEYS>(cur, q, zero, lane, f);
        else tile_sweep<T, D, false, TKEYS>(cur, q, zero, lane, f);
        // lanes holding the same key (different rows) add up; every such lane
        // then holds the total and stores it
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int off = M::BM; off < 64; off <<= 1) cs[kb] += __shfl_xor(cs[kb], off, 64);
            csum[t & 1][wave][kb * M::BM + lane % M::BM] = cs[kb];
        }
    };
    const int nfull = full_tiles(key_begin, ntile, KT::TK, N, W);
    int t = 0;
    for (; t + 1 < nfull; t += 2) {
        step(t, kbA, kbB, std::false_type{});
        step(t + 1, kbB, kbA, std::false_type{});
    }
    for (; t < ntile; ++t) {
        if (t & 1) step(t, kbB, kbA, std::true_type{});
        else step(t, kbA, kbB, std::true_type{});
    }
    __syncthreads();
    flush(ntile - 1);
}

template <typename T, int D, int NW>
static void launch_topshare(hipStream_t s, const ScorePlan &p, int B, int L, int Hq, int Hkv, int W,
                            const int32_t *cu_seqlens, int64_t ntok, int max_seqlen, const void *q_win,
                            const void *k, int64_t k_layer_rows, int ratio_bp, float *counts, void *wsp) {
    const int R = (Hq / Hkv) * W;
    const int64_t units = (int64_t)L * Hkv * B, nrows = units * R;
    TsWork ws;
    ws.xa = reinterpret_cast<float *>(wsp);
    ws.xb = ws.xa + nrows;
    ws.need = reinterpret_cast<uint32_t *>(ws.xb + nrows);
    ws.above = ws.need + nrows;
    ws.gcount = ws.above + nrows;
    ws.thr = reinterpret_cast<float *>(ws.gcount + nrows);
    ws.hist = reinterpret_cast<uint32_t *>(ws.thr + nrows);
    ws.list = ws.hist;
    ws.fail = ws.hist + nrows * TS_CMAX;
    ws.again = ws.fail + units;
    const T *q = reinterpret_cast<const T *>(q_win);
    const T *kk = reinterpret_cast<const T *>(k);
    const dim3 grid((unsigned)(units * p.nchunk));
    // a larger sample for longer prompts: the interval, and so a bin, then holds
    // about as many keys (8K keys: about 22 of the 92 a row may gather; 32K: 45)
    // (sample, radix and pick have more threads per unit than the others: calls
    // of some million units take more than one launch of them)
#define SG_SAMPLE(NWV, ROWS)                                                                            \
    launch_slices(units, ceil_div(R, ROWS) * 64 * NWV, [&](int64_t u0, int64_t n) {                      \
        ts_sample_kernel<T, D, NWV, ROWS><<<(unsigned)(n * ceil_div(R, ROWS)), 64 * NWV, 0, s>>>(        \
            B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows, ratio_bp, u0, ws);                  \
    })
    // fp32 at d = 128: 64 rows' queries beside as many values spill; 32 rows at a
    // time read the sample twice, which pays up to 256 rows (4 layers of 4K keys,
    // 64 / 256 / 512 rows: 301, 577, 1,161 against 315, 588, 1,141 us)
    bool half = false;
    if constexpr (sizeof(T) * D > 256) {
        half = R <= 256;
        if (half && max_seqlen <= 12288) SG_SAMPLE(2, 32);
        else if (half && max_seqlen <= 24576) SG_SAMPLE(4, 32);
    }
    if (max_seqlen > 24576) SG_SAMPLE(8, 32);              // 2048 keys
    else if (!half && max_seqlen > 12288) SG_SAMPLE(8, 64);    // 1024
    else if (!half) SG_SAMPLE(4, 64);                      // 512
#undef SG_SAMPLE
    const dim3 dgrid((unsigned)units, (unsigned)ceil_div(R, TS_DIGIT_THREADS));
    ts_hist_kernel<T, D, NW, false><<<grid, 64 * NW, 0, s>>>(B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows,
                                                             p.nchunk, p.chunk_keys, ws);
    ts_digit_kernel<false><<<dgrid, TS_DIGIT_THREADS, 0, s>>>(R, W, B, Hkv, cu_seqlens, ntok, ratio_bp, ws);
    ts_hist_kernel<T, D, NW, true><<<grid, 64 * NW, 0, s>>>(B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows,
                                                            p.nchunk, p.chunk_keys, ws);
    ts_digit_kernel<true><<<dgrid, TS_DIGIT_THREADS, 0, s>>>(R, W, B, Hkv, cu_seqlens, ntok, ratio_bp, ws);
    ts_gather_kernel<T, D, NW><<<grid, 64 * NW, 0, s>>>(B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows,
                                                        p.nchunk, p.chunk_keys, ws);
    launch_slices(ceil_div(nrows, 4 * PICK_ROWS), 256, [&](int64_t group0, int64_t n) {
        ts_pick_kernel<<<(unsigned)n, 256, 0, s>>>(nrows, R, group0, ws);
    });
    launch_slices(units, ceil_div(R, 32) * 64 * TS_RADIX_WAVES, [&](int64_t u0, int64_t n) {
        ts_radix_kernel<T, D><<<(unsigned)(n * ceil_div(R, 32)), 64 * TS_RADIX_WAVES, 0, s>>>(
            B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows, ratio_bp, u0, ws);
    });
    ts_count_kernel<T, D, NW><<<grid, 64 * NW, 0, s>>>(B, L, Hq, Hkv, W, cu_seqlens, ntok, q, kk, k_layer_rows,
                                                      p.nchunk, p.chunk_keys, ws.thr, counts);
}

template <typename T, int D>
static int topshare_dispatch(hipStream_t s, int B, int L, int Hq, int Hkv, int W, const int32_t *cu_seqlens,
                             int64_t ntok, int max_seqlen, const void *q_win, const void *k, int64_t k_layer_rows,
                             int ratio_bp, float *counts, void *ws) {
    const int R = (Hq / Hkv) * W;
    const int nw = (int)ceil_div(R, 64);
    const ScorePlan p = score_plan(B, L, Hkv, max_seqlen);
    if (nw <= 1) launch_topshare<T, D, 1>(s, p, B, L, Hq, Hkv, W, cu_seqlens, ntok, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    else if (nw <= 2) launch_topshare<T, D, 2>(s, p, B, L, Hq, Hkv, W, cu_seqlens, ntok, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    else if (nw <= 4) launch_topshare<T, D, 4>(s, p, B, L, Hq, Hkv, W, cu_seqlens, ntok, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    else launch_topshare<T, D, 8>(s, p, B, L, Hq, Hkv, W, cu_seqlens, ntok, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    return launch_status("sg_score_topshare");
}

}  // namespace sg

using namespace sg;

extern "C" size_t sg_score_topshare_workspace_size(int B, int L, int Hq, int Hkv, int d, int W, int max_seqlen) {
    if (B <= 0 || L <= 0 || Hkv <= 0 || Hq <= 0 || W <= 0 || max_seqlen <= 0 || d <= 0) return 0;
    const int64_t units = (int64_t)L * Hkv * B, rows = units * (Hq / Hkv) * W;
    return (size_t)(rows * TS_ROW_WORDS + units * TS_UNIT_WORDS) * sizeof(uint32_t);
}

extern "C" int sg_score_topshare(void *stream, sg_dtype dt, int B, int L, int Hq, int Hkv, int d, int W,
                                 const int32_t *cu_seqlens, int64_t T, int max_seqlen, const void *q_win,
                                 const void *k, int64_t k_layer_rows, int ratio_bp, float *counts, void *ws,
                                 size_t ws_bytes) {
    const char *name = "sg_score_topshare";
    SG_REQUIRE(dt == SG_F32 || dt == SG_BF16, SG_EINVAL, "%s: unknown dtype %d", name, (int)dt);
    SG_REQUIRE(B >= 1 && L >= 1 && Hq >= 1 && Hkv >= 1 && Hq % Hkv == 0, SG_EINVAL,
               "%s: need B, L, Hq, Hkv >= 1 and Hq %% Hkv == 0", name);
    SG_REQUIRE(d == 64 || d == 128, SG_EUNSUPPORTED, "%s: head dimension %d not supported (64 or 128)", name, d);
    SG_REQUIRE(W >= 1, SG_EINVAL, "%s: window must be >= 1", name);
    SG_REQUIRE((int64_t)(Hq / Hkv) * W <= SC_MAXR, SG_EUNSUPPORTED, "%s: G*W = %d above %d", name, (Hq / Hkv) * W,
               SC_MAXR);
    SG_REQUIRE(ratio_bp >= 1 && ratio_bp <= 10000, SG_EINVAL, "%s: ratio_bp %d outside [1, 10000]", name, ratio_bp);
    SG_REQUIRE(T >= 0 && max_seqlen >= 0 && k_layer_rows >= 0, SG_EINVAL, "%s: negative size", name);
    SG_REQUIRE(max_seqlen <= (1 << 30), SG_EINVAL, "%s: max_seqlen too large", name);
    if (T == 0 || max_seqlen == 0) return SG_OK;
    SG_REQUIRE(cu_seqlens && q_win && k && counts, SG_EINVAL, "%s: null pointer", name);
    SG_REQUIRE(aligned16(q_win) && aligned16(k), SG_EINVAL, "%s: q_win and k must be 16-byte aligned", name);
    const int64_t units = (int64_t)L * Hkv * B;
    SG_REQUIRE(units * ceil_div(max_seqlen, 128) <= 0x7fffffff, SG_EINVAL, "%s: grid too large", name);
    SG_REQUIRE(units * (Hq / Hkv) * W <= (int64_t)0x7fffffff, SG_EINVAL, "%s: too many rows", name);
    const size_t need = sg_score_topshare_workspace_size(B, L, Hq, Hkv, d, W, max_seqlen);
    SG_REQUIRE(ws && ws_bytes >= need, SG_EWORKSPACE, "%s: workspace %zu < %zu", name, ws_bytes, need);
    SG_REQUIRE(aligned16(ws), SG_EINVAL, "%s: workspace must be 16-byte aligned", name);
    hipStream_t s = as_stream(stream);
    if (dt == SG_BF16) {
        if (d == 128) return topshare_dispatch<uint16_t, 128>(s, B, L, Hq, Hkv, W, cu_seqlens, T, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
        return topshare_dispatch<uint16_t, 64>(s, B, L, Hq, Hkv, W, cu_seqlens, T, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    }
    if (d == 128) return topshare_dispatch<float, 128>(s, B, L, Hq, Hkv, W, cu_seqlens, T, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
    return topshare_dispatch<float, 64>(s, B, L, Hq, Hkv, W, cu_seqlens, T, max_seqlen, q_win, k, k_layer_rows, ratio_bp, counts, ws);
}
