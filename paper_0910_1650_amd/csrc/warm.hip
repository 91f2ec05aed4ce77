// warm.hip -- learned warm start for Algorithm 1 (Section 2).
//
// Algorithm 1 starts from zero availabilities (Eq. (1)); the paper's only warm
// start is PAP's merge of sub-problem availabilities (Section 3, Algorithm 2,
// steps 3-4).  This file replaces that merge with a prediction made per point
// from its row of S:
//
//   features   16 numbers per point: order statistics of the off-diagonal row
//              (1st..32nd largest, their top-32 mean, five quantiles),
//              s(k,k) against the row median and the top-32 mean, the share
//              of the row above s(k,k), ln(n)/10; similarities are divided
//              by sigma, the magnitude of the median of the row medians.
//   network    16 -> 128 -> 128 -> 2 with GELU; bf16 weights and activations
//              on the matrix cores with FP32 accumulation; FP32 backward with
//              fixed-order reductions; Adam on FP32 master weights.
//   targets    the column quantities of Eqs. (3)-(4) of a converged run,
//              t_k = r(k,k) + c_k and c_k = sum_{i != k} max(0, r(i,k)),
//              divided by sigma.
//   A_0        a(i,k) = min(0, sigma y0_k) off the diagonal and
//              a(k,k) = max(0, sigma y1_k): Eqs. (3)-(4) with the predicted
//              column quantities.  R_0 = one undamped Eq. (2) step from A_0.
//
// Order statistics are exact: the keys of the eleven intervals of a row that
// hold its ranks are collected and ranked by counting (k_row_stats; crowded
// rows by repeated cuts, k_row_stats_crowded); the median of medians goes
// through a most-significant-digit radix select over the order-preserving
// integer image of the FP32 values (8-bit digits, four passes).
#include <cmath>
#include <cstring>
#include <type_traits>

#include "apx_internal.h"

using namespace apx;

namespace {

constexpr int NF = APX_MLP_FEATURES;   // 16
constexpr int NH = 128;
constexpr int NO = 2;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + NF * NH;
constexpr int OFF_W2 = OFF_B1 + NH;
constexpr int OFF_B2 = OFF_W2 + NH * NH;
constexpr int OFF_W3 = OFF_B2 + NH;
constexpr int OFF_B3 = OFF_W3 + NH * NO;
constexpr int NPARAM = OFF_B3 + NO;
static_assert(NPARAM == APX_MLP_PARAMS, "parameter layout");

#define HIP_TRY(expr, what)                                   \
    do {                                                      \
        hipError_t _e = (expr);                               \
        if (_e != hipSuccess) return hip_err(ctx, _e, what);  \
    } while (0)
#define APX_TRY(expr)                       \
    do {                                    \
        apx_status _st = (expr);            \
        if (_st != APX_OK) return _st;      \
    } while (0)

// ---------------------------------------------------------------------------
// Exact multi-rank selection
// ---------------------------------------------------------------------------
constexpr int SEL_T = 1024;
constexpr int NTGT = 11;               // 6 descending ranks + 5 quantiles
constexpr int TOP = 32;

__device__ __forceinline__ uint32_t fkey(float v) {
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float keyf(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

struct SelShared {
    uint32_t hist[NTGT][256];
    uint32_t pref[NTGT];       // key digits found so far
    int32_t rank[NTGT];        // rank still to find among keys with that prefix
    int32_t slot[NTGT];        // histogram each target reads
    uint32_t slot_pref[NTGT];  // prefix counted by each histogram
    int32_t nslots;
};

// On entry sm.rank[t] (t < ntgt) holds the ascending rank wanted; on return
// sm.pref[t] is the key of that order statistic.  Targets whose prefixes
// agree share a histogram; prefixes of one pass have equal length, so each
// element feeds at most one histogram.  get(j) returns the key of element j
// of [0, count).  Called by every thread of the block.
template <class Get>
__device__ void radix_select(SelShared &sm, int64_t count, int ntgt, Get get) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwaves = blockDim.x >> 6;
    if (tid < ntgt) {
        sm.pref[tid] = 0;
        sm.slot[tid] = 0;
    }
    if (tid == 0) {
        sm.nslots = 1;
        sm.slot_pref[0] = 0;
    }
    __syncthreads();
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        const int ns = sm.nslots;
        for (int e = tid; e < ns * 256; e += blockDim.x) (&sm.hist[0][0])[e] = 0u;
        __syncthreads();
        for (int64_t j = tid; j < count; j += blockDim.x) {
            const uint32_t key = get(j);
            int s = 0;
            if (pass > 0) {
                const uint32_t hi = key >> (shift + 8);
                s = -1;
                for (int q = 0; q < ns; ++q)
                    if (sm.slot_pref[q] == hi) s = q;
            }
            if (s >= 0) atomicAdd(&sm.hist[s][(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        for (int t = wave; t < ntgt; t += nwaves) {
            const uint32_t *h = sm.hist[sm.slot[t]];
            uint32_t c[4], tot = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = h[4 * lane + q];
                tot += c[q];
            }
            uint32_t inc = tot;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(inc, off, 64);
                if (lane >= off) inc += o;
            }
            const uint32_t before = inc - tot;
            const uint32_t r = (uint32_t)sm.rank[t];
            if (r >= before && r < inc) {
                uint32_t acc = before;
                int d = 0;
                while (d < 3 && r >= acc + c[d]) acc += c[d++];
                sm.pref[t] = (sm.pref[t] << 8) | (uint32_t)(4 * lane + d);
                sm.rank[t] = (int32_t)(r - acc);
            }
        }
        __syncthreads();
        if (tid == 0) {
            int n2 = 0;
            for (int t = 0; t < ntgt; ++t) {
                int s = -1;
                for (int q = 0; q < n2; ++q)
                    if (sm.slot_pref[q] == sm.pref[t]) s = q;
                if (s < 0) {
                    s = n2++;
                    sm.slot_pref[s] = sm.pref[t];
                }
                sm.slot[t] = s;
            }
            sm.nslots = n2;
        }
        __syncthreads();
    }
}

// Per-row statistics (64 bytes).
struct RowStats {
    float v[NTGT];      // 1st, 2nd, 4th, 8th, 16th, 32nd largest; quantiles 1, 10, 25, 50, 75 %
    float diag;         // s(k,k)
    int32_t above;      // #{j != k : s(k,j) > s(k,k)}
    int32_t pad;
    double top_sum;     // sum of the min(32, n-1) largest
};
static_assert(sizeof(RowStats) == 64, "RowStats layout");
constexpr int Q50 = 9;  // index of the median in RowStats::v

__constant__ int kDesc[6] = {0, 1, 3, 7, 15, 31};
__constant__ int kQuant[5] = {1, 10, 25, 50, 75};

// Ascending rank of the q-th order statistic among the row's m values.
__device__ __forceinline__ int32_t stat_rank(int q, int64_t m) {
    if (q >= 6) return (int32_t)(((int64_t)kQuant[q - 6] * (m - 1)) / 100);
    const int64_t j = kDesc[q];
    return (int32_t)(m - 1 - (j < m - 1 ? j : m - 1));
}

// From the keys of the order statistics: the sum of the 32 largest and the
// elements above the diagonal; writes the row's statistics.
template <int T, class Each>
__device__ __forceinline__ void row_tail(Each each, const uint32_t *keys, float dg, int64_t m, double *wsum,
                                         int32_t *wcnt, RowStats *out) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t key32 = keys[5];
    double s = 0.0;
    int32_t gt = 0, above = 0;
    each([&](float x) {
        if (fkey(x) > key32) {
            s += (double)x;
            ++gt;
        }
        above += (x > dg) ? 1 : 0;
    });
    // (the counts as one word: at most 65536 and 31)
    int32_t both = above << 6 | gt;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_down(s, off, 64);
        both += __shfl_down(both, off, 64);
    }
    if (lane == 0) {
        wsum[wave] = s;
        wcnt[wave] = both;
    }
    __syncthreads();
    if (tid < NTGT) out->v[tid] = keyf(keys[tid]);
    if (wave == 1) {
        double tot = lane < T / 64 ? wsum[lane] : 0.0;
        both = lane < T / 64 ? wcnt[lane] : 0;
#pragma unroll
        for (int off = T / 128; off > 0; off >>= 1) {
            tot += __shfl_down(tot, off, 64);
            both += __shfl_down(both, off, 64);
        }
        if (lane > 0) return;
        const int32_t a = both >> 6, g = both & 63;
        const int32_t cnt = m < TOP ? (int32_t)m : TOP;
        out->diag = dg;
        out->above = a;
        out->pad = 0;
        out->top_sum = tot + (double)(cnt - g) * (double)keyf(key32);
    }
}

// Order statistics of one row, all eleven at once.  The row is cut into
// kBins intervals of equal width between its least and largest value; the
// cut is a monotone function of the value, so the counts of the intervals
// tell which one holds each rank.  The few keys of those intervals are
// collected and ranked by counting.  Against the digits of a radix select
// (four passes, whose first digits are the exponent and put most of a row on
// a few LDS counters) a row takes two passes over registers: 5000 rows of
// 5000 85 us, 514 before.  A row whose values crowd (ties, a far outlier:
// more than kCand keys in the eleven intervals, or many_keys in one, where
// counting costs a multiple of the rest) is left to k_row_stats_crowded, and
// so is one that holds a value that is not finite.
constexpr int ST_T = 512;
constexpr int kBins = 2048, kCand = 1024;
static_assert(kBins == 4 * ST_T, "four intervals per thread");
// Keys of an interval that are still ranked by counting.  Counting grows with
// the square (64: 2 us of a row, 256: 25), another cut with the row: 300 points
// with one far out 27 us at 64, 95 at 256; 5000 with one far out 319 us at 128,
// 412 at 64; a mixture of 20000 points (a hundred keys in many intervals) 1.2 ms
// at 256, 3.1 at 64.
__device__ __forceinline__ int many_keys(int n) { return n <= 2048 ? 64 : n <= 8192 ? 128 : 256; }

// Counts intervals one element at a time; MERGE (long rows, read again in
// every pass): a thread's elements of one interval in a row are added at once,
// so a crowded row does not wait for one LDS counter (20000 points, one of
// them far out: 5.3 ms for all rows, 5.8 without).
template <bool MERGE>
struct Counter {
    uint32_t *hist;
    int at = -1;
    uint32_t held = 0u;
    __device__ __forceinline__ void add(int b) {
        if constexpr (MERGE) {
            if (b != at) {
                if (held) atomicAdd(&hist[at], held);
                at = b;
                held = 0u;
            }
            ++held;
        } else {
            atomicAdd(&hist[b], 1u);
        }
    }
    __device__ __forceinline__ void flush() {
        if (MERGE && held) atomicAdd(&hist[at], held);
    }
};

struct BinShared {
    uint32_t hist[kBins];
    uint8_t mark[kBins];       // 1 + list of an interval that holds a rank
    uint32_t cand[kCand];      // keys of those intervals, list by list
    uint32_t wtot[ST_T / 64];
    int32_t bin[NTGT], rank[NTGT], cnt[NTGT];   // a rank's interval, its rank in it, the interval's keys
    int32_t off[NTGT];         // first key of a rank's list
    int32_t cursor[NTGT];      // by list
    int32_t total, most;       // keys of the lists, of the longest
    float lo[ST_T / 16], hi[ST_T / 16];
    uint32_t key[NTGT];
};

// From the counts of the intervals (bs.hist, complete): the interval, rank
// inside it and list of every rank lane q of `want` asks for (lane < NTGT; a
// rank beyond the counted keys is not looked up).  Ranks in one interval
// share the list of the first of them.  Ends with a barrier.
__device__ __forceinline__ void find_intervals(BinShared &bs, int32_t want) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    {
        const uint4 h = *reinterpret_cast<const uint4 *>(&bs.hist[4 * tid]);
        const uint32_t c[4] = {h.x, h.y, h.z, h.w}, tot = h.x + h.y + h.z + h.w;
        uint32_t inc = tot;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (lane == 63) bs.wtot[wave] = inc;
        __syncthreads();
        uint32_t before = inc - tot;
        for (int w = 0; w < wave; ++w) before += bs.wtot[w];
#pragma unroll
        for (int q = 0; q < NTGT; ++q) {
            const uint32_t r = (uint32_t)__builtin_amdgcn_readlane(want, q);
            if (r >= before && r < before + tot) {
                uint32_t acc = before;
                int d = 0;
                while (d < 3 && r >= acc + c[d]) acc += c[d++];
                bs.bin[q] = 4 * tid + d;
                bs.rank[q] = (int32_t)(r - acc);
                bs.cnt[q] = (int32_t)c[d];
            }
        }
    }
    __syncthreads();
    // one list per interval: lane q has rank q; equal intervals share the
    // first one's list
    if (wave == 0) {
        const bool live = lane < NTGT && want >= 0;
        const int b = live ? bs.bin[lane] : -1 - lane;
        const int c = live ? bs.cnt[lane] : 0;
        int first = lane;
#pragma unroll
        for (int q = NTGT - 1; q >= 0; --q)
            if (__builtin_amdgcn_readlane(b, q) == b && q < first) first = q;
        const bool own = live && first == lane;
        int at = 0, total = 0, most = 0;
#pragma unroll
        for (int q = 0; q < NTGT; ++q) {
            const int cq = __builtin_amdgcn_readlane(own ? c : 0, q);
            if (q < first) at += cq;
            total += cq;
            most = cq > most ? cq : most;
        }
        if (lane < NTGT) bs.off[lane] = at;
        if (own) {
            bs.mark[b] = (uint8_t)(1 + lane);
            bs.cursor[lane] = at;
        }
        if (lane == 0) {
            bs.total = total;
            bs.most = most;
        }
    }
    __syncthreads();
}

// The keys of the ranks in `want` from their lists in bs.cand, by counting.
__device__ __forceinline__ void rank_lists(BinShared &bs, int32_t want) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = wave; q < NTGT; q += ST_T / 64) {
        if (__builtin_amdgcn_readlane(want, q) < 0) continue;
        const uint32_t *l = bs.cand + bs.off[q];
        const int c = bs.cnt[q], r = bs.rank[q];
        for (int e = lane; e < c; e += 64) {
            const uint32_t x = l[e];
            int less = 0, same = 0;
#pragma unroll 4
            for (int i = 0; i < c; ++i) {
                less += l[i] < x;
                same += l[i] == x;
            }
            if (r >= less && r < less + same) bs.key[q] = x;   // (equal keys write the same)
        }
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
// E > 0: the row (n <= E * ST_T) is held in registers; 0: read again.  (8 to 20
// bytes per lane go through scratch from E = 4 on: the bounds are for four
// workgroups to a compute unit, three with 16 elements.)
template <int E>
__global__ __launch_bounds__(ST_T, E > 8 ? 6 : 8) void k_row_stats(const float *S, int64_t ld, int32_t n, RowStats *out) {
    __shared__ BinShared bs;
    __shared__ double wsum[ST_T / 64];
    __shared__ int32_t wcnt[ST_T / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t m = n - 1;
    const int32_t want = lane < NTGT ? stat_rank(lane, m) : -1;   // the ranks, lane by lane
    for (int64_t k = blockIdx.x; k < n; k += gridDim.x) {
        const float *row = S + k * ld;
        float v[E > 0 ? E : 1];
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int j = tid + e * ST_T;
                v[e] = j < n ? row[j] : 0.0f;
            }
        }
        auto each = [&](auto f) {
            if constexpr (E > 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int j = tid + e * ST_T;
                    if (j < n && j != (int)k) f(v[e]);
                }
            } else {
                // eight loads in flight (20000 points 1.69 -> 1.10 ms)
                for (int j0 = tid; j0 < n; j0 += 8 * ST_T) {
                    float x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = j0 + u * ST_T < n ? row[j0 + u * ST_T] : 0.0f;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int j = j0 + u * ST_T;
                        if (j < n && j != (int)k) f(x[u]);
                    }
                }
            }
        };
        float lo = INFINITY, hi = -INFINITY;
        bool nan = false;
        each([&](float x) {
            lo = fminf(lo, x);
            hi = fmaxf(hi, x);
            nan |= x != x;
        });
        if (nan) lo = -INFINITY;
        // over each 16 lanes (quad swaps, half-row and row mirrors)
        lo = fminf(lo, dpp_mov<0xB1>(lo)), hi = fmaxf(hi, dpp_mov<0xB1>(hi));
        lo = fminf(lo, dpp_mov<0x4E>(lo)), hi = fmaxf(hi, dpp_mov<0x4E>(hi));
        lo = fminf(lo, dpp_mov<0x141>(lo)), hi = fmaxf(hi, dpp_mov<0x141>(hi));
        lo = fminf(lo, dpp_mov<0x140>(lo)), hi = fmaxf(hi, dpp_mov<0x140>(hi));
        if ((lane & 15) == 0) {
            bs.lo[tid >> 4] = lo;
            bs.hi[tid >> 4] = hi;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) bs.hist[tid + q * ST_T] = 0u;
        reinterpret_cast<uint32_t *>(bs.mark)[tid] = 0u;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < ST_T / 64; ++w) {
            const float4 a = *reinterpret_cast<const float4 *>(&bs.lo[4 * w]);
            const float4 b = *reinterpret_cast<const float4 *>(&bs.hi[4 * w]);
            lo = fminf(fminf(fminf(lo, a.x), fminf(a.y, a.z)), a.w);
            hi = fmaxf(fmaxf(fmaxf(hi, b.x), fmaxf(b.y, b.z)), b.w);
        }
        // A row that cannot be cut into equal widths (an infinity, a NaN, whose
        // place is that of its key, a range beyond FP32, one value only) has no
        // interval here.
        if (!(hi - lo < INFINITY) || (hi == lo && m > many_keys(n))) {
            if (tid == 0) out[k].pad = 1;      // left to k_row_stats_crowded
            __syncthreads();
            continue;
        }
        const float inv = (float)(kBins - 1) / (hi - lo);
        auto bin_of = [&](float x) -> int {
            const int b = (int)((x - lo) * inv);
            return b < 0 ? 0 : b > kBins - 1 ? kBins - 1 : b;
        };
        Counter<E == 0> count{bs.hist};
        each([&](float x) { count.add(bin_of(x)); });
        count.flush();
        __syncthreads();
        find_intervals(bs, want);
        const bool crowded = bs.total > kCand || bs.most > many_keys(n);
        if (!crowded) {
            each([&](float x) {
                const int q = bs.mark[bin_of(x)];
                if (q) bs.cand[atomicAdd(&bs.cursor[q - 1], 1)] = fkey(x);
            });
            __syncthreads();
            rank_lists(bs, want);
        }
        __syncthreads();
        if (crowded) {
            if (tid == 0) out[k].pad = 1;
            continue;
        }
        row_tail<ST_T>(each, bs.key, row[k], m, wsum, wcnt, out + k);
        __syncthreads();
    }
}

// The rows that k_row_stats left.  Here the cut is of the keys, so that the
// width of an interval follows the exponent (a far outlier costs a tenth of
// the intervals, not all but one), and it is repeated: the interval of a rank
// that holds too many keys is cut again, between the least and the largest of
// them, until few keys are left or one key only (ties).  A cut divides a
// range of keys by at least 128 (2048 intervals over at most eleven lists),
// so five serve any row; most take one or two.  1000 points of which one lies
// far out: 42 us for all rows, 1718 by counting one long list, 76 with the
// digits of a radix select; 5000: 319 us, 520 with the digits.
template <int E>
__global__ __launch_bounds__(ST_T) void k_row_stats_crowded(const float *S, int64_t ld, int32_t n, RowStats *out) {
    __shared__ BinShared bs;
    __shared__ double wsum[ST_T / 64];
    __shared__ int32_t wcnt[ST_T / 64];
    __shared__ uint32_t la[NTGT], lb[NTGT];   // the lists of the cut: least and largest key, ascending
    __shared__ int32_t lsh[NTGT];             // ... keys to an interval (a power of two: its exponent)
    __shared__ uint32_t kmin[NTGT], kmax[NTGT];
    __shared__ int32_t nlists, lbits, wanted[NTGT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m = n - 1;
    unsigned long long left = 0ull;           // of 64 rows of this workgroup, those still to do
    for (int64_t base = blockIdx.x, k;;) {
        if (left == 0ull) {
            if (base >= n) break;
            const int64_t mine = base + (int64_t)lane * gridDim.x;
            left = __ballot(mine < n && out[mine < n ? mine : 0].pad != 0);
            base += 64 * (int64_t)gridDim.x;
            __syncthreads();                  // (row_tail rewrites pad)
            continue;
        }
        k = base + ((int64_t)__builtin_ctzll(left) - 64) * gridDim.x;
        left &= left - 1ull;
        const float *row = S + k * ld;
        float v[E > 0 ? E : 1];
        if constexpr (E > 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int j = tid + e * ST_T;
                v[e] = j < n ? row[j] : 0.0f;
            }
        }
        auto each = [&](auto f) {
            if constexpr (E > 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int j = tid + e * ST_T;
                    if (j < n && j != (int)k) f(v[e]);
                }
            } else {
                // eight loads in flight
                for (int j0 = tid; j0 < n; j0 += 8 * ST_T) {
                    float x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = j0 + u * ST_T < n ? row[j0 + u * ST_T] : 0.0f;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int j = j0 + u * ST_T;
                        if (j < n && j != (int)k) f(x[u]);
                    }
                }
            }
        };
        // the first list: every key
        if (tid == 0) {
            kmin[0] = 0xffffffffu;
            kmax[0] = 0u;
        }
        if (tid < NTGT) {
            wanted[tid] = bs.rank[tid] = stat_rank(tid, m);
            bs.bin[tid] = 0;
            bs.cnt[tid] = (int32_t)m;
        }
        __syncthreads();
        uint32_t a = 0xffffffffu, b = 0u;
        each([&](float x) {
            a = min(a, fkey(x));
            b = max(b, fkey(x));
        });
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            a = min(a, (uint32_t)__shfl_xor((int)a, off, 64));
            b = max(b, (uint32_t)__shfl_xor((int)b, off, 64));
        }
        if (lane == 0) {
            atomicMin(&kmin[0], a);
            atomicMax(&kmax[0], b);
        }
        __syncthreads();
        bool done = false;
        while (!done) {
            // Lane q has rank q, in the list of the first rank that shares its
            // interval, whose bounds are kmin and kmax: a list of one key has
            // the answer, the others are cut again.
            if (wave == 0) {
                const bool live = lane < NTGT && wanted[lane < NTGT ? lane : 0] >= 0;
                const int b0 = live ? bs.bin[lane] : -1 - lane;
                int own = lane;
#pragma unroll
                for (int q = NTGT - 1; q >= 0; --q)
                    if (__builtin_amdgcn_readlane(b0, q) == b0 && q < own) own = q;
                const uint32_t x = live ? kmin[own] : 0u, y = live ? kmax[own] : 0u;
                const bool cut = live && x != y, mine = cut && own == lane;
                if (live && !cut) bs.key[lane] = x;
                // lists in ascending order of their keys; keys before this rank's list
                int at = 0, before = 0, lists = 0;
#pragma unroll
                for (int q = 0; q < NTGT; ++q) {
                    const int bq = __builtin_amdgcn_readlane(b0, q);
                    const int cq = __builtin_amdgcn_readlane(mine ? bs.cnt[lane] : 0, q);
                    if (cq > 0) {
                        ++lists;
                        if (bq < b0) {
                            ++at;
                            before += cq;
                        }
                    }
                }
                const int bits = lists > 8 ? 7 : lists > 4 ? 8 : lists > 2 ? 9 : lists > 1 ? 10 : 11;
                if (mine) {
                    const int span = 32 - __builtin_clz(y - x);
                    la[at] = x;
                    lb[at] = y;
                    lsh[at] = span > bits ? span - bits : 0;
                }
                if (lane < NTGT) wanted[lane] = cut ? before + bs.rank[lane] : -1;
                if (lane == 0) {
                    nlists = lists;
                    lbits = bits;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) bs.hist[tid + q * ST_T] = 0u;
            reinterpret_cast<uint32_t *>(bs.mark)[tid] = 0u;
            __syncthreads();
            const int lists = nlists, bits = lbits;
            if (lists == 0) break;
            const int32_t want = lane < NTGT ? wanted[lane] : -1;
            auto slot = [&](uint32_t key) -> int {      // interval of a key, -1: in no list
                int d = 0;
                for (int u = 1; u < lists; ++u) d += key >= la[u];
                return key >= la[d] && key <= lb[d] ? (int)(d << bits | (key - la[d]) >> lsh[d]) : -1;
            };
            Counter<E == 0> count{bs.hist};
            each([&](float x) {
                const int b1 = slot(fkey(x));
                if (b1 >= 0) count.add(b1);
            });
            count.flush();
            __syncthreads();
            find_intervals(bs, want);
            done = bs.total <= kCand && bs.most <= many_keys(n);
            if (tid < NTGT) {
                kmin[tid] = 0xffffffffu;
                kmax[tid] = 0u;
            }
            __syncthreads();
            each([&](float x) {
                const uint32_t key = fkey(x);
                const int b1 = slot(key);
                const int q = b1 >= 0 ? bs.mark[b1] : 0;
                if (q == 0) return;
                if (done) {
                    bs.cand[atomicAdd(&bs.cursor[q - 1], 1)] = key;
                } else {
                    // (the bounds only ever widen: most keys change neither)
                    if (key < __atomic_load_n(&kmin[q - 1], __ATOMIC_RELAXED)) atomicMin(&kmin[q - 1], key);
                    if (key > __atomic_load_n(&kmax[q - 1], __ATOMIC_RELAXED)) atomicMax(&kmax[q - 1], key);
                }
            });
            __syncthreads();
            if (done) rank_lists(bs, want);
        }
        __syncthreads();
        row_tail<ST_T>(each, bs.key, row[k], m, wsum, wcnt, out + k);
        __syncthreads();
    }
}

// sigma = |lower median of the row medians| (1 if that is 0 or not finite).
__global__ __launch_bounds__(SEL_T) void k_sigma(const RowStats *st, int32_t n, float *sigma) {
    __shared__ SelShared sm;
    if (threadIdx.x == 0) sm.rank[0] = (n - 1) / 2;
    radix_select(sm, n, 1, [&](int64_t j) { return fkey(st[j].v[Q50]); });
    if (threadIdx.x == 0) {
        float s = fabsf(keyf(sm.pref[0]));
        if (!(s > 0.0f) || !(s < INFINITY)) s = 1.0f;
        *sigma = s;
    }
}

__global__ void k_features(const RowStats *st, int32_t n, const float *sigma, float ln_n_10, float *F) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const RowStats r = st[k];
    const double sg = (double)*sigma;
    const int64_t m = n - 1;
    const double tm = r.top_sum / (double)(m < TOP ? m : TOP);
    float f[NF];
    for (int t = 0; t < 6; ++t) f[t] = (float)((double)r.v[t] / sg);
    f[6] = (float)(tm / sg);
    for (int q = 0; q < 5; ++q) f[7 + q] = (float)((double)r.v[6 + q] / sg);
    f[12] = (float)(((double)r.diag - (double)r.v[Q50]) / sg);
    f[13] = (float)(((double)r.diag - tm) / sg);
    f[14] = (float)((double)r.above / (double)m);
    f[15] = ln_n_10;
    float4 *o = reinterpret_cast<float4 *>(F + k * NF);
    for (int q = 0; q < 4; ++q) o[q] = make_float4(f[4 * q], f[4 * q + 1], f[4 * q + 2], f[4 * q + 3]);
}

// ---------------------------------------------------------------------------
// Network
// ---------------------------------------------------------------------------
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// gfx950's 32x32x16 bf16 matrix op (FP32 accumulate): lane l holds row (or
// column) l mod 32 and k = 8 (l / 32) .. + 7 of its operand.  The two halves
// of an operand come from 8-byte aligned LDS rows (their padding keeps the
// 8-byte loads free of bank conflicts).
__device__ __forceinline__ v16f mfma16(v4s a0, v4s a1, v4s b0, v4s b1, v16f c) {
    const v8s a = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    const v8s b = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0,
                                                   0, 0);
}

__device__ __forceinline__ v16f zero16() {
    v16f z;
#pragma unroll
    for (int q = 0; q < 16; ++q) z[q] = 0.0f;
    return z;
}

// Round to bfloat16, nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t bf16_bits(float x) {
    const uint32_t b = __float_as_uint(x);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((b >> 16) | 0x40u);
    return (uint16_t)((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf16_val(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// GELU z Phi(z) and its derivative Phi(z) + z phi(z).
__device__ __forceinline__ float gelu(float z) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// The network runs on tiles of 32 points, one workgroup of four wavefronts per
// tile at a time; wavefront w has units 32 w .. + 31 of both hidden layers.
// Small tiles because the batches are small: 32 points make 256 workgroups
// out of 8192 rows, and the chain of dependent steps of a tile (three layers,
// two of them with a GELU per element, then three products backward), not
// arithmetic, is what a pass waits for.  The weights are rounded to bf16 into
// LDS once per workgroup.
constexpr int TW = 256;             // threads
constexpr int TP = 32;              // points per tile
constexpr int LW1 = NF + 4;         // padded row of W1^T in LDS (bf16)
constexpr int LW2 = NH + 4;         // padded row of W2^T and of the activations
constexpr int LDZ = NH + 1;         // padded row of a pre-activation gradient
constexpr int kMaxTileBlocks = 256; // workgroups of the gradient kernel
// Partial gradients are FP32 sums over at most 64 points and are added in
// FP64: a slot is one tile or two, whichever gives the busiest workgroup fewer
// tiles (two on a tie: half the partials).  At most kMaxSlots of them (154 MB) are held at a time.
constexpr int64_t kMaxSlots = 2048;

struct TileShared {
    uint16_t w1t[NH * LW1];         // W1^T [unit][feature]
    uint16_t w2t[NH * LW2];         // W2^T [unit out][unit in]
    uint16_t h1[TP * LW2], h2[TP * LW2];   // activations [point][unit]
    float w3[NH * NO];              // bf16-rounded W3 [unit][output]
    float b1[NH], b2[NH], b3[4];
};

// Thread -> one output unit and half of the inputs: the loads of a wavefront
// are consecutive, and four inputs at a time go to the unit's row as one
// 8-byte write (one 2-byte write per weight took 18 us on conflicting banks).
__device__ __forceinline__ void tile_weights(TileShared &sh, const float *theta) {
    const int tid = threadIdx.x, j = tid & (NH - 1), half = tid >> 7;
    const float *w1 = theta + OFF_W1 + half * (NF / 2) * NH + j, *w2 = theta + OFF_W2 + half * (NH / 2) * NH + j;
    auto pack = [](float x, float y, float z, float w) {
        return v4s{(short)bf16_bits(x), (short)bf16_bits(y), (short)bf16_bits(z), (short)bf16_bits(w)};
    };
#pragma unroll
    for (int i = 0; i < NF / 2; i += 4)
        *reinterpret_cast<v4s *>(sh.w1t + j * LW1 + half * (NF / 2) + i) =
            pack(w1[i * NH], w1[(i + 1) * NH], w1[(i + 2) * NH], w1[(i + 3) * NH]);
#pragma unroll
    for (int i = 0; i < NH / 2; i += 4)
        *reinterpret_cast<v4s *>(sh.w2t + j * LW2 + half * (NH / 2) + i) =
            pack(w2[i * NH], w2[(i + 1) * NH], w2[(i + 2) * NH], w2[(i + 3) * NH]);
    sh.w3[tid] = bf16_val(bf16_bits(theta[OFF_W3 + tid]));
    if (tid < NH) {
        sh.b1[tid] = theta[OFF_B1 + tid];
        sh.b2[tid] = theta[OFF_B2 + tid];
    }
    if (tid < NO) sh.b3[tid] = theta[OFF_B3 + tid];
}

// The features of point lane % 32 of the tile, k = 8 (lane / 32) .. + 7
// (zeros outside the batch), as bf16.
__device__ __forceinline__ void tile_features(const float *F, const int64_t *rows, int64_t count, int64_t p0,
                                              int lane, v4s (&xa)[2]) {
    const int64_t p = p0 + (lane & 31);
    const int64_t src = p < count ? (rows ? rows[p] : p) : -1;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float4 f = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (src >= 0) f = *reinterpret_cast<const float4 *>(F + src * NF + (lane >> 5) * 8 + 4 * h);
        xa[h] = v4s{(short)bf16_bits(f.x), (short)bf16_bits(f.y), (short)bf16_bits(f.z), (short)bf16_bits(f.w)};
    }
}

// Bias, GELU and bf16 rounding of this wavefront's 32 x 32 layer output held
// in MFMA accumulators (lane l holds unit l % 32 and points 8 (v / 4) + 4 (l /
// 32) + v % 4); GRAD: the GELU's slopes stay in `slope`, in the same places.
template <bool GRAD>
__device__ __forceinline__ void tile_epilogue(const v16f &acc, const float *bias, uint16_t *h, int lane, int wave,
                                              float (&slope)[16]) {
    const int j = 32 * wave + (lane & 31);
    const float bj = bias[j];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        const float z = acc[v] + bj;
        h[r * LW2 + j] = bf16_bits(gelu(z));
        if (GRAD) slope[v] = gelu_grad(z);
    }
}

// Both hidden layers of a tile; ends with a barrier, h1 and h2 complete.
template <bool GRAD>
__device__ __forceinline__ void tile_hidden(TileShared &sh, const v4s (&xa)[2], int lane, int wave,
                                            float (&g1)[16], float (&g2)[16]) {
    const int li = lane & 31, lk = (lane >> 5) * 8;
    {
        const uint16_t *w = sh.w1t + (32 * wave + li) * LW1 + lk;
        const v16f acc = mfma16(xa[0], xa[1], *reinterpret_cast<const v4s *>(w),
                                *reinterpret_cast<const v4s *>(w + 4), zero16());
        tile_epilogue<GRAD>(acc, sh.b1, sh.h1, lane, wave, g1);
    }
    __syncthreads();
    // Layer 2: K = 128 in 8 steps of 16
    v16f acc = zero16();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const uint16_t *hr = sh.h1 + li * LW2 + 16 * ks + lk;
        const uint16_t *w = sh.w2t + (32 * wave + li) * LW2 + 16 * ks + lk;
        acc = mfma16(*reinterpret_cast<const v4s *>(hr), *reinterpret_cast<const v4s *>(hr + 4),
                     *reinterpret_cast<const v4s *>(w), *reinterpret_cast<const v4s *>(w + 4), acc);
    }
    tile_epilogue<GRAD>(acc, sh.b2, sh.h2, lane, wave, g2);
    __syncthreads();
}

// Output lane / 32 of point lane % 32 (128 -> 2 on the vector units), summed
// over the units in their order by one wavefront: the value does not depend on
// how the units are split, and a sum of the four wavefronts' parts is no faster
// (8192 rows 44.2 us, 44.3 so).
__device__ __forceinline__ float tile_output(const TileShared &sh, int lane) {
    const int o = lane >> 5;
    const uint16_t *hr = sh.h2 + (lane & 31) * LW2;
    const float *w3 = sh.w3 + o;
    float y = 0.0f;
#pragma unroll 8
    for (int j = 0; j < NH; j += 4) {
        const v4s h = *reinterpret_cast<const v4s *>(hr + j);
        y = fmaf(bf16_val((uint16_t)h.x), w3[j * NO], y);
        y = fmaf(bf16_val((uint16_t)h.y), w3[(j + 1) * NO], y);
        y = fmaf(bf16_val((uint16_t)h.z), w3[(j + 2) * NO], y);
        y = fmaf(bf16_val((uint16_t)h.w), w3[(j + 3) * NO], y);
    }
    return y + sh.b3[o];
}

struct FwdArgs {
    const float *theta;             // FP32 master parameters
    const float *F;                 // features, count x 16
    int64_t count;
    float *Y;                       // count x 2
};

// 5000 points: 15 us (47 us with 128 points to a workgroup, 40 of them); the
// weights' way into LDS and the GELUs take most of it.
__global__ __launch_bounds__(TW) void k_mlp_fwd(FwdArgs a) {
    __shared__ __align__(16) TileShared sh;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v4s xa[2];
    tile_features(a.F, nullptr, a.count, (int64_t)blockIdx.x * TP, lane, xa);   // in flight with the weights
    tile_weights(sh, a.theta);
    __syncthreads();
    const int64_t tiles = (a.count + TP - 1) / TP;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t p0 = tile * TP;
        if (tile != blockIdx.x) tile_features(a.F, nullptr, a.count, p0, lane, xa);
        float g1[16], g2[16];
        tile_hidden<false>(sh, xa, lane, wave, g1, g2);
        if (wave == 0) {
            const float y = tile_output(sh, lane);
            if (p0 + (lane & 31) < a.count) a.Y[(p0 + (lane & 31)) * NO + (lane >> 5)] = y;
        }
        // (h2 is written again only after the next tile's first barrier)
    }
}

struct BwdShared {
    TileShared t;
    float dz[TP * LDZ];             // gradient at the second, then the first pre-activation
    float x[TP * (NF + 1)];         // bf16-rounded features
    float dy[TP * NO];
};

struct BwdArgs {
    const float *theta;
    const float *F, *T, *w;         // features (count x 16), targets (count x 2), weights (count)
    const int64_t *rows;            // nullable batch indices into F, T, w
    int64_t count;
    int64_t slot0;                  // first slot of this launch
    int32_t slots, per;             // slots of this launch, tiles of a slot
    float *gpart;                   // [slots][NPARAM]
    double *lpart;                  // [slots]
};

// Forward and backward of the workgroup's tiles in one kernel (activations
// and slopes never leave the chip); the products of the backward pass run on
// the FP32 matrix op (32x32x2: bf16 activations and weights are exact in
// FP32, gradients stay FP32).  Writes a partial gradient per slot.  8192
// rows: 37 us (forward 52 and backward 149 us while the activations went
// through memory and the products ran on the vector units).
// ONE: a workgroup has one tile.
template <bool ONE>
__global__ __launch_bounds__(TW) void k_mlp_bwd(BwdArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    BwdShared &sh = *reinterpret_cast<BwdShared *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, hi = lane >> 5;
    v4s xa[2];
    const int64_t first = (a.slot0 + blockIdx.x) * a.per;
    tile_features(a.F, a.rows, a.count, first * TP, lane, xa);   // in flight with the weights
    tile_weights(sh.t, a.theta);
    __syncthreads();

    const int64_t tiles = (a.count + TP - 1) / TP;
    for (int slot = blockIdx.x; slot < a.slots; slot += ONE ? a.slots : gridDim.x) {
        float *g = a.gpart + (int64_t)slot * NPARAM;
        v16f dw2[4], dw1 = zero16();    // dW2 rows 32 wave + ., dW1^T-tile: features x units 32 wave + .
#pragma unroll
        for (int q = 0; q < 4; ++q) dw2[q] = zero16();
        float dw3 = 0.0f, db1 = 0.0f, db2 = 0.0f, db3 = 0.0f;
        double lsum = 0.0;

        const int64_t tile0 = (a.slot0 + slot) * a.per;
        for (int64_t tile = tile0; tile < tile0 + (ONE ? 1 : a.per) && tile < tiles; ++tile) {
            const int64_t p0 = tile * TP;
            if (!ONE && tile != first) tile_features(a.F, a.rows, a.count, p0, lane, xa);
            if (wave == 3) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sh.x[li * (NF + 1) + 8 * hi + 4 * h + e] = bf16_val((uint16_t)xa[h][e]);
            }
            float g1[16], g2[16];
            tile_hidden<true>(sh.t, xa, lane, wave, g1, g2);
            // Loss and its gradient at the outputs: w_p * Huber(y - t), delta 1
            if (wave == 0) {
                float d = 0.0f, wp = 0.0f, target = 0.0f;
                const int64_t p = p0 + li;
                if (p < a.count) {
                    const int64_t src = a.rows ? a.rows[p] : p;
                    target = a.T[src * NO + hi];
                    wp = a.w[src];
                }
                const float y = tile_output(sh.t, lane);
                if (p < a.count) {
                    const float e = y - target;
                    d = wp * fminf(1.0f, fmaxf(-1.0f, e));
                    const double ae = fabs((double)e);
                    lsum += (double)wp * (ae <= 1.0 ? 0.5 * (double)e * (double)e : ae - 0.5);
                }
                sh.dy[li * NO + hi] = d;
            }
            __syncthreads();
            // dz2 = (W3 dy) * GELU'(z2), in the layout of the layer's output
            {
                const int j = 32 * wave + li;
                const float wa = sh.t.w3[j * NO], wb = sh.t.w3[j * NO + 1];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 8 * (v >> 2) + 4 * hi + (v & 3);
                    sh.dz[r * LDZ + j] = fmaf(wa, sh.dy[r * NO], wb * sh.dy[r * NO + 1]) * g2[v];
                }
            }
            // dW3[j][o] = sum_p h2[p][j] dy[p][o]; db3
            {
                const int j = tid >> 1, o = tid & 1;
#pragma unroll 8
                for (int p = 0; p < TP; ++p) dw3 = fmaf(bf16_val(sh.t.h2[p * LW2 + j]), sh.dy[p * NO + o], dw3);
                if (tid < NO)
                    for (int p = 0; p < TP; ++p) db3 += sh.dy[p * NO + tid];
            }
            __syncthreads();
            // dW2[i][j] = sum_p h1[p][i] dz2[p][j]; db2
#pragma unroll 4
            for (int ks = 0; ks < TP / 2; ++ks) {
                const int p = 2 * ks + hi;
                const float av = bf16_val(sh.t.h1[p * LW2 + 32 * wave + li]);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    dw2[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, sh.dz[p * LDZ + 32 * q + li], dw2[q], 0, 0, 0);
            }
            if (tid < NH)
                for (int p = 0; p < TP; ++p) db2 += sh.dz[p * LDZ + tid];
            // dz1[p][i] = (sum_j dz2[p][j] W2[i][j]) * GELU'(z1): two chains of K
            v16f s0 = zero16(), s1 = zero16();
#pragma unroll 8
            for (int ks = 0; ks < NH / 2; ks += 2) {
                const int j0 = 2 * ks + hi, j1 = j0 + 2;
                s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(sh.dz[li * LDZ + j0],
                                                          bf16_val(sh.t.w2t[j0 * LW2 + 32 * wave + li]), s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(sh.dz[li * LDZ + j1],
                                                          bf16_val(sh.t.w2t[j1 * LW2 + 32 * wave + li]), s1, 0, 0, 0);
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + 4 * hi + (v & 3);
                sh.dz[r * LDZ + 32 * wave + li] = (s0[v] + s1[v]) * g1[v];
            }
            __syncthreads();
            // dW1[f][i] = sum_p x[p][f] dz1[p][i] (16 of the tile's 32 rows); db1
#pragma unroll 4
            for (int ks = 0; ks < TP / 2; ++ks) {
                const int p = 2 * ks + hi;
                const float av = li < NF ? sh.x[p * (NF + 1) + (li & (NF - 1))] : 0.0f;
                dw1 = __builtin_amdgcn_mfma_f32_32x32x2f32(av, sh.dz[p * LDZ + 32 * wave + li], dw1, 0, 0, 0);
            }
            if (tid < NH)
                for (int p = 0; p < TP; ++p) db1 += sh.dz[p * LDZ + tid];
            __syncthreads();
        }

#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + 4 * hi + (v & 3);
#pragma unroll
            for (int q = 0; q < 4; ++q) g[OFF_W2 + (32 * wave + r) * NH + 32 * q + li] = dw2[q][v];
            if (r < NF) g[OFF_W1 + r * NH + 32 * wave + li] = dw1[v];
        }
        g[OFF_W3 + tid] = dw3;
        if (tid < NH) {
            g[OFF_B1 + tid] = db1;
            g[OFF_B2 + tid] = db2;
        }
        if (tid < NO) g[OFF_B3 + tid] = db3;
        if (wave == 0) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) lsum += __shfl_down(lsum, off, 64);
            if (lane == 0) a.lpart[slot] = lsum;
        }
    }
}

// grad[e] = sum over the slots of the partials (FP64): 64 entries x 16
// slices of the partials per workgroup, slices added in order.  256 partials:
// 6 us (38 us for 128 with one serial sum per entry).  Where the slots come in
// several launches, acc (NPARAM + 1 doubles, the loss last) carries the sums:
// nullable, read unless first; grad and loss are written at the last.
__global__ __launch_bounds__(1024) void k_mlp_reduce(const float *gpart, const double *lpart, int32_t nblk,
                                                     float *grad, double *loss, double *acc, int first,
                                                     int last) {
    __shared__ double part[16][64];
    const int ex = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + ex;
    double s = 0.0;
    if (e < NPARAM) {
        int b = sl;
        for (; b + 7 * 16 < nblk; b += 8 * 16) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = gpart[(int64_t)(b + u * 16) * NPARAM + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)v[u];
        }
        for (; b < nblk; b += 16) s += (double)gpart[(int64_t)b * NPARAM + e];
    }
    part[sl][ex] = s;
    __syncthreads();
    if (sl == 0 && e < NPARAM) {
        double tot = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) tot += part[q][ex];
        if (!first) tot += acc[e];
        if (last) grad[e] = (float)tot;
        else acc[e] = tot;
    }
    if (loss && blockIdx.x == 0 && sl == 1) {
        double t = 0.0;
        for (int b = ex; b < nblk; b += 64) t += lpart[b];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
        if (ex == 0) {
            if (!first) t += acc[NPARAM];
            if (last) *loss = t;
            else acc[NPARAM] = t;
        }
    }
}

// Adam (Kingma and Ba, 2015) with bias correction factors c1 = 1/(1-beta1^t),
// c2 = 1/(1-beta2^t).
__global__ void k_adam(float *theta, float *m, float *v, const float *g, int64_t count, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    const float gi = g[e];
    const float mi = b1 * m[e] + (1.0f - b1) * gi;
    const float vi = b2 * v[e] + (1.0f - b2) * gi * gi;
    m[e] = mi;
    v[e] = vi;
    theta[e] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// ---------------------------------------------------------------------------
// Targets and A_0
// ---------------------------------------------------------------------------
// 64 columns x 16 row slices per block; slices combined in order (FP64).
__global__ __launch_bounds__(1024) void k_targets(const float *R, int64_t ld, int32_t n,
                                                  const float *sigma, float *Y) {
    __shared__ double part[16][64];
    const int c = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * 64 + c;
    double s = 0.0;
    if (k < n)
        for (int64_t i = sl; i < n; i += 16)
            if (i != k) s += (double)fmaxf(0.0f, R[i * ld + k]);
    part[sl][c] = s;
    __syncthreads();
    if (sl == 0 && k < n) {
        double cs = 0.0;
        for (int q = 0; q < 16; ++q) cs += part[q][c];
        const double sg = (double)*sigma;
        Y[k * NO + 0] = (float)(((double)R[k * ld + k] + cs) / sg);
        Y[k * NO + 1] = (float)(cs / sg);
    }
}

__device__ __forceinline__ float a0_value(const float *Y, float sg, int64_t i, int64_t k) {
    return k == i ? fmaxf(0.0f, sg * Y[i * NO + 1]) : fminf(0.0f, sg * Y[k * NO]);
}

__global__ void k_warm_a0(const float *Y, const float *sigma, int32_t n, float *A, int64_t ld) {
    const float sg = *sigma;
    const int64_t n4 = n & ~3;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        float *row = A + i * ld;
        for (int64_t k = 4 * threadIdx.x; k < n4; k += 4 * blockDim.x) {
            const float4 o = make_float4(a0_value(Y, sg, i, k), a0_value(Y, sg, i, k + 1),
                                         a0_value(Y, sg, i, k + 2), a0_value(Y, sg, i, k + 3));
            *reinterpret_cast<float4 *>(row + k) = o;
        }
        for (int64_t k = n4 + threadIdx.x; k < n; k += blockDim.x) row[k] = a0_value(Y, sg, i, k);
    }
}

// A_0 and R_0 of a row in one pass over S: A_0 as k_warm_a0 writes it and
// r(i,k) = s(i,k) - max_{k' != k} (a_0(i,k') + s(i,k')) (the undamped Eq. (2)).
// A workgroup takes whole rows; thread l of T holds the float4 chunks at
// columns 4 (l + j T) of the row and of A_0's column values, which stay in
// registers over all its rows.  The largest a + s takes the second largest
// value; under a tie the two are equal, so comparing values names it.  Reads
// S, writes A and R: 12 bytes per element (5000 points 54 us, 5.5 TB/s; A_0, R = 0 and
// the general responsibility pass took 149 us and 24 bytes).  Above 16384 points
// 68 and above 32768 points 224 bytes per lane go through scratch.
template <int T, int J>
__global__ __launch_bounds__(T) void k_warm_start(const float *S, const float *Y, const float *sigma, int32_t n,
                                                  int64_t ld, float *A, float *R) {
#pragma clang fp contract(off)
    __shared__ float sh[2][T / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float sg = *sigma;
    float col[J][4];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 4 * (tid + j * T) + e;
            col[j][e] = k < n ? a0_value(Y, sg, -1, k) : 0.0f;
        }
    int slot = 0;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x, slot ^= 1) {
        const float *srow = S + i * ld;
        const float ad = a0_value(Y, sg, i, i);
        constexpr bool HOLD = J <= 8;        // else the row is read again after the reduction
        float x[HOLD ? J : 1][4];
        auto load = [&](int j, float (&o)[4]) {
            const int c = 4 * (tid + j * T);
            float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c < n) g = *reinterpret_cast<const float4 *>(srow + c);
            o[0] = g.x;
            o[1] = g.y;
            o[2] = g.z;
            o[3] = g.w;
        };
        if constexpr (HOLD)
#pragma unroll
            for (int j = 0; j < J; ++j) load(j, x[j]);
        float v1 = -INFINITY, v2 = -INFINITY;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            float (&xs)[4] = x[HOLD ? j : 0];
            if constexpr (!HOLD) load(j, xs);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 4 * (tid + j * T) + e;
                const float v = k < n ? (k == (int)i ? ad : col[j][e]) + xs[e] : -INFINITY;
                v2 = fmaxf(v2, fminf(v1, v));
                v1 = fmaxf(v1, v);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float o1 = __shfl_xor(v1, off, 64), o2 = __shfl_xor(v2, off, 64);
            v2 = fmaxf(fmaxf(v2, o2), fminf(v1, o1));
            v1 = fmaxf(v1, o1);
        }
        if (lane == 0) {
            sh[slot][wave][0] = v1;
            sh[slot][wave][1] = v2;
        }
        __syncthreads();
        v1 = v2 = -INFINITY;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            const float o1 = sh[slot][w][0], o2 = sh[slot][w][1];
            v2 = fmaxf(fmaxf(v2, o2), fminf(v1, o1));
            v1 = fmaxf(v1, o1);
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = 4 * (tid + j * T);
            if (c >= n) continue;
            float (&xs)[4] = x[HOLD ? j : 0];
            if constexpr (!HOLD) load(j, xs);
            float ao[4], ro[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                asm volatile("" : "+v"(xs[e]));      // a + s is formed again, not held
                ao[e] = c + e == (int)i ? ad : col[j][e];
                ro[e] = xs[e] - (ao[e] + xs[e] == v1 ? v2 : v1);
            }
            float *ar = A + i * ld + c, *rr = R + i * ld + c;
            if (c + 3 < n) {
                *reinterpret_cast<float4 *>(ar) = make_float4(ao[0], ao[1], ao[2], ao[3]);
                *reinterpret_cast<float4 *>(rr) = make_float4(ro[0], ro[1], ro[2], ro[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < n) {
                        ar[e] = ao[e];
                        rr[e] = ro[e];
                    }
            }
        }
    }
}

template <int T, int J>
void launch_warm_start(const float *S, const float *Y, const float *sigma, int64_t n, int64_t ld, float *A, float *R,
                       int num_cus, hipStream_t s) {
    // as many workgroups as are resident, so that a column vector is read once
    const int64_t g = (int64_t)num_cus * (T == 256 ? 8 : 2);
    k_warm_start<T, J><<<(unsigned)(n < g ? n : g), T, 0, s>>>(S, Y, sigma, (int32_t)n, ld, A, R);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct DevGuard {
    int prev = -1;
    explicit DevGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DevGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

apx_status check_sq(apx_ctx *ctx, const float *M, const char *name, int64_t n, int64_t ld) {
    if (M == nullptr) return set_err(ctx, APX_EINVAL, "%s is null", name);
    if (!aligned16(M)) return set_err(ctx, APX_EINVAL, "%s is not 16-byte aligned", name);
    if (ld < n || ld % 4 != 0) return set_err(ctx, APX_EINVAL, "%s: need ld >= n and ld %% 4 == 0", name);
    return APX_OK;
}

unsigned grid_rows(int64_t n, int num_cus) {
    const int64_t g = (int64_t)num_cus * 2;
    return (unsigned)(n < g ? n : g);
}

// Features into F using `stats` (n RowStats) and `sigma` (device float).
apx_status run_features(apx_ctx *ctx, const float *S, int64_t n, int64_t ld, RowStats *stats,
                        float *F, float *sigma) {
    hipStream_t s = ctx->stream;
    const unsigned rows = grid_rows(n, ctx->num_cus * 4);     // four workgroups fit a compute unit
    auto both = [&](auto held) {
        constexpr int E = decltype(held)::value;
        k_row_stats<E><<<rows, ST_T, 0, s>>>(S, ld, (int32_t)n, stats);
        // (mostly nothing is left to do: no more workgroups than its registers let run)
        k_row_stats_crowded<E><<<grid_rows(n, ctx->num_cus), ST_T, 0, s>>>(S, ld, (int32_t)n, stats);
    };
    if (n <= 2 * ST_T) both(std::integral_constant<int, 2>{});
    else if (n <= 4 * ST_T) both(std::integral_constant<int, 4>{});
    else if (n <= 8 * ST_T) both(std::integral_constant<int, 8>{});
    else if (n <= 16 * ST_T) both(std::integral_constant<int, 16>{});
    else both(std::integral_constant<int, 0>{});
    HIP_TRY(hipGetLastError(), "row statistics");
    k_sigma<<<1, SEL_T, 0, s>>>(stats, (int32_t)n, sigma);
    HIP_TRY(hipGetLastError(), "sigma");
    const float ln10 = (float)(std::log((double)n) / 10.0);
    k_features<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(stats, (int32_t)n, sigma, ln10, F);
    HIP_TRY(hipGetLastError(), "features");
    return APX_OK;
}

apx_status run_forward(apx_ctx *ctx, const FwdArgs &fa) {
    const int64_t tiles = (fa.count + TP - 1) / TP;
    const int64_t most = 2 * (int64_t)ctx->num_cus;      // two workgroups fit a compute unit
    k_mlp_fwd<<<(unsigned)(tiles < most ? tiles : most), TW, 0, ctx->stream>>>(fa);
    HIP_TRY(hipGetLastError(), "network forward");
    return APX_OK;
}


struct BwdLayout {
    size_t o_gp, o_lp, o_acc, bytes;
    int64_t slots, held;     // partial gradients, of which so many in a launch
    int32_t per;             // tiles of one
};
BwdLayout bwd_layout(int64_t count) {
    const int64_t tiles = (count + TP - 1) / TP;
    WsLayout W;
    BwdLayout o{};
    const int64_t wg = kMaxTileBlocks, ones = (tiles + wg - 1) / wg, pairs = ((tiles + 1) / 2 + wg - 1) / wg;
    o.per = ones < 2 * pairs ? 1 : 2;
    o.slots = (tiles + o.per - 1) / o.per;
    o.held = o.slots < kMaxSlots ? o.slots : kMaxSlots;
    o.o_gp = W.take(sizeof(float) * NPARAM * (size_t)o.held);
    o.o_lp = W.take(sizeof(double) * (size_t)o.held);
    o.o_acc = W.take(o.slots > o.held ? sizeof(double) * (NPARAM + 1) : 0);
    o.bytes = W.off;
    return o;
}

struct WarmLayout {
    size_t o_st, o_f, o_y, o_s, head;
};
WarmLayout warm_layout(int64_t n) {
    WsLayout W;
    WarmLayout o{};
    o.o_st = W.take(sizeof(RowStats) * (size_t)n);
    o.o_f = W.take(sizeof(float) * NF * (size_t)n);
    o.o_y = W.take(sizeof(float) * NO * (size_t)n);
    o.o_s = W.take(sizeof(float) * 4);
    o.head = W.off;
    return o;
}

}  // namespace

namespace apx {
size_t features_ws_bytes(int64_t n) {
    WsLayout W;
    W.take(sizeof(RowStats) * (size_t)n);
    return W.off;
}
size_t mlp_backward_ws_bytes(int64_t count) { return bwd_layout(count).bytes; }
size_t warmstart_ws_bytes(int64_t n) { return warm_layout(n).head; }
}  // namespace apx

extern "C" {

apx_status apx_features(apx_ctx *ctx, const float *S, int64_t n, int64_t ld, float *F, float *sigma) {
    if (!ctx) return APX_EINVAL;
    if (n < 2) return set_err(ctx, APX_EINVAL, "apx_features needs n >= 2");
    if (n > 65536) return set_err(ctx, APX_ENOTIMPL, "n = %lld exceeds 65536", (long long)n);
    APX_TRY(check_sq(ctx, S, "S", n, ld));
    if (!F || !aligned16(F) || !sigma) return set_err(ctx, APX_EINVAL, "F (16-byte aligned) and sigma are required");
    DevGuard g(ctx->device);
    WsLayout W;
    const size_t o_st = W.take(sizeof(RowStats) * (size_t)n);
    APX_TRY(ws_reserve(ctx, ctx->ws_base + W.off));
    char *b = static_cast<char *>(ctx->ws) + ctx->ws_base;
    return run_features(ctx, S, n, ld, reinterpret_cast<RowStats *>(b + o_st), F, sigma);
}

apx_status apx_mlp_forward(apx_ctx *ctx, const float *theta, const float *F, int64_t count, float *Y) {
    if (!ctx) return APX_EINVAL;
    if (!theta || !F || !Y || !aligned16(F)) return set_err(ctx, APX_EINVAL, "null or misaligned argument");
    if (count < 0) return set_err(ctx, APX_EINVAL, "count < 0");
    if (count == 0) return APX_OK;
    DevGuard g(ctx->device);
    FwdArgs fa{};
    fa.theta = theta;
    fa.F = F;
    fa.count = count;
    fa.Y = Y;
    return run_forward(ctx, fa);
}

apx_status apx_mlp_backward(apx_ctx *ctx, const float *theta, const float *F, const float *T,
                            const float *w, const int64_t *rows, int64_t count, float *grad,
                            double *loss) {
    if (!ctx) return APX_EINVAL;
    if (!theta || !F || !T || !w || !grad || !aligned16(F))
        return set_err(ctx, APX_EINVAL, "null or misaligned argument");
    if (count < 1) return set_err(ctx, APX_EINVAL, "count must be >= 1");
    DevGuard g(ctx->device);
    const BwdLayout BL = bwd_layout(count);
    APX_TRY(ws_reserve(ctx, ctx->ws_base + BL.bytes));
    char *b = static_cast<char *>(ctx->ws) + ctx->ws_base;
    BwdArgs ba{};
    ba.theta = theta;
    ba.F = F;
    ba.T = T;
    ba.w = w;
    ba.rows = rows;
    ba.count = count;
    ba.gpart = reinterpret_cast<float *>(b + BL.o_gp);
    ba.lpart = reinterpret_cast<double *>(b + BL.o_lp);
    const size_t lds = sizeof(BwdShared);
    const auto kern = BL.per == 1 && BL.slots <= kMaxTileBlocks ? k_mlp_bwd<true> : k_mlp_bwd<false>;
    HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds), "lds");
    ba.per = BL.per;
    for (ba.slot0 = 0; ba.slot0 < BL.slots; ba.slot0 += BL.held) {
        const int64_t left = BL.slots - ba.slot0;
        ba.slots = (int32_t)(left < BL.held ? left : BL.held);
        kern<<<ba.slots < kMaxTileBlocks ? ba.slots : kMaxTileBlocks, TW, lds, ctx->stream>>>(ba);
        HIP_TRY(hipGetLastError(), "network backward");
        k_mlp_reduce<<<(NPARAM + 63) / 64, 1024, 0, ctx->stream>>>(ba.gpart, ba.lpart, ba.slots, grad, loss,
                                                                   reinterpret_cast<double *>(b + BL.o_acc),
                                                                   ba.slot0 == 0, left <= BL.held);
        HIP_TRY(hipGetLastError(), "gradient reduce");
    }
    return APX_OK;
}

apx_status apx_mlp_adam(apx_ctx *ctx, float *theta, float *m, float *v, const float *grad,
                        int64_t count, int32_t step, float lr, float beta1, float beta2, float eps) {
    if (!ctx) return APX_EINVAL;
    if (!theta || !m || !v || !grad) return set_err(ctx, APX_EINVAL, "null argument");
    if (count < 0 || step < 1) return set_err(ctx, APX_EINVAL, "need count >= 0 and step >= 1");
    if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps > 0.0f))
        return set_err(ctx, APX_EINVAL, "need 0 <= beta < 1 and eps > 0");
    if (count == 0) return APX_OK;
    DevGuard g(ctx->device);
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    k_adam<<<(unsigned)((count + 255) / 256), 256, 0, ctx->stream>>>(theta, m, v, grad, count, lr, beta1,
                                                                    beta2, eps, c1, c2);
    HIP_TRY(hipGetLastError(), "adam");
    return APX_OK;
}

apx_status apx_targets(apx_ctx *ctx, const float *R, int64_t n, int64_t ld, const float *sigma, float *Y) {
    if (!ctx) return APX_EINVAL;
    if (n < 1) return set_err(ctx, APX_EINVAL, "n must be >= 1");
    APX_TRY(check_sq(ctx, R, "R", n, ld));
    if (!sigma || !Y) return set_err(ctx, APX_EINVAL, "null argument");
    DevGuard g(ctx->device);
    k_targets<<<(unsigned)((n + 63) / 64), 1024, 0, ctx->stream>>>(R, ld, (int32_t)n, sigma, Y);
    HIP_TRY(hipGetLastError(), "targets");
    return APX_OK;
}

apx_status apx_warm_a0(apx_ctx *ctx, const float *Y, const float *sigma, int64_t n, float *A, int64_t ld) {
    if (!ctx) return APX_EINVAL;
    if (n < 1) return set_err(ctx, APX_EINVAL, "n must be >= 1");
    APX_TRY(check_sq(ctx, A, "A", n, ld));
    if (!sigma || !Y) return set_err(ctx, APX_EINVAL, "null argument");
    DevGuard g(ctx->device);
    k_warm_a0<<<grid_rows(n, ctx->num_cus * 4), 256, 0, ctx->stream>>>(Y, sigma, (int32_t)n, A, ld);
    HIP_TRY(hipGetLastError(), "A_0");
    return APX_OK;
}

apx_status ap_warmstart(apx_ctx *ctx, const float *S, int64_t n, int64_t ld, const float *theta,
                        float *R, float *A, float *sigma) {
    if (!ctx) return APX_EINVAL;
    if (n < 2) return set_err(ctx, APX_EINVAL, "ap_warmstart needs n >= 2");
    if (n > 65536) return set_err(ctx, APX_ENOTIMPL, "n = %lld exceeds 65536", (long long)n);
    APX_TRY(check_sq(ctx, S, "S", n, ld));
    APX_TRY(check_sq(ctx, R, "R", n, ld));
    APX_TRY(check_sq(ctx, A, "A", n, ld));
    if (!theta) return set_err(ctx, APX_EINVAL, "theta is null");
    DevGuard g(ctx->device);
    const WarmLayout WL = warm_layout(n);
    const size_t o_st = WL.o_st, o_f = WL.o_f, o_y = WL.o_y, o_s = WL.o_s;
    const size_t base = ctx->ws_base;
    APX_TRY(ws_reserve(ctx, base + WL.head));
    char *b = static_cast<char *>(ctx->ws) + base;
    RowStats *stats = reinterpret_cast<RowStats *>(b + o_st);
    float *F = reinterpret_cast<float *>(b + o_f);
    float *Yp = reinterpret_cast<float *>(b + o_y);
    float *sg = sigma ? sigma : reinterpret_cast<float *>(b + o_s);
    APX_TRY(run_features(ctx, S, n, ld, stats, F, sg));
    FwdArgs fa{};
    fa.theta = theta;
    fa.F = F;
    fa.count = n;
    fa.Y = Yp;
    APX_TRY(run_forward(ctx, fa));
    // A_0, and R_0 = one undamped responsibility step (Eq. (2)) from it
    hipStream_t s = ctx->stream;
    const int64_t q = (n + 3) / 4;
    const int cus = ctx->num_cus;
    if (q <= 256) launch_warm_start<256, 1>(S, Yp, sg, n, ld, A, R, cus, s);
    else if (q <= 512) launch_warm_start<256, 2>(S, Yp, sg, n, ld, A, R, cus, s);
    else if (q <= 1024) launch_warm_start<256, 4>(S, Yp, sg, n, ld, A, R, cus, s);
    else if (q <= 2048) launch_warm_start<1024, 2>(S, Yp, sg, n, ld, A, R, cus, s);
    else if (q <= 4096) launch_warm_start<1024, 4>(S, Yp, sg, n, ld, A, R, cus, s);
    else if (q <= 8192) launch_warm_start<1024, 8>(S, Yp, sg, n, ld, A, R, cus, s);
    else launch_warm_start<1024, 16>(S, Yp, sg, n, ld, A, R, cus, s);
    HIP_TRY(hipGetLastError(), "starting messages");
    return APX_OK;
}

}  // extern "C"
