// similarity.hip -- S from points, preferences and tie-break noise.
//
//   s(i,k) = -||x_i - x_k||^2 = 2<x_i,x_k> - (||x_i||^2 + ||x_k||^2)   (Section 2)
//
// The Gram part runs on FP32 matrix cores (v_mfma_f32_32x32x2f32, FP32
// accumulate).  Only tiles on or above the block diagonal are computed; each
// result is written at (i,k) and mirrored to (k,i) from the accumulators,
// so S is exactly symmetric.  The preference is the median of the n(n-1) off-diagonal
// entries, found exactly without reading S again: a sample of pairs gives a
// narrow window of values that holds the median, the tiles count the upper
// entries below it and set aside those inside it, and the few set aside are
// ranked.  (The upper triangle holds every off-diagonal value twice by
// symmetry.)  Should the window miss, or too many values fall into it, a
// three-pass radix select over the stored upper triangle finds it instead.
#include <cmath>
#include <type_traits>

#include "apx_internal.h"

namespace apx {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int BM = 128;      // tile edge
// K chunk staged in LDS.  16 rather than 32 halves the registers that
// carry the next chunk's loads, so three workgroups fit a CU instead of two
// (168 registers instead of 192): the writes of S of one workgroup overlap
// the MFMAs of two others.  The MFMA sequence (two K values per step, in
// ascending order) is the same for any chunk size, so S is unchanged.
constexpr int KB = 16;
constexpr int NT = 256;      // threads per tile (4 wavefronts)
constexpr int SEL_BINS = 8192;   // bins per rank in the global select histogram (13-bit first digit)

// Ordered 32-bit key of a float: unsigned order equals float order.
__device__ __forceinline__ uint32_t fkey(float f) {
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float keyf(uint32_t k) {
    uint32_t b = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(b);
}

// Squared norms, summed in column order; bad (nullable): set where X holds a
// NaN or an infinity.  64 rows per workgroup go through LDS 64 columns at a
// time, so that the loads are coalesced (5003 x 62: 7.5 us against 14 with one
// thread reading along a row).
__global__ __launch_bounds__(256) void k_sqnorm(const float *X, int64_t n, int64_t d, int64_t ldx, float *nrm,
                                                int32_t *bad) {
    __shared__ float sh[64][65];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    float acc = 0.0f;
    uint32_t nonfinite = 0u;
    for (int64_t c0 = 0; c0 < d; c0 += 64) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = tid + 256 * u, r = e >> 6, c = e & 63;
            const float x = r0 + r < n && c0 + c < d ? X[(r0 + r) * ldx + c0 + c] : 0.0f;
            nonfinite |= (uint32_t)((__float_as_uint(x) & 0x7f800000u) == 0x7f800000u);
            sh[r][c] = x;
        }
        __syncthreads();
        if (tid < 64) {
            const int w = d - c0 < 64 ? (int)(d - c0) : 64;
            for (int c = 0; c < w; ++c) acc = fmaf(sh[tid][c], sh[tid][c], acc);
        }
    }
    if (tid < 64 && r0 + tid < n) nrm[r0 + tid] = acc;
    if (bad != nullptr && __any(nonfinite) && (tid & 63) == 0) atomicOr(bad, 1);
}

// ---- the median's window ---------------------------------------------------
// At n = 20000 (2e8 upper entries) about 1.7% of the keys are set aside; the
// sample takes 21 us, counting and ranking them 33 us, and the walk in the
// tiles' epilogue 110 us (GEMM 0.48 -> 0.595 ms), in place of two passes over S
// (204 and 216 us) and a digit counted in the epilogue (40): the whole build
// 991 -> 661 us.
constexpr int kSegs = 64;          // lists of set-aside keys (tile t appends to list t mod kSegs)
constexpr int kWinBins = 4096;     // intervals the window is cut into
constexpr int kWinList = 16384;    // keys of the intervals that hold the two ranks
constexpr int kSamples = 65536;    // sampled pairs ...
constexpr int kSampleTail = 512;   // ... the window spans the sample's median rank +- 4 sigma (sqrt(65536) / 2
                                   // each): it misses once in 16000 calls
// Up to here every key is set aside and the window is the range of S (no
// sample: 300 points 78 us instead of 91).
constexpr int64_t kWholeN = 512;
// Samples an interval that holds an end of the window may have (0.4% of them
// on either side: the lists hold twice what the window makes expected).
constexpr uint32_t kEdgeMany = 256;
constexpr uint32_t kNoBin = 0xffffffffu;   // SelWin::bin of a rank whose key is known
// Keys up to which the last workgroup of the ranking cuts crowded intervals
// again by itself (300 points of two clusters: 132 us, 162 with the select over
// S).  Above, the host starts another count and ranking of the lists (20000
// points of two far clusters, whose median lies at an edge of the gap: 2.36 ms
// with the noise, 3.35 with the select).
constexpr uint32_t kRecut = 1u << 18;
constexpr int32_t kCutAgain = 2;
// How k_win_count and k_win_rank cut the keys set aside: the sample's window,
// the bounds of S, or the crowded interval of a cut before.
enum { CUT_WINDOW, CUT_WHOLE, CUT_AGAIN };

struct SelSeg {                    // one 128-byte line per list
    uint32_t count, pad;
    unsigned long long below;      // keys below the window
    unsigned long long at[2];      // ties: keys equal to its lower and its upper end
    uint32_t fill[24];
};
struct SelWin {
    float vlo, vhi;                // the window, both inclusive; neither is a zero, so values
                                   // compare as their keys do
    uint32_t lo;                   // key of vlo (a repeated cut: least key of the interval cut again)
    uint32_t shift;                // interval of a key: (key - lo) >> shift < kWinBins
    uint32_t hi;                   // repeated cut: largest key of the interval
    int32_t miss;                  // 1: the median was not found this way; kCutAgain: its interval is too
                                   // crowded to be ranked
    // Similarities crowd near an end, which is then a value that many entries
    // may share: entries equal to an end are counted, not set aside (an end may
    // be +0 here; S holds no -0: the Gram sum starts from +0 and x - x is +0).
    int32_t ties;
    uint32_t bin[2];               // intervals of the two ranks ...
    uint32_t rank[2];              // ... and the ranks inside them
    uint32_t kmin[2], kmax[2];     // bounds of the keys in the two intervals
    uint32_t done[3], nlist;
};
// Set-aside keys a list holds: all of its tiles' where everything is set
// aside, else twice what the window's share of the sample makes expected,
// and one full tile.
int64_t seg_cap(int64_t n) {
    const int64_t t = (n + BM - 1) / BM, tiles = t * (t + 1) / 2;
    const int64_t per = (tiles + kSegs - 1) / kSegs * (BM * BM);
    if (n <= kWholeN) return per;
    const int64_t want = (int64_t)((double)n * (double)n / kSegs * 2.2 * kSampleTail / kSamples) + BM * BM;
    return want < per ? want : per;
}

struct SimArgs {
    const float *X;
    int64_t n, d, ldx;
    const float *nrm;
    float *S;
    int64_t ld;
    int64_t tiles_per_side;
    uint32_t *minmax;     // [0] = min key, [1] = max key of off-diagonal entries
    // median preference (else null): the window, the lists of keys set aside
    const SelWin *win;
    SelSeg *segs;
    uint32_t *cand;       // kSegs lists of cap keys
    uint32_t cap;
    const int32_t *bad;   // nonzero: the input failed the finite check, write nothing
};

// One 128 x 128 tile per workgroup.  X rows are staged through LDS one K
// chunk at a time, the next chunk's global loads in flight during the
// current chunk's MFMAs; the epilogue writes S straight from the
// accumulators (no LDS tile): lane l of
// block (x, y) holds column c = l mod 32 and rows 8g + 4(l / 32) + q
// (g, q = 0..3), written directly (one float per row, 128-byte row
// segments per half wavefront) and mirrored (the four rows q are
// consecutive columns of S's row c: one float4).  With the median
// preference (COUNT) the epilogue also counts the upper entries below the
// window and sets aside the keys inside it: every wavefront collects its own
// in LDS and appends them to the tile's list.
constexpr int LDA = BM + 1;   // padded LDS rows: conflict-free transposed stores

// Gram block <x_i, x_k> of rows row0.. and columns col0.. (BM each) into the
// accumulators: wavefront (wm, wn) holds the 2 x 2 32x32 blocks at rows
// wm*64 + 32x, columns wn*64 + 32y.  Every entry sums its products in the
// same order (K chunks of KB, two per MFMA), whichever tile it lies in and
// whichever of x_i, x_k is the A operand, so an entry has one value.
__device__ __forceinline__ void gram_tile(const float *X, int64_t n, int64_t d, int64_t ldx, int64_t row0,
                                          int64_t col0, v16f (&acc)[2][2], float *As, float *Bs) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[x][y][v] = 0.0f;

    // X[row0 .. +BM, k0 .. +KB] and X[col0 .. +BM, k0 .. +KB] into registers
    constexpr int SU = BM * KB / NT;
    float va[SU], vb[SU];
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int e = tid + u * NT;
            const int m = e / KB, kk = e % KB;
            const int64_t kg = k0 + kk;
            const int64_t ra = row0 + m, rb = col0 + m;
            va[u] = (ra < n && kg < d) ? X[ra * ldx + kg] : 0.0f;
            vb[u] = (rb < n && kg < d) ? X[rb * ldx + kg] : 0.0f;
        }
    };
    fetch(0);
    for (int64_t k0 = 0; k0 < d; k0 += KB) {
        // staged k-major; the previous chunk's MFMAs are done (barrier below)
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int e = tid + u * NT;
            const int m = e / KB, kk = e % KB;
            As[kk * LDA + m] = va[u];
            Bs[kk * LDA + m] = vb[u];
        }
        __syncthreads();
        if (k0 + KB < d) fetch(k0 + KB);
#pragma unroll
        for (int kk = 0; kk < KB; kk += 2) {
            const int kr = kk + (lane >> 5);
            float av[2], bv[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) av[x] = As[kr * LDA + wm * 64 + x * 32 + (lane & 31)];
#pragma unroll
            for (int y = 0; y < 2; ++y) bv[y] = Bs[kr * LDA + wn * 64 + y * 32 + (lane & 31)];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[x], bv[y], acc[x][y], 0, 0, 0);
        }
        __syncthreads();
    }
}

template <bool COUNT>
__global__ __launch_bounds__(NT, 3) void k_sim_gemm(SimArgs a) {
    if (*a.bad) return;
    // Decode the upper-triangle tile (bi <= bj) from the linear block index.
    const int64_t T = a.tiles_per_side;
    int64_t t = blockIdx.x, bi = 0;
    while (t >= T - bi) {
        t -= T - bi;
        ++bi;
    }
    const int64_t bj = bi + t;
    const int64_t row0 = bi * BM, col0 = bj * BM;

    __shared__ float As[KB * LDA], Bs[KB * LDA];    // 16.5 KB of staging
    __shared__ float nr[BM], nc[BM];                // squared norms of the tile's rows and columns
    constexpr int kHold = 1024;                     // keys a wavefront holds before it appends them
    __shared__ uint32_t held[COUNT ? NT / 64 : 1][COUNT ? kHold : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    for (int e = tid; e < BM; e += NT) {
        nr[e] = row0 + e < a.n ? a.nrm[row0 + e] : 0.0f;
        nc[e] = col0 + e < a.n ? a.nrm[col0 + e] : 0.0f;
    }
    float wlo = 0.0f, whi = 0.0f;
    int wties = 0;
    uint32_t below = 0u, at_lo = 0u, at_hi = 0u;
    int nheld = 0;
    SelSeg *const seg = COUNT ? a.segs + blockIdx.x % kSegs : nullptr;
    uint32_t *const list = COUNT ? a.cand + (int64_t)(blockIdx.x % kSegs) * a.cap : nullptr;
    if constexpr (COUNT) {
        wlo = a.win->vlo;
        whi = a.win->vhi;
        wties = a.win->ties;
    }
    auto append = [&]() {
        uint32_t at = 0u;
        if (lane == 0) at = atomicAdd(&seg->count, (uint32_t)nheld);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int e = lane; e < nheld; e += 64)
            if (at + e < a.cap) list[at + e] = held[wave][e];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        nheld = 0;
    };
    v16f acc[2][2];
    gram_tile(a.X, a.n, a.d, a.ldx, row0, col0, acc, As, Bs);

    uint32_t kmin = 0xffffffffu, kmax = 0u;
    const bool diag_tile = (bi == bj);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int c = wn * 64 + y * 32 + (lane & 31);   // tile column
            const int64_t k = col0 + c;
            const float ncc = nc[c];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int mb = wm * 64 + x * 32 + 8 * g + 4 * (lane >> 5);   // first of four rows
                const int64_t ib = row0 + mb;
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = 2.0f * acc[x][y][4 * g + q] - (nr[mb + q] + ncc);
                if (k >= a.n) continue;
                if (!diag_tile) {
                    // every (i, k) here has i < k: direct, mirror, bounds
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (ib + q < a.n) {
                            a.S[(ib + q) * a.ld + k] = v[q];
                            const uint32_t key = fkey(v[q]);
                            kmin = min(kmin, key);
                            kmax = max(kmax, key);
                        }
                    }
                    float *dst = a.S + k * a.ld + ib;
                    if (ib + 3 < a.n) {
                        *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (ib + q < a.n) dst[q] = v[q];
                    }
                } else {
                    // diagonal tile: the upper entries (m < c) are written at
                    // (m, c) and (c, m), so S is symmetric; the diagonal gets
                    // a value that the preference pass overwrites
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int m = mb + q;
                        if (ib + q >= a.n || m > c) continue;
                        a.S[(ib + q) * a.ld + k] = v[q];
                        if (m < c) {
                            a.S[k * a.ld + ib + q] = v[q];
                            const uint32_t key = fkey(v[q]);
                            kmin = min(kmin, key);
                            kmax = max(kmax, key);
                        }
                    }
                }
            }
        }
    // The window: upper entries below it counted, those inside set aside.  A
    // walk of its own (the values are formed again, two operations each), so
    // that all lanes take part; tiles above the diagonal and inside S need no
    // test of the indices.
    if constexpr (COUNT) {
        // with ties: entries equal to an end are counted apart (both ends one
        // value: in at_lo; no value lies between then)
        const float one = wlo == whi ? __builtin_nanf("") : whi;
        auto walk = [&](auto every, auto ties) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const int c = wn * 64 + y * 32 + (lane & 31);
                    const float ncc = nc[c];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int mb = wm * 64 + x * 32 + 8 * g + 4 * (lane >> 5);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float v = 2.0f * acc[x][y][4 * g + q] - (nr[mb + q] + ncc);
                            bool up = true;
                            if constexpr (!decltype(every)::value)
                                up = col0 + c < a.n && row0 + mb + q < a.n && (!diag_tile || mb + q < c);
                            below += __popcll(__ballot(up && v < wlo));
                            unsigned long long m;
                            if constexpr (decltype(ties)::value) {
                                at_lo += __popcll(__ballot(up && v == wlo));
                                at_hi += __popcll(__ballot(up && v == one));
                                m = __ballot(up && v > wlo && v < one);
                            } else {
                                m = __ballot(up && v >= wlo && v <= whi);
                            }
                            if (m == 0ull) continue;
                            if ((m >> lane) & 1ull) held[wave][nheld + __popcll(m & ((1ull << lane) - 1ull))] = fkey(v);
                            nheld += __popcll(m);
                        }
                        if (nheld > kHold - 256) append();   // (four more entries fill at most 256)
                    }
                }
        };
        if (wties) {
            walk(std::false_type{}, std::true_type{});
            if (lane == 0 && at_lo) atomicAdd(&seg->at[0], (unsigned long long)at_lo);
            if (lane == 0 && at_hi) atomicAdd(&seg->at[1], (unsigned long long)at_hi);
        } else if (!diag_tile && row0 + BM <= a.n && col0 + BM <= a.n) {
            walk(std::true_type{}, std::false_type{});
        } else {
            walk(std::false_type{}, std::false_type{});
        }
        if (nheld) append();
        if (lane == 0 && below) atomicAdd(&seg->below, (unsigned long long)below);
    }
    // Block min/max of the upper off-diagonal entries: wavefronts, then the
    // tile, then one atomic per bound, skipped when it cannot change the value
    // (all tiles update the same two words).
    for (int off = 32; off >= 1; off >>= 1) {
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off, 64));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off, 64));
    }
    __shared__ uint32_t red[2][NT / 64];
    if (lane == 0) {
        red[0][wave] = kmin;
        red[1][wave] = kmax;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) {
            kmin = min(kmin, red[0][w]);
            kmax = max(kmax, red[1][w]);
        }
        if (kmin < __atomic_load_n(&a.minmax[0], __ATOMIC_RELAXED)) atomicMin(&a.minmax[0], kmin);
        if (kmax > __atomic_load_n(&a.minmax[1], __ATOMIC_RELAXED)) atomicMax(&a.minmax[1], kmax);
    }
}

// ---- exact order statistics of the upper triangle -------------------------
// sel[0..1]: state of the two ranks (lo, hi): prefix key bits so far.
struct SelState {
    uint32_t prefix[2];
    uint32_t pad0[2];
    unsigned long long rank[2];   // remaining rank inside the current prefix
};

// Digits of the 32-bit key: 13 bits (the first pass, when both ranks share
// the empty prefix and one histogram counts for both: more bins spread the
// counter contention of keys that share their exponent), then 10 and 9.
__device__ __forceinline__ void sel_digit(int pass, int &shift, int &bits, uint32_t &hmask) {
    shift = pass == 0 ? 19 : (pass == 1 ? 9 : 0);
    bits = pass == 0 ? 13 : (pass == 1 ? 10 : 9);
    hmask = pass == 0 ? 0u : (pass == 1 ? 0xfff80000u : 0xfffffe00u);
}

// Start of the select; of the window (win nullable: everything set aside
// until a sample narrows it), of the finite-check flag (nullable).
__global__ void k_sel_init(SelState *st, uint32_t *minmax, unsigned long long lo, unsigned long long hi,
                           unsigned long long *hist, SelWin *win, SelSeg *segs, uint32_t *whist, int32_t *bad) {
    if (win != nullptr) {
        if (threadIdx.x == 0) {
            SelWin w{};
            w.vlo = -INFINITY;
            w.vhi = INFINITY;
            w.kmin[0] = w.kmin[1] = 0xffffffffu;
            *win = w;
        }
        uint32_t *sw = reinterpret_cast<uint32_t *>(segs);
        for (int b = threadIdx.x; b < (int)(kSegs * sizeof(SelSeg) / 4); b += blockDim.x) sw[b] = 0u;
        for (int b = threadIdx.x; b < kWinBins; b += blockDim.x) whist[b] = 0u;
    }
    if (bad != nullptr && threadIdx.x == 0) *bad = 0;
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        st->prefix[0] = st->prefix[1] = 0u;
        st->rank[0] = lo;
        st->rank[1] = hi;
        minmax[0] = 0xffffffffu;
        minmax[1] = 0u;
    }
    for (int b = threadIdx.x; b < 2 * SEL_BINS; b += blockDim.x) hist[b] = 0ull;
}

// Histogram of the keys of upper-triangle entries whose high bits match the
// current prefix of each rank.  shift/bits select the digit of this pass.
// f(k, v) for the entries v = row[k], k = i+1 .. n-1, of row i: the unaligned
// head one by one, then 16-byte pieces (rows start 16-byte aligned: ld is a
// multiple of 4), U per thread in flight in every step, the row's ragged end
// included (its last piece read element by element, nothing at or beyond n).
typedef float sv4 __attribute__((ext_vector_type(4)));
template <int U, class F>
__device__ __forceinline__ void upper_row(const float *row, int64_t i, int64_t n, F &&f) {
    const int64_t k4 = (i + 4) & ~int64_t(3);          // first multiple of 4 above i
    const int64_t kh = k4 < n ? k4 : n;
    if (i + 1 + threadIdx.x < kh) f(i + 1 + threadIdx.x, row[i + 1 + threadIdx.x]);
    const int64_t st = 4 * (int64_t)blockDim.x;
    for (int64_t kb = k4 + 4 * (int64_t)threadIdx.x; kb < n; kb += U * st) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = kb + u * st;
            if (k + 3 < n) {
                // read once per pass: nontemporal
                const sv4 w = __builtin_nontemporal_load(reinterpret_cast<const sv4 *>(row + k));
                v[u] = make_float4(w.x, w.y, w.z, w.w);
            } else {
                v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (k < n) v[u].x = row[k];
                if (k + 1 < n) v[u].y = row[k + 1];
                if (k + 2 < n) v[u].z = row[k + 2];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = kb + u * st;
            if (k < n) f(k, v[u].x);
            if (k + 1 < n) f(k + 1, v[u].y);
            if (k + 2 < n) f(k + 2, v[u].z);
            if (k + 3 < n) f(k + 3, v[u].w);
        }
    }
}

// Workgroups of a row-walking pass: as many as are resident on the chip
// at once (workgroup b walks rows b, b + grid, ...: a second, partial round
// would leave most CUs idle while it finishes), at most one per row.
int walk_grid(const void *kern, size_t lds, int64_t rows) {
    int dev = 0, cus = 0, occ = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 256, lds) != hipSuccess || occ < 1) occ = 1;
    const int64_t g = (int64_t)occ * cus;
    return (int)(rows < g ? rows : g);
}

// Rows [r0, r1) of S (row i at S + i * ld).
__global__ __launch_bounds__(256) void k_sel_hist(const float *S, int64_t n, int64_t ld,
                                                  const SelState *st, int pass,
                                                  unsigned long long *hist, int64_t r0, int64_t r1) {
    // dynamic LDS: one histogram of nb bins on the first pass (both ranks
    // start from the same empty prefix), two on the others
    extern __shared__ uint32_t hsh[];
    int shift, bits;
    uint32_t hmask;
    sel_digit(pass, shift, bits, hmask);
    const uint32_t nb = 1u << bits;
    const uint32_t nh = pass == 0 ? 1u : 2u;
    for (uint32_t b = threadIdx.x; b < nh * nb; b += blockDim.x) hsh[b] = 0u;
    __syncthreads();
    const uint32_t p0 = st->prefix[0], p1 = st->prefix[1];
    // both ranks inside one prefix (always on the first pass): one count
    // serves both histograms
    const bool same = p0 == p1;
    uint32_t *const h0 = hsh;
    uint32_t *const h1 = hsh + (nh - 1) * nb;
    auto count = [&](int64_t, float v) {
        const uint32_t key = fkey(v);
        const uint32_t dig = (key >> shift) & (nb - 1u);
        if ((key & hmask) == p0) atomicAdd(&h0[dig], 1u);
        if (!same && (key & hmask) == p1) atomicAdd(&h1[dig], 1u);
    };
    const int64_t re = r1 < n - 1 ? r1 : n - 1;
    for (int64_t i = r0 + blockIdx.x; i < re; i += gridDim.x) upper_row<8>(S + i * ld, i, n, count);
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) {
        const uint32_t c0 = h0[b], c1 = same ? c0 : h1[b];
        if (c0) atomicAdd(&hist[b], (unsigned long long)c0);
        if (c1) atomicAdd(&hist[SEL_BINS + b], (unsigned long long)c1);
    }
}

// Inclusive prefix sum over the 256 threads: wavefront shuffles, then the
// wavefront totals through LDS (ws: 4 entries).
__device__ __forceinline__ unsigned long long block_scan256(unsigned long long x, unsigned long long *ws) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) ws[w] = x;
    __syncthreads();
    unsigned long long add = 0ull;
    for (int k = 0; k < w; ++k) add += ws[k];
    __syncthreads();
    return x + add;
}

// Pick the digit holding each rank; extend the prefixes; clear the histogram.
// 256 threads: each sums nb/256 consecutive digits, a block scan of the
// sums finds the segment holding the rank, its owner walks its digits
// (held in registers since the sum).
__global__ __launch_bounds__(256) void k_sel_pick(SelState *st, int pass, unsigned long long *hist) {
    int shift, bits;
    uint32_t hmask;
    sel_digit(pass, shift, bits, hmask);
    const uint32_t nb = 1u << bits;
    const uint32_t per = nb / 256;               // digits per thread (32, 4 or 2)
    constexpr int MAXPER = SEL_BINS / 256;
    __shared__ unsigned long long ws[4];
    const int t = threadIdx.x;
    for (int r = 0; r < 2; ++r) {
        const unsigned long long *hr = hist + r * SEL_BINS;
        // the thread's segment of digits, all loads in flight at once
        unsigned long long v[MAXPER];
#pragma unroll
        for (int q = 0; q < MAXPER; ++q) v[q] = (uint32_t)q < per ? hr[t * per + q] : 0ull;
        unsigned long long own = 0ull;
#pragma unroll
        for (int q = 0; q < MAXPER; ++q) own += v[q];
        // read before the scan's barriers: the owner rewrites it below
        const unsigned long long rank = st->rank[r];
        const unsigned long long incl = block_scan256(own, ws);
        const unsigned long long before = incl - own;   // digits below this thread's segment
        if (rank >= before && rank < incl) {
            unsigned long long cum = before;
            uint32_t b = t * per;
            bool found = false;
#pragma unroll
            for (int q = 0; q < MAXPER; ++q) {
                if (!found && (uint32_t)q < per) {
                    if (rank < cum + v[q]) {
                        found = true;
                        b = t * per + q;
                    } else {
                        cum += v[q];
                    }
                }
            }
            st->rank[r] = rank - cum;
            st->prefix[r] |= (b << shift);
        }
        __syncthreads();
    }
    for (int b = t; b < 2 * SEL_BINS; b += blockDim.x) hist[b] = 0ull;
}

// True in every thread of the last workgroup of the grid to come here; the
// others' device-scope stores are then visible to device-scope loads.
__device__ __forceinline__ bool last_block(uint32_t *done) {
    __shared__ int last;
    // the workgroup's device-scope stores and atomics have arrived (no cache
    // holds them back, so nothing is flushed)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(done, 1u) == gridDim.x - 1u;
    __syncthreads();
    return last != 0;
}
__device__ __forceinline__ uint32_t ld_dev(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The keys of ranks r0 and r1 (ascending) among the workgroup's, which lie
// between least and most (others: 0xffffffff, above both ranks), bit by bit
// from the highest in which they differ: count the keys below.  under: a pair
// of zeros for each bit.
template <int N>
__device__ __forceinline__ void two_ranks(const uint32_t (&key)[N], int r0, int r1, uint32_t least, uint32_t most,
                                          uint32_t (*under)[2], uint32_t &e0, uint32_t &e1) {
    const int bits = least == most ? 0 : 32 - __builtin_clz(least ^ most);
    e0 = e1 = bits < 32 ? least >> bits << bits : 0u;
    for (int bit = bits - 1; bit >= 0; --bit) {
        const uint32_t t0 = e0 | 1u << bit, t1 = e1 | 1u << bit;
        uint32_t n0 = 0u, n1 = 0u;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            n0 += __popcll(__ballot(key[e] < t0));
            n1 += __popcll(__ballot(key[e] < t1));
        }
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&under[bit][0], n0);
            atomicAdd(&under[bit][1], n1);
        }
        __syncthreads();
        if (r0 >= (int)under[bit][0]) e0 = t0;
        if (r1 >= (int)under[bit][1]) e1 = t1;
    }
}

// Similarities of kSamples pseudo-random pairs (16 lanes to a pair), then, in
// the last workgroup, the window: the values of the sample's ranks at kSampleTail
// either side of the middle, widened to the intervals (of kWinBins over the
// sample's range) that hold them.  Where an interval has many samples (a far
// point or cluster stretches the range, ties) the ends are values of samples
// at those ranks.  The window only has to hold the median; nothing
// else depends on it.
constexpr int SMP_T = 1024, SMP_BLOCKS = 128;
__global__ __launch_bounds__(SMP_T) void k_sel_sample(const float *X, int64_t n, int64_t d, int64_t ldx,
                                                      const float *nrm, uint32_t *smp, SelWin *win,
                                                      const int32_t *bad) {
    if (*bad) return;
    __shared__ uint32_t hist[kWinBins];
    __shared__ float red[2][SMP_T / 64];
    __shared__ uint32_t wtot[SMP_T / 64];
    __shared__ int edge[2];
    __shared__ uint32_t held[4], under[2][32][2];   // samples in the ends' intervals; below a key, by its bit
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // four pairs at a time per 16 lanes
    constexpr int PER = kSamples / SMP_BLOCKS / (SMP_T / 16);
    static_assert(PER % 4 == 0, "pairs per group");
    for (int it = 0; it < PER; it += 4) {
        const float *xi[4], *xk[4];
        float nn[4], acc[4];
        int p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            p[u] = (blockIdx.x * PER + it + u) * (SMP_T / 16) + (tid >> 4);
            uint64_t z = (uint64_t)(p[u] + 1) * 0x9E3779B97F4A7C15ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            const int64_t i = (int64_t)(((z & 0xffffffffull) * (uint64_t)n) >> 32);
            int64_t k = (int64_t)(((z >> 32) * (uint64_t)(n - 1)) >> 32);
            k += k >= i;
            xi[u] = X + i * ldx;
            xk[u] = X + k * ldx;
            nn[u] = nrm[i] + nrm[k];
            acc[u] = 0.0f;
        }
        for (int64_t j = tid & 15; j < d; j += 16)
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u] = fmaf(xi[u][j], xk[u][j], acc[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) acc[u] += __shfl_xor(acc[u], off, 64);
            if ((tid & 15) == 0) st_dev(&smp[p[u]], __float_as_uint(2.0f * acc[u] - nn[u]));
        }
    }
    if (!last_block(&win->done[0])) return;
    constexpr int E = kSamples / SMP_T;
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = __uint_as_float(ld_dev(&smp[tid + e * SMP_T]));
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        lo = fminf(lo, v[e]);
        hi = fmaxf(hi, v[e]);
    }
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off, 64));
        hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
        red[0][wave] = lo;
        red[1][wave] = hi;
    }
    for (int b = tid; b < kWinBins; b += SMP_T) hist[b] = 0u;
    __syncthreads();
    for (int w = 0; w < SMP_T / 64; ++w) {
        lo = fminf(lo, red[0][w]);
        hi = fmaxf(hi, red[1][w]);
    }
    const float inv = (float)(kWinBins - 1) / (hi - lo);
    auto bin_of = [&](float x) {
        const int b = (int)((x - lo) * inv);
        return b < 0 ? 0 : b > kWinBins - 1 ? kWinBins - 1 : b;
    };
    // (an eighth first: where a quarter of it lies in one interval, the others
    // would only wait for that counter)
#pragma unroll
    for (int e = 0; e < E / 8; ++e) atomicAdd(&hist[bin_of(v[e])], 1u);
    if (tid < 128) (&under[0][0][0])[tid] = 0u;
    __syncthreads();
    bool crowded = __syncthreads_or(hist[bin_of(v[0])] > kSamples / 8 / 4);
    if (!crowded) {
#pragma unroll
        for (int e = E / 8; e < E; ++e) atomicAdd(&hist[bin_of(v[e])], 1u);
        __syncthreads();
        const uint4 h = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
        const uint32_t c[4] = {h.x, h.y, h.z, h.w}, tot = h.x + h.y + h.z + h.w;
        uint32_t inc = tot;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (lane == 63) wtot[wave] = inc;
        __syncthreads();
        uint32_t before = inc - tot;
        for (int w = 0; w < wave; ++w) before += wtot[w];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t r = kSamples / 2 + (q ? kSampleTail : -kSampleTail);
            if (r >= before && r < before + tot) {
                uint32_t acc = before;
                int e = 0;
                while (e < 3 && r >= acc + c[e]) acc += c[e++];
                edge[q] = 4 * tid + e;
                held[q] = c[e];
            }
        }
        __syncthreads();
        crowded = held[0] > kEdgeMany || held[1] > kEdgeMany;
        __syncthreads();                      // (held is used again below)
    }
    uint32_t end[2] = {0u, 0u};
    if (crowded) {
        // An eighth of the samples gives a window four of its deviations wide
        // (4.4% of the similarities), the samples inside it the two ranks.
        constexpr int N = E / 8, TAIL = kSampleTail * 46 / 128;    // (sqrt(8) = 2.83, 46 / 128 = 1 / 2.78)
        uint32_t key[N];
#pragma unroll
        for (int e = 0; e < N; ++e) key[e] = fkey(v[e]);
        uint32_t from, to;
        two_ranks<N>(key, kSamples / 16 - TAIL, kSamples / 16 + TAIL, fkey(lo), fkey(hi), under[0], from, to);
        if (tid < 4) held[tid] = 0u;
        __syncthreads();
        uint32_t below = 0u, at_from = 0u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t k = fkey(v[e]);
            below += __popcll(__ballot(k < from));
            at_from += __popcll(__ballot(k == from));
            const unsigned long long m = __ballot(k > from && k < to);
            if (m == 0ull) continue;
            uint32_t at = 0u;
            if (lane == 0) at = atomicAdd(&held[2], (uint32_t)__popcll(m));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + __popcll(m & ((1ull << lane) - 1ull));
            if ((m >> lane & 1ull) && at < (uint32_t)kWinBins) hist[at] = k;
        }
        if (lane == 0) {
            atomicAdd(&held[0], below);
            atomicAdd(&held[1], at_from);
        }
        __syncthreads();
        const uint32_t inside = held[2];
        constexpr int NI = kWinBins / SMP_T;
        uint32_t in[NI];
#pragma unroll
        for (int e = 0; e < NI; ++e) in[e] = tid + e * SMP_T < inside ? hist[tid + e * SMP_T] : 0xffffffffu;
        // ranks among the samples between the two ends; outside them the end itself
        const int base = (int)(held[0] + held[1]), r0 = kSamples / 2 - kSampleTail - base, r1 = r0 + 2 * kSampleTail;
        two_ranks<NI>(in, r0, r1, from, to, under[1], end[0], end[1]);
        if (inside > (uint32_t)kWinBins || r0 < 0) end[0] = from;
        if (inside > (uint32_t)kWinBins || r1 >= (int)inside) end[1] = to;
        if (r0 >= (int)inside) end[0] = to;
        if (r1 < 0) end[1] = from;
    }
    if (tid == 0) {
        const float w = (hi - lo) / (float)(kWinBins - 1);
        float a = lo + (float)edge[0] * w, b = lo + (float)(edge[1] + 1) * w;
        const int ties = crowded;
        if (ties) {
            a = keyf(end[0]) + 0.0f;
            b = keyf(end[1]) + 0.0f;
        }
        if (!ties && a == 0.0f) a = -1.0e-30f;
        if (!ties && b == 0.0f) b = 1.0e-30f;
        win->ties = ties;
        win->vlo = a;
        win->vhi = b;
        win->lo = fkey(a);
        const uint32_t span = fkey(b) - fkey(a);      // (b >= a)
        const int bits = span ? 32 - __builtin_clz(span) : 0;
        win->shift = bits > 12 ? bits - 12 : 0;
    }
}

// The first key and the interval width of the cut.
__device__ __forceinline__ void win_cut(const SelWin *win, const uint32_t *minmax, int cut, uint32_t &lo,
                                        uint32_t &shift) {
    lo = win->lo;
    shift = win->shift;
    if (cut == CUT_WHOLE) {
        lo = minmax[0];
        const uint32_t span = minmax[1] - lo;
        const int bits = span ? 32 - __builtin_clz(span) : 0;
        shift = bits > 12 ? bits - 12 : 0;
    }
}

// Counts the set-aside keys by interval; the last workgroup finds the
// intervals of the two ranks.
constexpr int RANK_T = 1024;      // one workgroup per list
__global__ __launch_bounds__(RANK_T) void k_win_count(SelState *st, SelWin *win, const SelSeg *segs,
                                                      const uint32_t *cand, uint32_t cap, uint32_t *whist,
                                                      const uint32_t *minmax, int cut, const int32_t *bad) {
    if (*bad) return;
    __shared__ uint32_t hist[kWinBins];
    __shared__ uint32_t wtot[RANK_T / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int b = tid; b < kWinBins; b += RANK_T) hist[b] = 0u;
    __syncthreads();
    const int sg = blockIdx.x;
    const uint32_t cnt = segs[sg].count < cap ? segs[sg].count : cap;
    const uint32_t *list = cand + (int64_t)sg * cap;
    uint32_t lo, shift;
    win_cut(win, minmax, cut, lo, shift);
    const uint32_t hi = cut == CUT_AGAIN ? win->hi : 0xffffffffu;
    for (uint32_t e = tid; e < cnt; e += 8 * RANK_T) {
        uint32_t key[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) key[u] = e + u * RANK_T < cnt ? list[e + u * RANK_T] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e + u * RANK_T < cnt && key[u] >= lo && key[u] <= hi) atomicAdd(&hist[(key[u] - lo) >> shift], 1u);
    }
    __syncthreads();
    for (int b = tid; b < kWinBins; b += RANK_T)
        if (hist[b]) atomicAdd(&whist[b], hist[b]);
    if (!last_block(&win->done[1])) return;
    // keys below the window and in it: lane s of every wavefront has list s
    static_assert(kSegs == 64, "a list per lane");
    unsigned long long below = segs[lane].below, total = segs[lane].count;
    unsigned long long at_lo = 0ull, at_hi = 0ull;
    if (cut != CUT_WHOLE && win->ties) {
        at_lo = segs[lane].at[0];
        at_hi = segs[lane].at[1];
        for (int off = 32; off >= 1; off >>= 1) {
            at_lo += __shfl_xor(at_lo, off, 64);
            at_hi += __shfl_xor(at_hi, off, 64);
        }
    }
    const bool over = __any(segs[lane].count > cap);
    for (int off = 32; off >= 1; off >>= 1) {
        below += __shfl_xor(below, off, 64);
        total += __shfl_xor(total, off, 64);
    }
    constexpr int PER = kWinBins / RANK_T;
    uint32_t c[PER], own = 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) c[q] = ld_dev(&whist[tid * PER + q]);
#pragma unroll
    for (int q = 0; q < PER; ++q) own += c[q];
    uint32_t incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wtot[w];
    const uint32_t before = incl - own;
    uint32_t in_bin[2] = {0u, 0u}, in_rank[2] = {0u, 0u};
    if (cut == CUT_AGAIN) {
        for (int r = 0; r < 2; ++r) {
            in_bin[r] = win->bin[r];
            in_rank[r] = win->rank[r];
        }
        __syncthreads();                     // (they are rewritten below)
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        // in ascending order: below the window, equal to its lower end, set
        // aside, equal to its upper end (the equal ones counted with ties only)
        unsigned long long rank = st->rank[r];
        if (cut == CUT_AGAIN) {
            if (in_bin[r] == kNoBin) continue;
            rank = below + at_lo + in_rank[r];
        }
        const bool under = rank < below;
        rank -= below;
        const bool lower = rank < at_lo;
        if (!lower) rank -= at_lo;
        const bool upper = !lower && rank >= total && rank - total < at_hi;
        if (!under && (lower || upper)) {
            if (tid == 0) {
                st->prefix[r] = fkey(lower ? win->vlo : win->vhi);
                win->bin[r] = kNoBin;
            }
            continue;
        }
        if (under || over || rank >= total) {
            if (tid == 0) win->miss = 1;
            continue;
        }
        const uint32_t in = (uint32_t)rank;
        if (in >= before && in < incl) {
            uint32_t cum = before;
            int q = 0;
            while (q < PER - 1 && in >= cum + c[q]) cum += c[q++];
            win->bin[r] = (uint32_t)(tid * PER + q);
            win->rank[r] = in - cum;
        }
    }
}

// Before another cut of the lists (select null) or the select over S.
__global__ __launch_bounds__(1024) void k_win_again(SelWin *win, uint32_t *whist, SelState *select) {
    for (int b = threadIdx.x; b < kWinBins; b += blockDim.x) whist[b] = 0u;
    if (threadIdx.x != 0) return;
    win->miss = 0;
    win->nlist = win->done[1] = win->done[2] = 0u;
    win->kmin[0] = win->kmin[1] = 0xffffffffu;
    win->kmax[0] = win->kmax[1] = 0u;
    if (select != nullptr) select->prefix[0] = select->prefix[1] = 0u;
}

// Collects the keys of the two intervals; the last workgroup ranks them: ten
// bits at a time below the interval's.
__global__ __launch_bounds__(RANK_T) void k_win_rank(SelState *st, SelWin *win, const SelSeg *segs,
                                                     const uint32_t *cand, uint32_t cap, uint32_t *list2,
                                                     const uint32_t *minmax, int cut, const int32_t *bad) {
    if (*bad || win->miss) return;
    extern __shared__ uint32_t keys[];       // kWinList
    __shared__ uint32_t hist[1024], wtot[RANK_T / 64], found[3], held, at0, bmin[2], bmax[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sg = blockIdx.x;
    const uint32_t cnt = segs[sg].count < cap ? segs[sg].count : cap;
    const uint32_t *list = cand + (int64_t)sg * cap;
    const uint32_t b0 = win->bin[0], b1 = win->bin[1];
    if (b0 == kNoBin && b1 == kNoBin) return;
    uint32_t lo, shift;
    win_cut(win, minmax, cut, lo, shift);
    const uint32_t hi = cut == CUT_AGAIN ? win->hi : 0xffffffffu;
    if (tid == 0) held = 0u;
    if (tid < 2) {
        bmin[tid] = 0xffffffffu;
        bmax[tid] = 0u;
    }
    __syncthreads();
    uint32_t kmin[2] = {0xffffffffu, 0xffffffffu}, kmax[2] = {0u, 0u};
    for (uint32_t e0 = 0u; e0 < cnt; e0 += 8 * RANK_T) {
        const uint32_t e = e0 + (uint32_t)tid;
        uint32_t key[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) key[u] = e + u * RANK_T < cnt ? list[e + u * RANK_T] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t b = (key[u] - lo) >> shift;
            const bool hit = e + u * RANK_T < cnt && key[u] >= lo && key[u] <= hi && (b == b0 || b == b1);
            const unsigned long long m = __ballot(hit);
            if (m == 0ull) continue;
            uint32_t at = 0u;
            if (lane == 0) at = atomicAdd(&held, (uint32_t)__popcll(m));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + __popcll(m & ((1ull << lane) - 1ull));
            if (!hit) continue;
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (b == (r ? b1 : b0)) {
                    kmin[r] = min(kmin[r], key[u]);
                    kmax[r] = max(kmax[r], key[u]);
                }
            if (at < (uint32_t)kWinList) keys[at] = key[u];
        }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (kmin[r] <= kmax[r]) {
            atomicMin(&bmin[r], kmin[r]);
            atomicMax(&bmax[r], kmax[r]);
        }
    __syncthreads();
    if (tid == 0) at0 = atomicAdd(&win->nlist, held);
    if (tid < 2 && bmin[tid] <= bmax[tid]) {
        atomicMin(&win->kmin[tid], bmin[tid]);
        atomicMax(&win->kmax[tid], bmax[tid]);
    }
    __syncthreads();
    for (uint32_t e = tid; e < held && e < (uint32_t)kWinList; e += RANK_T)
        if (at0 + e < (uint32_t)kWinList) st_dev(&list2[at0 + e], keys[e]);
    if (!last_block(&win->done[2])) return;
    const uint32_t nl = ld_dev(&win->nlist);
    if (nl > (uint32_t)kWinList) {
        // Many keys in the intervals: one value only (points on a grid), or
        // they are cut again, out of all lists, until one key is left; from
        // more than kRecut keys on the select over S is faster.
        uint32_t all = segs[lane].count < cap ? segs[lane].count : cap;
        for (int off = 32; off >= 1; off >>= 1) all += __shfl_xor(all, off, 64);
        const int first = b0 == kNoBin;          // a rank whose key is not known
        const uint32_t k0 = ld_dev(&win->kmin[first]), k1 = ld_dev(&win->kmax[first]);
        const bool one = b0 == b1 || first || b1 == kNoBin;   // one interval in question
        if (all > kRecut && (!one || k0 != k1)) {
            if (tid == 0) {
                const int bits = k0 != k1 ? 32 - __builtin_clz(k1 - k0) : 0;
                win->lo = k0;
                win->hi = k1;
                win->shift = bits > 12 ? bits - 12 : 0;
                win->miss = one ? kCutAgain : 1;
            }
            return;
        }
        // a few long lists where everything is set aside, else many short ones
        const int per = cut == CUT_WHOLE ? RANK_T : 64;
        bool both = b0 == b1;                    // the ranks still share an interval
        uint32_t from1 = ld_dev(&win->kmin[1]), to1 = ld_dev(&win->kmax[1]), rank1 = win->rank[1];
        for (int r = 0; r < 2; ++r) {
            if ((r ? b1 : b0) == kNoBin) continue;
            uint32_t from = r ? from1 : ld_dev(&win->kmin[0]), to = r ? to1 : ld_dev(&win->kmax[0]);
            uint32_t rank = r ? rank1 : win->rank[0];
            while (from != to) {
                const int bits = 32 - __builtin_clz(to - from);
                const uint32_t sh = bits > 11 ? bits - 11 : 0;
                for (int b = tid; b < 2048; b += RANK_T) keys[b] = 0u;
                __syncthreads();
                for (int q = tid / per; q < kSegs; q += RANK_T / per) {
                    const uint32_t c = segs[q].count < cap ? segs[q].count : cap;
                    const uint32_t *l = cand + (int64_t)q * cap;
                    for (uint32_t e = tid % per; e < c; e += 8 * per) {
                        uint32_t key[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) key[u] = e + u * per < c ? l[e + u * per] : 0u;
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (e + u * per < c && key[u] >= from && key[u] <= to) atomicAdd(&keys[(key[u] - from) >> sh], 1u);
                    }
                }
                __syncthreads();
                const uint32_t c0 = keys[2 * tid], own = c0 + keys[2 * tid + 1];
                uint32_t incl = own;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t o = __shfl_up(incl, off, 64);
                    if (lane >= off) incl += o;
                }
                if (lane == 63) wtot[wave] = incl;
                __syncthreads();
                for (int w = 0; w < wave; ++w) incl += wtot[w];
                const uint32_t before = incl - own;
                if (rank >= before && rank < incl) {
                    const bool second = rank - before >= c0;
                    found[0] = 2u * (uint32_t)tid + second;
                    found[1] = before + (second ? c0 : 0u);
                    found[2] = second ? own - c0 : c0;
                }
                __syncthreads();
                // (rank 1 is not below rank 0)
                both = both && r == 0 && rank1 - found[1] < found[2];
                from += found[0] << sh;
                rank -= found[1];
                const uint32_t last = from + ((1u << sh) - 1u);
                to = last < to ? last : to;
                if (both) {
                    from1 = from;
                    to1 = to;
                    rank1 -= found[1];
                }
                __syncthreads();
            }
            if (tid == 0) st->prefix[r] = from;
        }
        return;
    }
    for (uint32_t e = tid; e < nl; e += RANK_T) keys[e] = ld_dev(&list2[e]) - lo;
    __syncthreads();
    for (int r = 0; r < 2; ++r) {
        uint32_t prefix = r ? b1 : b0, rank = win->rank[r];
        if (prefix == kNoBin) continue;
        if (nl > 1024u) {                        // one value only?
            const uint32_t least = ld_dev(&win->kmin[r]);
            if (least == ld_dev(&win->kmax[r])) {
                if (tid == 0) st->prefix[r] = least;
                continue;
            }
        }
        for (int left = (int)shift; left > 0;) {
            const int bits = left < 10 ? left : 10;
            const int sh = left - bits;
            hist[tid] = 0u;
            __syncthreads();
            for (uint32_t e = tid; e < nl; e += RANK_T)
                if (keys[e] >> left == prefix) atomicAdd(&hist[(keys[e] >> sh) & ((1u << bits) - 1u)], 1u);
            __syncthreads();
            const uint32_t own = hist[tid];
            uint32_t incl = own;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(incl, off, 64);
                if (lane >= off) incl += o;
            }
            if (lane == 63) wtot[wave] = incl;
            __syncthreads();
            for (int w = 0; w < wave; ++w) incl += wtot[w];
            if (rank >= incl - own && rank < incl) {
                found[0] = (uint32_t)tid;
                found[1] = rank - (incl - own);
            }
            __syncthreads();
            prefix = prefix << bits | found[0];
            rank = found[1];
            left = sh;
            __syncthreads();
        }
        if (tid == 0) st->prefix[r] = lo + prefix;
    }
}

// What the host reads at the end (pinned host memory).
struct SimReport {
    double pref;
    uint32_t bounds[2];
    int32_t bad, miss;
};

struct PrefArgs {
    float *S;
    int64_t n, ld;
    int mode;                 // APX_PREF_*
    const float *pref_vec;
    float pref_scalar;
    const SelState *sel;      // median mode
    const uint32_t *minmax;
    uint64_t seed;
    double noise_rel;
    double *pref_dev;         // out: the scalar preference (median/scalar)
    const int32_t *bad = nullptr;   // nonzero: the input failed the finite check, write nothing
    const SelWin *win = nullptr;    // miss set: the median is not known yet, write nothing
    SimReport *rep = nullptr;
};

__device__ __forceinline__ double pref_of(const PrefArgs &a, int64_t i, double pm) {
    if (a.mode == APX_PREF_VECTOR) return (double)a.pref_vec[i];
    return pm;
}

__device__ __forceinline__ double median_of(const PrefArgs &a) {
    if (a.mode == APX_PREF_MEDIAN)
        return 0.5 * ((double)keyf(a.sel->prefix[0]) + (double)keyf(a.sel->prefix[1]));
    return (double)a.pref_scalar;
}

// SplitMix64 output function (Steele, Lea, Flood 2014) on the counter
// seed + (i*n+k+1) * golden gamma; top 53 bits as a double in [0,1).
__device__ __forceinline__ double noise_u(uint64_t seed, int64_t n, int64_t i, int64_t k) {
    uint64_t z = seed + (uint64_t)(i * n + k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

// fl32((double)v + scale * u) for u in [0, 1).  When scale <= |v| 2^-27 the
// sum stays below v + 2^(e-26) (2^e <= |v|), far from the midpoint to v's
// upper neighbour (at least 2^(e-25) away, also when |v| is a power of two
// and v < 0), so it rounds back to v and the counter generator is skipped:
// the same value, without its 64-bit arithmetic (the tie noise is far below
// one FP32 ulp of most entries).
__device__ __forceinline__ float add_noise(float v, double scale, uint64_t seed, int64_t n, int64_t i, int64_t k) {
    const double dv = (double)v;
    if (scale <= fabs(dv) * 0x1p-27) return v;
    return (float)(dv + scale * noise_u(seed, n, i, k));
}

// The noise of an upper entry v = s(i,k) that the noise changes, written at
// (i,k) and, with its own draw, at (k,i).  Out of line: the row walks call
// it for few entries, and inlined into each of their unrolled element slots
// its 64-bit arithmetic would take the registers of their loads in flight.
__device__ __noinline__ void put_noise(float *S, int64_t ld, float v, double scale, uint64_t seed, int64_t n,
                                       int64_t i, int64_t k) {
    S[i * ld + k] = add_noise(v, scale, seed, n, i, k);
    S[k * ld + i] = add_noise(v, scale, seed, n, k, i);
}

// Range of S with the preferences on the diagonal (FP64).
__global__ void k_pref_range(PrefArgs a, double *range_out) {
    __shared__ float lo[256], hi[256];
    const double pm = median_of(a);
    float mn = keyf(a.minmax[0]), mx = keyf(a.minmax[1]);
    for (int64_t i = threadIdx.x; i < a.n; i += blockDim.x) {
        const float p = (float)pref_of(a, i, pm);
        mn = fminf(mn, p);
        mx = fmaxf(mx, p);
    }
    lo[threadIdx.x] = mn;
    hi[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
            lo[threadIdx.x] = fminf(lo[threadIdx.x], lo[threadIdx.x + w]);
            hi[threadIdx.x] = fmaxf(hi[threadIdx.x], hi[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *range_out = (double)hi[0] - (double)lo[0];
        *a.pref_dev = pm;
        if (a.rep != nullptr) {
            SimReport r;
            r.pref = pm;
            r.bounds[0] = a.minmax[0];
            r.bounds[1] = a.minmax[1];
            r.bad = *a.bad;
            r.miss = a.win != nullptr ? a.win->miss : 0;
            *a.rep = r;
        }
    }
}

// Diagonal := preference (+ its noise); with noise, every off-diagonal entry
// v becomes fl32(v + scale * u(i,k)).  S is symmetric before the noise, so
// the upper triangle alone is read: an entry the noise changes (add_noise)
// is written at (i,k) and, with its own draw, at (k,i); the others keep v.
// No entry of S is read where the largest one is so far below zero that the
// noise cannot change any (add_noise's bound at the largest value).
__global__ __launch_bounds__(256) void k_pref_noise(PrefArgs a, const double *range) {
    if ((a.bad != nullptr && *a.bad) || (a.win != nullptr && a.win->miss)) return;
    const double pm = median_of(a);
    const double scale = a.noise_rel * (*range);
    const bool noise = a.noise_rel > 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * 256) {
        const double base = pref_of(a, i, pm);
        a.S[i * a.ld + i] = noise ? (float)(base + scale * noise_u(a.seed, a.n, i, i)) : (float)base;
    }
    const float top = keyf(a.minmax[1]);
    if (!noise || (top < 0.0f && scale <= fabs((double)top) * 0x1p-27)) return;
    for (int64_t i = blockIdx.x; i < a.n; i += gridDim.x)
        upper_row<8>(a.S + i * a.ld, i, a.n, [&](int64_t k, float v) {
            if (scale <= fabs((double)v) * 0x1p-27) return;
            put_noise(a.S, a.ld, v, scale, a.seed, a.n, i, k);
        });
}

// ---- matrix-free S: row panels ---------------------------------------------
// Rows [p0, p1) of S into a panel (row i at Sp + (i - p0) * ld), every tile
// of the panel computed (nothing mirrored).  An entry gets the value that
// ap_similarity stores: the same Gram sum (gram_tile), then, with final set,
// the preference on the diagonal and the tie noise as the median or the
// preference pass adds it (the off-diagonal noise scale is the range of the
// off-diagonal entries in median mode, of S with the preferences otherwise).
// final = 0: the values before both, and the bounds of the off-diagonal keys.
struct PanelArgs {
    const float *X;
    int64_t n, d, ldx;
    const float *nrm;
    float *Sp;
    int64_t ld, p0, p1;
    int final;
    PrefArgs pa;              // preference mode and values, select state, bounds, noise
    const double *range;      // final: range of S with the preferences
    uint32_t *minmax;         // final = 0: bounds of the off-diagonal keys (atomic)
    const ApState *st;        // nullable: a frozen run skips the panel
};

__global__ __launch_bounds__(NT) void k_sim_panel(PanelArgs a) {
    if (a.st != nullptr && a.st->frozen) return;
    const int64_t tn = (a.n + BM - 1) / BM;
    const int64_t bi = blockIdx.x / tn, bj = blockIdx.x % tn;
    const int64_t row0 = a.p0 + bi * BM, col0 = bj * BM;
    __shared__ float As[KB * LDA], Bs[KB * LDA];
    __shared__ float nr[BM], nc[BM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    for (int e = tid; e < BM; e += NT) {
        nr[e] = row0 + e < a.n ? a.nrm[row0 + e] : 0.0f;
        nc[e] = col0 + e < a.n ? a.nrm[col0 + e] : 0.0f;
    }
    v16f acc[2][2];
    gram_tile(a.X, a.n, a.d, a.ldx, row0, col0, acc, As, Bs);

    double pm = 0.0, sc_off = 0.0, sc_diag = 0.0;
    if (a.final) {
        pm = median_of(a.pa);
        sc_diag = a.pa.noise_rel * (*a.range);
        sc_off = a.pa.mode == APX_PREF_MEDIAN
            ? a.pa.noise_rel * ((double)keyf(a.pa.minmax[1]) - (double)keyf(a.pa.minmax[0]))
            : sc_diag;
    }
    const bool noise = a.pa.noise_rel > 0.0;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int c = wn * 64 + y * 32 + (lane & 31);
            const int64_t k = col0 + c;
            const float ncc = nc[c];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int mb = wm * 64 + x * 32 + 8 * g + 4 * (lane >> 5);
                const int64_t ib = row0 + mb;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t i = ib + q;
                    if (k >= a.n || i >= a.p1) continue;
                    const float v = 2.0f * acc[x][y][4 * g + q] - (nr[mb + q] + ncc);
                    float out = v;
                    if (!a.final) {
                        if (k != i) {
                            const uint32_t key = fkey(v);
                            kmin = min(kmin, key);
                            kmax = max(kmax, key);
                        }
                    } else if (k == i) {
                        const double base = pref_of(a.pa, i, pm);
                        out = noise ? (float)(base + sc_diag * noise_u(a.pa.seed, a.n, i, i)) : (float)base;
                    } else if (noise) {
                        out = add_noise(v, sc_off, a.pa.seed, a.n, i, k);
                    }
                    a.Sp[(i - a.p0) * a.ld + k] = out;
                }
            }
        }
    if (!a.final) {
        for (int off = 32; off >= 1; off >>= 1) {
            kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off, 64));
            kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off, 64));
        }
        if (lane == 0) {
            if (kmin < __atomic_load_n(&a.minmax[0], __ATOMIC_RELAXED)) atomicMin(&a.minmax[0], kmin);
            if (kmax > __atomic_load_n(&a.minmax[1], __ATOMIC_RELAXED)) atomicMax(&a.minmax[1], kmax);
        }
    }
}

}  // namespace
}  // namespace apx

using namespace apx;

#define HIP_TRY(expr, what)                                   \
    do {                                                      \
        hipError_t _e = (expr);                               \
        if (_e != hipSuccess) return hip_err(ctx, _e, what);  \
    } while (0)

namespace {
struct SimLayout {
    size_t o_n, o_mm, o_sel, o_h, o_r, base;                  // also the matrix-free sweeps'
    size_t o_win, o_seg, o_wh, o_l, o_smp, o_cand, bytes;     // the median's window
    int64_t cap;
};
SimLayout sim_layout(int64_t n) {
    WsLayout L;
    SimLayout o{};
    o.o_n = L.take(sizeof(float) * (size_t)n);
    o.o_mm = L.take(sizeof(uint32_t) * 2);
    o.o_sel = L.take(sizeof(SelState));
    o.o_h = L.take(sizeof(unsigned long long) * 2 * SEL_BINS);
    o.o_r = L.take(sizeof(double) * 2);
    o.base = L.off;
    o.cap = seg_cap(n);
    o.o_win = L.take(sizeof(SelWin));
    o.o_seg = L.take(sizeof(SelSeg) * kSegs);
    o.o_wh = L.take(sizeof(uint32_t) * kWinBins);
    o.o_l = L.take(sizeof(uint32_t) * kWinList);
    o.o_smp = L.take(sizeof(uint32_t) * kSamples);
    o.o_cand = L.take(sizeof(uint32_t) * (size_t)kSegs * (size_t)o.cap);
    o.bytes = L.off;
    return o;
}
}  // namespace

size_t apx::similarity_ws_bytes(int64_t n) { return sim_layout(n).bytes; }
size_t apx::similarity_ws_least(int64_t n) { return sim_layout(n).base; }

extern "C" apx_status ap_similarity(apx_ctx *ctx, const float *X, int64_t n, int64_t d, int64_t ldx,
                                    float *S, int64_t ld, int32_t pref_mode, const float *pref_vec,
                                    float pref_scalar, uint64_t noise_seed, double noise_rel,
                                    double *pref_out) {
    if (!ctx) return APX_EINVAL;
    if (!X || !S) return set_err(ctx, APX_EINVAL, "X and S must be non-null");
    if (n < 2 || d < 1) return set_err(ctx, APX_EINVAL, "need n >= 2 and d >= 1");
    if (n > (int64_t)1 << 31) return set_err(ctx, APX_ENOTIMPL, "n too large");
    if (ldx < d) return set_err(ctx, APX_EINVAL, "ldx < d");
    if (ld < n || ld % 4) return set_err(ctx, APX_EINVAL, "ld must be >= n and a multiple of 4");
    if ((reinterpret_cast<uintptr_t>(S) & 15u) != 0) return set_err(ctx, APX_EINVAL, "S not 16-byte aligned");
    if (pref_mode < APX_PREF_MEDIAN || pref_mode > APX_PREF_VECTOR)
        return set_err(ctx, APX_EINVAL, "bad pref_mode");
    if (pref_mode == APX_PREF_VECTOR && !pref_vec) return set_err(ctx, APX_EINVAL, "pref_vec is null");
    if (pref_mode == APX_PREF_SCALAR && !std::isfinite(pref_scalar))
        return set_err(ctx, APX_EINVAL, "pref_scalar is not finite");
    if (!(noise_rel >= 0.0) || !std::isfinite(noise_rel)) return set_err(ctx, APX_EINVAL, "bad noise_rel");
    int cur = -1;
    (void)hipGetDevice(&cur);
    if (cur != ctx->device) (void)hipSetDevice(ctx->device);
    hipStream_t s = ctx->stream;

    const SimLayout SL = sim_layout(n);
    const size_t o_n = SL.o_n, o_mm = SL.o_mm, o_sel = SL.o_sel, o_h = SL.o_h, o_r = SL.o_r;
    // The median's window needs room for the keys set aside (1.7% of S); where
    // there is none (a caller's workspace without it, a device without that
    // much memory left) the radix select runs.  The workspace does not grow
    // for it while a caller inside the library keeps data below ws_base.
    const bool median = pref_mode == APX_PREF_MEDIAN;
    bool windowed = median;
    if (windowed && ctx->ws_base + SL.bytes > ctx->ws_bytes)
        windowed = !ctx->ws_external && ctx->ws_base == 0 && ws_reserve(ctx, SL.bytes) == APX_OK;
    apx_status st = ws_reserve(ctx, ctx->ws_base + (windowed ? SL.bytes : SL.base));
    if (st != APX_OK) return st;

    char *b = static_cast<char *>(ctx->ws) + ctx->ws_base;
    float *nrm = reinterpret_cast<float *>(b + o_n);
    uint32_t *mm = reinterpret_cast<uint32_t *>(b + o_mm);
    SelState *sel = reinterpret_cast<SelState *>(b + o_sel);
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(b + o_h);
    double *dvals = reinterpret_cast<double *>(b + o_r);   // [0] range, [1] preference
    SelWin *win = windowed ? reinterpret_cast<SelWin *>(b + SL.o_win) : nullptr;
    SelSeg *segs = reinterpret_cast<SelSeg *>(b + SL.o_seg);
    uint32_t *whist = reinterpret_cast<uint32_t *>(b + SL.o_wh);
    uint32_t *cand = reinterpret_cast<uint32_t *>(b + SL.o_cand);
    SimReport *rep = reinterpret_cast<SimReport *>(static_cast<char *>(ctx->pinned) + 1024);

    const unsigned long long M = (unsigned long long)n * (unsigned long long)(n - 1) / 2ull;
    const unsigned long long lo = (M % 2) ? (M - 1) / 2 : M / 2 - 1;
    const unsigned long long hi = (M % 2) ? (M - 1) / 2 : M / 2;
    // Non-finite input is rejected before S is written: every kernel that
    // writes S reads the flag first and returns when it is set; the host
    // reads it at the end.
    int32_t *bad = static_cast<int32_t *>(ctx->dflag);
    k_sel_init<<<1, 1024, 0, s>>>(sel, mm, lo, hi, hist, win, segs, whist, bad);
    HIP_TRY(hipGetLastError(), "select init");
    if (pref_mode == APX_PREF_VECTOR) HIP_TRY(launch_check_finite(pref_vec, 1, n, n, bad, s), "finite check");
    k_sqnorm<<<(unsigned)((n + 63) / 64), 256, 0, s>>>(X, n, d, ldx, nrm, bad);
    HIP_TRY(hipGetLastError(), "sqnorm");
    if (windowed && n > kWholeN) {
        k_sel_sample<<<SMP_BLOCKS, SMP_T, 0, s>>>(X, n, d, ldx, nrm, reinterpret_cast<uint32_t *>(b + SL.o_smp), win,
                                                  bad);
        HIP_TRY(hipGetLastError(), "median sample");
    }
    SimArgs sa{X, n, d, ldx, nrm, S, ld, (n + BM - 1) / BM, mm, win, segs, cand, (uint32_t)SL.cap, bad};
    const int64_t ntiles = sa.tiles_per_side * (sa.tiles_per_side + 1) / 2;
    if (windowed) k_sim_gemm<true><<<(unsigned)ntiles, NT, 0, s>>>(sa);
    else k_sim_gemm<false><<<(unsigned)ntiles, NT, 0, s>>>(sa);
    HIP_TRY(hipGetLastError(), "similarity gemm");
    PrefArgs pa{S, n, ld, pref_mode, pref_vec, pref_scalar, sel, mm, noise_seed, noise_rel, &dvals[1], bad, win, rep};
    const int noise_grid = (int)(n < 4096 ? n : 4096);
    uint32_t *list2 = reinterpret_cast<uint32_t *>(b + SL.o_l);
    auto from_lists = [&](int cut) -> apx_status {
        const uint32_t cap = (uint32_t)SL.cap;
        k_win_count<<<kSegs, RANK_T, 0, s>>>(sel, win, segs, cand, cap, whist, mm, cut, bad);
        HIP_TRY(hipGetLastError(), "median count");
        constexpr size_t lds = sizeof(uint32_t) * kWinList;
        HIP_TRY(hipFuncSetAttribute((const void *)k_win_rank, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
                "lds");
        k_win_rank<<<kSegs, RANK_T, lds, s>>>(sel, win, segs, cand, cap, list2, mm, cut, bad);
        HIP_TRY(hipGetLastError(), "median rank");
        return APX_OK;
    };
    if (windowed) {
        st = from_lists(n <= kWholeN ? CUT_WHOLE : CUT_WINDOW);
        if (st != APX_OK) return st;
    }
    bool searched = windowed || !median;
    for (;;) {
        if (!searched) {
            // three digits of the keys, a pass over the upper triangle each
            for (int pass = 0; pass < 3; ++pass) {
                const size_t lds = sizeof(uint32_t) * (pass == 0 ? 8192 : 2 * (pass == 1 ? 1024 : 512));
                const int g = walk_grid((const void *)k_sel_hist, lds, n - 1);
                k_sel_hist<<<g, 256, lds, s>>>(S, n, ld, sel, pass, hist, 0, n);
                HIP_TRY(hipGetLastError(), "select histogram");
                k_sel_pick<<<1, 256, 0, s>>>(sel, pass, hist);
                HIP_TRY(hipGetLastError(), "select pick");
            }
            pa.win = nullptr;
        }
        k_pref_range<<<1, 256, 0, s>>>(pa, &dvals[0]);
        HIP_TRY(hipGetLastError(), "preference range");
        k_pref_noise<<<noise_grid, 256, 0, s>>>(pa, &dvals[0]);
        HIP_TRY(hipGetLastError(), "preference/noise");
        HIP_TRY(hipStreamSynchronize(s), "sync");
        if (rep->bad || !rep->miss) break;
        // (nothing of the preferences has been written)
        const bool again = rep->miss == kCutAgain;
        k_win_again<<<1, 1024, 0, s>>>(win, whist, again ? nullptr : sel);
        HIP_TRY(hipGetLastError(), "median again");
        if (again) {
            // (a cut leaves 2^-12 of a range of keys: three at most)
            st = from_lists(CUT_AGAIN);
            if (st != APX_OK) return st;
        } else {
            searched = false;
        }
    }
    // The bounds of the off-diagonal keys tell whether a similarity overflowed
    // (a key at or beyond the one of +inf or -inf: infinities and NaNs).
    if (rep->bad) return set_err(ctx, APX_EINVAL, "X or pref_vec holds a NaN or infinite value");
    const uint32_t key_pinf = 0xff800000u, key_ninf = 0x007fffffu;   // fkey(+inf), fkey(-inf)
    if (rep->bounds[1] >= key_pinf || rep->bounds[0] <= key_ninf)
        return set_err(ctx, APX_EINVAL, "similarities overflow FP32 (S holds non-finite values)");
    if (pref_out) *pref_out = pref_mode == APX_PREF_VECTOR ? NAN : rep->pref;
    return APX_OK;
}

// ---- matrix-free similarity: the row panels of ap_solve_mf -----------------
namespace apx {

size_t mf_sim_bytes(int64_t n) { return sim_layout(n).base; }

namespace {
struct MfPtrs {
    float *nrm;
    uint32_t *mm;
    SelState *sel;
    unsigned long long *hist;
    double *dvals;   // [0] range, [1] preference
};
MfPtrs mf_ptrs(const MfSim &m) {
    const SimLayout L = sim_layout(m.n);
    MfPtrs q;
    q.nrm = reinterpret_cast<float *>(m.ws + L.o_n);
    q.mm = reinterpret_cast<uint32_t *>(m.ws + L.o_mm);
    q.sel = reinterpret_cast<SelState *>(m.ws + L.o_sel);
    q.hist = reinterpret_cast<unsigned long long *>(m.ws + L.o_h);
    q.dvals = reinterpret_cast<double *>(m.ws + L.o_r);
    return q;
}
PanelArgs panel_args(const MfSim &m, const MfPtrs &q, float *panel, int64_t ld, int64_t p0, int64_t p1, int final,
                     const ApState *st) {
    PanelArgs a{};
    a.X = m.X;
    a.n = m.n;
    a.d = m.d;
    a.ldx = m.ldx;
    a.nrm = q.nrm;
    a.Sp = panel;
    a.ld = ld;
    a.p0 = p0;
    a.p1 = p1;
    a.final = final;
    a.pa = PrefArgs{nullptr, m.n, ld, m.pref_mode, m.pref_vec, m.pref_scalar, q.sel, q.mm, m.seed, m.noise_rel,
                    &q.dvals[1]};
    a.range = &q.dvals[0];
    a.minmax = q.mm;
    a.st = st;
    return a;
}
hipError_t launch_panel(const PanelArgs &a, hipStream_t s) {
    const int64_t tiles = ((a.p1 - a.p0 + BM - 1) / BM) * ((a.n + BM - 1) / BM);
    k_sim_panel<<<(unsigned)tiles, NT, 0, s>>>(a);
    return hipGetLastError();
}
}  // namespace

const double *mf_sim_pref(const MfSim &m) { return &mf_ptrs(m).dvals[1]; }
const uint32_t *mf_sim_bounds(const MfSim &m) { return mf_ptrs(m).mm; }

// Norms, the bounds of the off-diagonal entries, the median (three digit
// sweeps of the upper triangle, one panel at a time) and the range of S with
// the preferences: what ap_similarity derives from the stored S.
hipError_t mf_sim_setup(const MfSim &m, float *panel, int64_t ld, int64_t prows, hipStream_t s) {
    const MfPtrs q = mf_ptrs(m);
    const int64_t n = m.n;
    const unsigned long long M = (unsigned long long)n * (unsigned long long)(n - 1) / 2ull;
    const unsigned long long lo = (M % 2) ? (M - 1) / 2 : M / 2 - 1;
    const unsigned long long hi = (M % 2) ? (M - 1) / 2 : M / 2;
    k_sel_init<<<1, 256, 0, s>>>(q.sel, q.mm, lo, hi, q.hist, nullptr, nullptr, nullptr, nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_sqnorm<<<(unsigned)((n + 63) / 64), 256, 0, s>>>(m.X, n, m.d, m.ldx, q.nrm, nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int sweeps = m.pref_mode == APX_PREF_MEDIAN ? 3 : 1;
    for (int pass = 0; pass < sweeps; ++pass) {
        for (int64_t p0 = 0; p0 < n; p0 += prows) {
            const int64_t p1 = p0 + prows < n ? p0 + prows : n;
            if ((e = launch_panel(panel_args(m, q, panel, ld, p0, p1, 0, nullptr), s)) != hipSuccess) return e;
            if (m.pref_mode == APX_PREF_MEDIAN) {
                const size_t lds = sizeof(uint32_t) * (pass == 0 ? 8192 : 2 * (pass == 1 ? 1024 : 512));
                const int g = walk_grid((const void *)k_sel_hist, lds, p1 - p0);
                k_sel_hist<<<g, 256, lds, s>>>(panel - p0 * ld, n, ld, q.sel, pass, q.hist, p0, p1);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
        if (m.pref_mode == APX_PREF_MEDIAN) {
            k_sel_pick<<<1, 256, 0, s>>>(q.sel, pass, q.hist);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    const PanelArgs a = panel_args(m, q, panel, ld, 0, 0, 1, nullptr);
    k_pref_range<<<1, 256, 0, s>>>(a.pa, &q.dvals[0]);
    return hipGetLastError();
}

hipError_t mf_sim_panel(const MfSim &m, float *panel, int64_t ld, int64_t p0, int64_t p1, const ApState *st,
                        hipStream_t s) {
    return launch_panel(panel_args(m, mf_ptrs(m), panel, ld, p0, p1, 1, st), s);
}

}  // namespace apx
