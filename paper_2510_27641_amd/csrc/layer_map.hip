// Offline layer mapping (Section 3.3, Eq. 4; Appendix B, Algorithm 3).
//
// 1. Similarity: S[i][j] = -(1/rows) * sum_r D_KL(A^v_j[r] || A^d_i[r]) over aligned attention rows of the two
//    models (Eq. 4, averaged over the rows a representative data set yields).  fp32 probabilities in, fp64
//    logarithms, products and sums.  Written as  sum p_j log p_j - sum p_j log q_i  the second sum is a contraction
//    [draft layers x entries] . [entries x verifier layers], so every logarithm is taken once per layer instead of
//    once per layer pair, and the products run on the fp64 matrix cores (v_mfma_f64_16x16x4).
// 2. Alignment: the non-decreasing map f (verifier layer -> draft layer) that maximises sum_j S[f(j)][j],
//    by the recurrence of Algorithm 3 (its "above" transition contains the other two):
//    best[i][j] = S[i][j] + max_{k <= i} best[k][j-1], first maximum at ties.  One workgroup, thread i holds
//    draft layer i; up to 64 of them go through the table by diagonals, more take a prefix maximum over the threads per column.
#include "common.h"

#include <cmath>
#include <mutex>

namespace specattn {
namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // layers start at any multiple of four bytes

constexpr int KL_WAVES = 8, KL_FEW_WAVES = 4;        // per workgroup (kl_plan)
constexpr int KL_WAVE_K = 64;                        // entries of a layer one wave takes per iteration
constexpr int KL_TI = 32, KL_TJ = 32;                // draft and verifier layers per workgroup
constexpr int KL_ROW = KL_WAVE_K + 2;                // doubles per staged row: rows start four banks apart
constexpr int KL_SUMS = 4 * 256 + 2 * 64;            // doubles of a wave's sums: four tiles of pairs, two of the small products
constexpr int KL_WAVE_LDS = KL_TI * KL_ROW > KL_SUMS ? KL_TI * KL_ROW : KL_SUMS;     // doubles
constexpr int LOG_FIRST = 64, LOG_ENTRIES = 118;     // table of logarithms: of 64/128 to 181/128
constexpr int kl_lds_bytes(int waves) { return (waves * KL_WAVE_LDS + 2 * LOG_ENTRIES) * (int)sizeof(double); }
constexpr int MAP_THREADS = 1024;      // most draft layers the alignment kernel takes
constexpr int MAP_LDS_BACK = 24576;    // back pointers kept in LDS (16 bits each); larger tables use the workspace

// What stands for log(q) where there is none: a draft entry of 0 makes the divergence infinite as soon as a verifier
// entry above 0 meets it (p >= 2^-149 leaves at least 1e115 in the sum, far beyond any finite divergence) and must not
// disturb the sum otherwise (0 * -infinity would).  Entries that are no probabilities (negative, infinite, NaN) drown
// everything else (at least 1e245, against 4e210 of the zeros); the finish kernel adds such pairs up term by term.
constexpr double LOG_OF_ZERO = -1e160, LOG_OF_INVALID = 1e290, DIVERGENCE_LIMIT = 1e100;

// Natural logarithm in fp64 of a positive finite fp32 value from a table of logarithms (P. T. P. Tang, "Table-driven
// implementation of the logarithm function in IEEE floating-point arithmetic", 1990).  x = 2^e y / 128 with y / 128 in
// [sqrt(1/2), sqrt(2)) (the last subnormal values: from 1/2 on), j the integer next to y: log x = e log 2 + log(j / 128) +
// log1p((y - j) / j).  e, y, j and the difference are exact in fp32, so the reduction runs there; the table holds 1/j and
// log(j / 128), the series has degree 8 (|r| <= 2^-7.5: remainder below 2^-63 of it).  Next to 1, j is 128 and the result
// r's series alone.  Within 1.4 units in the last place over all of fp32; about 25 instructions, against more than 100 of the
// general fp64 logarithm.  Values that have no logarithm are taken as the nearest one that has.
__device__ __forceinline__ double log_positive(float x, const f64x2 *tab)
{
    x = __builtin_amdgcn_fmed3f(x, 1.4012985e-45f, 3.4028235e38f);
    const int e = __builtin_amdgcn_frexp_expf(x * 0.70710678f);
    const float y = __builtin_amdgcn_ldexpf(x, 7 - e);
    const float j = rintf(y);
    const f64x2 t = tab[(int)j - LOG_FIRST];
    const double r = (double)(y - j) * t[0];
    double p = fma(r, -1.0 / 8, 1.0 / 7);
    p = fma(p, r, -1.0 / 6);
    p = fma(p, r, 1.0 / 5);
    p = fma(p, r, -1.0 / 4);
    p = fma(p, r, 1.0 / 3);
    p = fma(p, r, -0.5);
    p = fma(p * r, r, r);
    return fma((double)e, 0.69314718055994530942, t[1]) + p;
}
__device__ __forceinline__ bool has_log(float q) { return q > 0.0f && q < INFINITY; }
__device__ __forceinline__ double log_draft(float q, const f64x2 *tab)
{
    const double l = log_positive(q, tab);
    return has_log(q) ? l : (q == 0.0f ? LOG_OF_ZERO : LOG_OF_INVALID);
}

// Entries k .. k+3 of a layer, zero at and beyond `end`; `whole`: none of the wave's lanes reaches that far.
__device__ __forceinline__ f32x4u load4(const float *layer, int64_t k, int64_t end, bool whole)
{
    if (whole) return *reinterpret_cast<const f32x4u *>(layer + k);
    f32x4u v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (k + c < end) v[c] = layer[k + c];
    return v;
}

// Orders a wave's LDS accesses before those after it (the LDS unit serves a wave's accesses in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup (chunk, draft group, verifier group): partial sums of 32 x 32 layer pairs over `iters` runs of 64 entries per wave.
// Every wave works on 64 entries of its own and meets the others only at the end: it takes the logarithms of its
// draft entries into its part of LDS ([layer][entry], fp64), then goes through its verifier entries, 16 layers x 16
// entries at a time, straight from memory: lane l holds entries 4 * (l / 16) .. + 3 of layer l % 16, which is
// a B operand of four matrix instructions; their logarithms are the A operand of a third product, in four blocks of 4 x 4 layers, whose
// diagonals are sum p log p - taken in the same order as the other sums, so that a layer compared with itself gives exactly zero.
// Bound by the logarithms (25 instructions each, m + n of them per entry) and the fp64 products (64 cycles per 16 x 16 x 4), which overlap
// only across the two waves of a SIMD, behind one unhidden trip to memory.  22 x 32 layers, 64 rows x 2048 positions (28 MB, 92 M
// terms): the diagonal from 16 x 16 products, the sums in two rounds 19.6 us / now 17.8 us; two general logarithms per term, one
// workgroup per layer pair and chunk, took 329 us.
__global__ __launch_bounds__(KL_WAVES * 64) void layer_kl_kernel(const float *__restrict__ ad, const float *__restrict__ av, int m,
                                                                 int n, int64_t per_layer, int iters, double *__restrict__ partial)
{
    extern __shared__ __align__(16) double kl_lds[];
    const int waves = blockDim.x >> 6;
    f64x2 *tab = reinterpret_cast<f64x2 *>(kl_lds + waves * KL_WAVE_LDS);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    const int i0 = blockIdx.y * KL_TI, j0 = blockIdx.z * KL_TJ;
    double *lq = kl_lds + wave * KL_WAVE_LDS;
    constexpr int VEC = KL_WAVE_K / 4, QROWS = 64 / VEC;  // lanes that load a draft layer's entries; layers per load
    constexpr int QT = KL_TI / QROWS, PS = KL_WAVE_K / 16;    // vectors of draft and verifier entries per lane (and verifier tile)
    const int lv = lane & (VEC - 1), gv = lane / VEC;
    f32x4u q[QT], p[2][PS];
    // (Layers past the last one repeat it: their sums are not read.)
    auto request = [&](int64_t k0) {
        if (k0 >= per_layer) return;                  // (uniform over the wave)
        const bool whole = k0 + KL_WAVE_K <= per_layer;
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            const int i = i0 + QROWS * t + gv;
            q[t] = load4(ad + (int64_t)(i < m ? i : m - 1) * per_layer, k0 + 4 * lv, per_layer, whole);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int s = 0; s < PS; ++s) {
                const int j = j0 + 16 * a + l16;
                p[a][s] = load4(av + (int64_t)(j < n ? j : n - 1) * per_layer, k0 + 16 * s + 4 * g, per_layer, whole);
            }
    };
    const int64_t step = waves * KL_WAVE_K, first = (int64_t)blockIdx.x * iters * step + wave * KL_WAVE_K;
    request(first);                                   // (on its way while the table is made)
    if (tid < LOG_ENTRIES) {
        const double j = (double)(LOG_FIRST + tid);
        tab[tid] = (f64x2){1.0 / j, log(j / 128.0)};
    }
    __syncthreads();
    f64x4 acc[2][2];                                  // [verifier tile][draft tile]
    double own[2] = {0.0, 0.0};                       // products with the verifier's own logarithms
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[a][t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    for (int it = 0; it < iters; ++it) {
        const int64_t k0 = first + it * step;
        if (k0 >= per_layer) break;                   // (uniform over the wave)
        if (it) request(k0);
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            if (i0 + QROWS * t >= m) break;           // (uniform)
            f64x2 *dst = reinterpret_cast<f64x2 *>(lq + (QROWS * t + gv) * KL_ROW + 4 * lv);
            dst[0] = (f64x2){log_draft(q[t][0], tab), log_draft(q[t][1], tab)};
            dst[1] = (f64x2){log_draft(q[t][2], tab), log_draft(q[t][3], tab)};
        }
        wave_sync();
#pragma unroll
        for (int s = 0; s < PS; ++s) {
            f64x2 a0[2], a1[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                a0[c] = *reinterpret_cast<const f64x2 *>(lq + l16 * KL_ROW + 16 * s + 4 * g + 2 * c);
                a1[c] = *reinterpret_cast<const f64x2 *>(lq + (16 + l16) * KL_ROW + 16 * s + 4 * g + 2 * c);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (j0 + 16 * a >= n) continue;       // (uniform)
                // 0 * log(0 / q) = 0: entries that are not above 0 add nothing (nor do their logarithms).  Where a causal
                // row has ended, whole waves have nothing to do.
                const f32x4u v = p[a][s];
                double lp[4] = {0.0, 0.0, 0.0, 0.0};
                if (fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) > 0.0f)
#pragma unroll
                    for (int c = 0; c < 4; ++c) lp[c] = log_positive(v[c], tab);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double x = fmaxf(v[c], 0.0f);
                    acc[a][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[c >> 1][c & 1], x, acc[a][0], 0, 0, 0);
                    if (i0 + 16 < m) acc[a][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[c >> 1][c & 1], x, acc[a][1], 0, 0, 0);
                    own[a] = __builtin_amdgcn_mfma_f64_4x4x4f64(lp[c], x, own[a], 0, 0, 0);
                }
            }
        }
        wave_sync();
    }
    // the waves' sums, in wave order.  Element (row 4 v + g, column l16) of a tile sits in register v of lane (g, l16), element (i, j) of
    // block b of the small products in lane 16 i + 4 b + j.
    constexpr int OWN = 4 * 256;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) lq[((a * 2 + t) * 16 + 4 * v + g) * 16 + l16] = acc[a][t][v];
        lq[OWN + a * 64 + lane] = own[a];
    }
    __syncthreads();
    auto sum_of_waves = [&](const double *src) {
        double s = 0.0;
        for (int w0 = 0; w0 < waves; w0 += 8) {
            double x[8];
#pragma unroll
            for (int w = 0; w < 8; ++w) x[w] = src[(w0 + w < waves ? w0 + w : w0) * KL_WAVE_LDS];
#pragma unroll
            for (int w = 0; w < 8; ++w) s += w0 + w < waves ? x[w] : 0.0;
        }
        return s;
    };
    for (int e = tid; e < KL_TI * KL_TJ; e += (int)blockDim.x) {
        const int i = e >> 5, j = e & 31, a = j >> 4, jj = j & 15;
        if (i0 + i >= m || j0 + j >= n) continue;
        const double self = sum_of_waves(kl_lds + OWN + a * 64 + 16 * (jj & 3) + jj);
        const double cross = sum_of_waves(kl_lds + (a * 32 + i) * 16 + jj);
        partial[((int64_t)blockIdx.x * m + i0 + i) * n + j0 + j] = self - cross;
    }
}

// Eight pairs per workgroup: 64 threads per pair add its chunks in a fixed order.  A sum that met an entry that is no
// probability is taken again term by term, with the logarithms of the entries as they are.
__global__ __launch_bounds__(512) void layer_kl_finish_kernel(const double *__restrict__ partial, int m, int n, int chunks, double rows,
                                                              const float *__restrict__ ad, const float *__restrict__ av, int64_t per_layer,
                                                              double *__restrict__ S)
{
    __shared__ double red[2][8][8];
    const int pp = threadIdx.x & 7, cl = threadIdx.x >> 3, wave = threadIdx.x >> 6;
    const int pairs = m * n, pair = blockIdx.x * 8 + pp;
    // sums over the threads of a pair: of its eight lanes of a wave, then of the waves
    auto sum_of_threads = [&](double s, double (&part)[8][8]) -> double {
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) s += __shfl_xor(s, off, 64);
        if ((threadIdx.x & 63) < 8) part[wave][pp] = s;
        __syncthreads();
        s = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) s += part[w][pp];
        return s;
    };
    double s = 0.0;
    if (pair < pairs)
        for (int c0 = cl; c0 < chunks; c0 += 256) {   // four requests at a time
            double x[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = partial[(int64_t)(c0 + 64 * k < chunks ? c0 + 64 * k : c0) * pairs + pair];
#pragma unroll
            for (int k = 0; k < 4; ++k) s += c0 + 64 * k < chunks ? x[k] : 0.0;
        }
    s = sum_of_threads(s, red[0]);
    auto is_odd = [&](double x) { return !(x > -DIVERGENCE_LIMIT && x < INFINITY); };
    const bool odd = pair < pairs && is_odd(s);
    if (cl == 0 && pair < pairs && !odd) S[pair] = s > DIVERGENCE_LIMIT ? -INFINITY : -s / rows;
    if (!__any(odd)) return;                          // (every wave holds all eight sums)
    s = 0.0;
    if (odd) {
        const int i = pair / n, j = pair - i * n;
        const float *pd = ad + (int64_t)i * per_layer, *pv = av + (int64_t)j * per_layer;
        for (int64_t k = cl; k < per_layer; k += 64) {
            const double p = pv[k];
            if (p > 0.0) s += p * (log(p) - log((double)pd[k]));
        }
    }
    s = sum_of_threads(s, red[1]);
    if (cl == 0 && odd) S[pair] = -s / rows;
}

struct Best { double val; int idx; };

// (value, index) of the lanes before, or of the lane itself where it is larger: the candidates with lower indices win
// ties.  Lanes that a step has no source for keep what they have.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ void scan_step(Best &b)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(b.val), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)0xfff00000, __double2hiint(b.val), CTRL, ROW_MASK, 0xf, false);
    const int ix = __builtin_amdgcn_update_dpp(0x7fffffff, b.idx, CTRL, ROW_MASK, 0xf, false);
    const double left = __hiloint2double(hi, lo);
    if (ix != 0x7fffffff && !(b.val > left)) { b.val = left; b.idx = ix; }
}

// One thread per draft layer, up to 1024.  A column is a prefix maximum inside every wave on the vector ALU and, with more than 64
// draft layers, one over the wave totals through LDS (double-buffered: one barrier per column).  The columns of S are
// fetched eight at a time and ahead; back pointers stay in LDS as long as they fit.  Bound by the serial chain of n
// columns and n back pointers.  `waves`: those of the workgroup that are here (one has nothing to wait for).
struct AlignShared {
    double wval[2][MAP_THREADS / 64];
    int widx[2][MAP_THREADS / 64];
    int start;
    uint16_t back[MAP_LDS_BACK];
};
__device__ __forceinline__ void align_threads(const double *__restrict__ S, int m, int n, int32_t *__restrict__ back, int32_t *__restrict__ f,
                              double *__restrict__ total, AlignShared &sh, int waves)
{
    const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
    const bool in_lds = (int64_t)m * n <= MAP_LDS_BACK;
    int turn = 0;
    // prefix maximum over the threads with the first index at ties; with more than one wave a barrier
    auto prefix_max = [&](double v) -> Best {
        Best b = {v, i};
        scan_step<0x111, 0xf>(b);     // row_shr:1
        scan_step<0x112, 0xf>(b);     // row_shr:2
        scan_step<0x114, 0xf>(b);     // row_shr:4
        scan_step<0x118, 0xf>(b);     // row_shr:8
        scan_step<0x142, 0xa>(b);     // row_bcast:15 into rows 1 and 3
        scan_step<0x143, 0xc>(b);     // row_bcast:31 into rows 2 and 3
        if (waves > 1) {
            if (lane == 63) { sh.wval[turn][wave] = b.val; sh.widx[turn][wave] = b.idx; }
            __syncthreads();
            for (int w = wave - 1; w >= 0; --w)
                if (!(b.val > sh.wval[turn][w])) { b.val = sh.wval[turn][w]; b.idx = sh.widx[turn][w]; }
            turn ^= 1;
        }
        return b;
    };
    constexpr int AHEAD = 8;
    const double *row = S + (int64_t)(i < m ? i : m - 1) * n;
    double cur[AHEAD], nxt[AHEAD];
#pragma unroll
    for (int c = 0; c < AHEAD; ++c) cur[c] = row[c < n ? c : n - 1];
    double best = -INFINITY;                                   // threads past m never win a maximum
    for (int j0 = 0; j0 < n; j0 += AHEAD) {
#pragma unroll
        for (int c = 0; c < AHEAD; ++c) nxt[c] = row[j0 + AHEAD + c < n ? j0 + AHEAD + c : n - 1];
#pragma unroll
        for (int c = 0; c < AHEAD; ++c) {
            const int j = j0 + c;
            if (j >= n) break;                                 // (uniform)
            if (j == 0) {
                if (i < m) best = cur[c];
                continue;
            }
            const Best b = prefix_max(best);
            if (i < m) {
                if (in_lds) sh.back[i * n + j] = (uint16_t)b.idx;
                else back[(int64_t)i * n + j] = b.idx;
                best = cur[c] + b.val;
            }
        }
#pragma unroll
        for (int c = 0; c < AHEAD; ++c) cur[c] = nxt[c];
    }
    const Best last = prefix_max(best);
    if (i == waves * 64 - 1) {
        sh.start = last.idx < m ? last.idx : 0;                   // first maximum of the last column (all entries -infinity or NaN: layer 0)
        *total = last.val;
    }
    if (waves > 1) __syncthreads();                            // also orders the back pointers
    else __threadfence_block();
    if (i == 0) {
        int at = sh.start;
        f[n - 1] = at;
        for (int j = n - 1; j > 0; --j) {
            at = in_lds ? sh.back[at * n + j] : __hip_atomic_load(&back[(int64_t)at * n + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            f[j - 1] = at;
        }
    }
}

__global__ __launch_bounds__(MAP_THREADS) void layer_map_kernel(const double *__restrict__ S, int m, int n, int32_t *__restrict__ back,
                                                                int32_t *__restrict__ f, double *__restrict__ total)
{
    __shared__ AlignShared sh;
    align_threads(S, m, n, back, f, total, sh, (int)blockDim.x >> 6);
}

// Up to 64 draft layers: lane i of one wave holds draft layer i and works on verifier layer t - i in step t, one behind its neighbour: the maximum
// over the layers before it, which that neighbour found a step ago, and its own of the verifier layer before are all it needs, so a step is one
// lane move, one sum and one maximum.  No indices are carried: a column's records, the lanes above everything before them, say where its prefix
// maxima lie (the first maximum over the lanes up to i is the last record up to i), and the way back is three scalar instructions per column.
// Bound by that serial chain of n + m - 1 steps and n columns back behind one trip to memory; the other waves only fetch.  A prefix maximum over
// the lanes per column, six dependent lane moves and maxima each / a step per diagonal, us: 32 x 48 layers 10.6 / 6.9, 32 x 80 16.7 / 8.8, 64 x 80 19.6 / 12.5, 64 x 1000 213 /
// 85, similarity and alignment of 22 x 32 layers 28.0 / 25.2; 16 x 24 and smaller, bound by the host, 6.0 both.
// S waits in LDS by steps (lane i's entry of step t is that of column t - i), so that a step's entries lie side by side.  Records: a word
// per block of 64 columns and layer; in LDS, or, where there are too many, in the workspace (an eighth of m bytes per column, of the 4 m it holds).
// A NaN, for which an order of maxima has no meaning, and entries above 1e300 beside others below -1e300, whose sums may end in one
// (infinity and -infinity; 65535 columns of less do not overflow), leave the call to the general form, by one wave.  (By all four, and with
// any entry above 1e300, us: 32 x 48 layers with an infinity 36.5 / 7.5, 64 x 1000 with a NaN 745 / 455, with both infinities 745 / 455.)
constexpr int WAVE_MOST = 64;                                  // draft layers
constexpr int WAVE_THREADS = 256, WAVE_BLOCK = 64, WAVE_RING = 2 * WAVE_BLOCK;       // steps between two fetches; steps held
constexpr int WAVE_PITCH = WAVE_MOST + 1;                      // doubles of a step (odd: a layer's columns, a step apart, fall on different banks)
constexpr int WAVE_RECORDS = MAP_LDS_BACK / 4;                 // words of records that are kept in LDS
__host__ __device__ inline int wave_records(int m, int n) { return (n + 63) / 64 * m; }
size_t wave_lds_bytes(int m, int n)
{
    const int words = wave_records(m, n);
    const size_t bytes = ((size_t)WAVE_PITCH * WAVE_RING + (words <= WAVE_RECORDS ? words : 0)) * sizeof(double);
    return bytes > sizeof(AlignShared) ? bytes : sizeof(AlignShared);
}
// Eight steps of a wave.  left: the lane before's; best = entry + own; a record (another bit of rec) where best > left; own = the larger.  Written
// out because this is the chain that a call waits for: a wave by itself issues an instruction in 4 to 8 cycles.  (The lane moves need two wait
// states behind what they read, the carry as many behind the comparison.)
__device__ __forceinline__ void diagonal_steps(double &own, double &left, uint32_t &rec, const double (&entry)[8])
{
#define SPECATTN_STEP(E) \
    "v_mov_b32_dpp v102, v100 wave_shr:1 row_mask:0xf bank_mask:0xf\n" \
    "v_mov_b32_dpp v103, v101 wave_shr:1 row_mask:0xf bank_mask:0xf\n" \
    "v_add_f64 v[104:105], " E ", v[100:101]\n" \
    "v_cmp_gt_f64 vcc, v[104:105], v[102:103]\n" \
    "v_max_f64 v[100:101], v[104:105], v[102:103]\n" \
    "s_nop 0\n" \
    "v_addc_co_u32 %2, vcc, %2, %2, vcc\n"
    asm("s_nop 1\n" SPECATTN_STEP("%3") SPECATTN_STEP("%4") SPECATTN_STEP("%5") SPECATTN_STEP("%6")
        SPECATTN_STEP("%7") SPECATTN_STEP("%8") SPECATTN_STEP("%9") SPECATTN_STEP("%10")
        : "+{v[100:101]}"(own), "+{v[102:103]}"(left), "+v"(rec)
        : "v"(entry[0]), "v"(entry[1]), "v"(entry[2]), "v"(entry[3]), "v"(entry[4]), "v"(entry[5]), "v"(entry[6]), "v"(entry[7])
        : "vcc", "v104", "v105");
#undef SPECATTN_STEP
}
__global__ __launch_bounds__(WAVE_THREADS) void layer_map_wave_kernel(const double *__restrict__ S, int m, int n, int32_t *__restrict__ back,
                                                                      int32_t *__restrict__ f, double *__restrict__ total)
{
    extern __shared__ __align__(16) double map_lds[];
    double *ring = map_lds;                                    // [WAVE_RING][WAVE_PITCH]: step t at t % WAVE_RING
    unsigned long long *records = wave_records(m, n) <= WAVE_RECORDS ? reinterpret_cast<unsigned long long *>(ring + WAVE_RING * WAVE_PITCH) : reinterpret_cast<unsigned long long *>(back);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = n + m - 1;
    constexpr int WAVES = WAVE_THREADS / 64, MOST_ROWS = WAVE_MOST / WAVES;
    // Columns a lane has not reached yet and columns past the last one count as -0.0, which leaves a lane what it has.
    auto cell = [&](int t, int i) -> double & { return ring[(t & (WAVE_RING - 1)) * WAVE_PITCH + i]; };
    for (int i = wave; i < m; i += WAVES)
        if (lane < i) cell(lane, i) = -0.0;
    double own = -0.0;                                         // maximum over the lanes up to this one, of the column the lane was at
    double left = -INFINITY;                                   // ... over the lanes before it, a step ahead; lane 0 keeps -infinity
    bool odd = false;
    // The records of a block of columns: column j0 + c of lane i was step j0 + c + i.  (Columns past the last one: none moves the way back.)
    auto keep_records = [&](int j0, unsigned long long steps0, unsigned long long steps1) {
        unsigned long long r = steps0 >> lane | (lane ? steps1 << (64 - lane) : ~0ull);        // (lane 0: always)
        if (lane == 0) r = ~0ull;
        if (n - j0 < 64) r |= ~0ull << (n - j0);
        if (lane < m) records[j0 / 64 * m + lane] = r;
    };
    unsigned long long before = 0ull;                          // records of the block of steps before
    for (int t0 = 0; t0 < steps; t0 += WAVE_BLOCK) {
        const int half = t0 & WAVE_BLOCK;
        double col[MOST_ROWS];
#pragma unroll
        for (int k = 0; k < MOST_ROWS; ++k) {
            const int i = wave + k * WAVES;
            if (i < m) col[k] = t0 + lane < n ? S[(int64_t)i * n + t0 + lane] : -0.0;
        }
#pragma unroll
        for (int k = 0; k < MOST_ROWS; ++k) {
            const int i = wave + k * WAVES;
            if (i < m) {
                cell(t0 + lane + i, i) = col[k];
                odd |= !(col[k] <= 1e300);
            }
        }
        __syncthreads();
        if (wave == 0) {
            constexpr int AHEAD = 8;
            const double *entry = ring + half * WAVE_PITCH + lane;                 // (lanes past m: nothing reads what they find)
            auto fetch = [&](double (&v)[AHEAD], int u0) {
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) v[u] = entry[(u0 + u) * WAVE_PITCH];
            };
            double cur[AHEAD], nxt[AHEAD];
            uint32_t rec[2] = {0u, 0u};                        // a bit per step, the first one highest
            fetch(cur, 0);
#pragma unroll
            for (int u0 = 0; u0 < WAVE_BLOCK; u0 += AHEAD) {
                if (t0 + u0 < steps) {                         // (uniform)
                    if (u0 + AHEAD < WAVE_BLOCK) fetch(nxt, u0 + AHEAD);
                    diagonal_steps(own, left, rec[u0 >> 5], cur);
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) cur[u] = nxt[u];
                } else {
                    rec[u0 >> 5] <<= AHEAD;
                }
            }
            const unsigned long long now = (unsigned long long)__brev(rec[1]) << 32 | __brev(rec[0]);
            if (t0) keep_records(t0 - WAVE_BLOCK, before, now);        // (complete: their last step lies at most 62 behind t0)
            if (t0 + WAVE_BLOCK >= steps && t0 < n) keep_records(t0, now, 0ull);
            before = now;
        }
        __syncthreads();
    }
    if (__syncthreads_or(odd)) {                               // (also orders the records)
        bool general = false;
        for (int e = tid; e < m * n; e += WAVE_THREADS) general |= !(S[e] >= -1e300);          // (below that, or NaN)
        if (__syncthreads_or(general)) {
            if (wave == 0) align_threads(S, m, n, back, f, total, *reinterpret_cast<AlignShared *>(map_lds), 1);
            return;
        }
    }
    if (wave) return;
    if (lane == m - 1) *total = own;
    int up = 64 - m;                                           // 63 - (the layer chosen)
    for (int j0 = (n - 1) & ~63; j0 >= 0; j0 -= 64) {
        const unsigned long long rec = lane < m ? records[j0 / 64 * m + lane] : 0ull;
        int chosen = 0;
#pragma unroll
        for (int k0 = 56; k0 >= 0; k0 -= 8) {
            if (j0 + k0 < n) {                                 // (uniform)
#pragma unroll
                for (int k = k0 + 7; k >= k0; --k) {
                    // (up = leading zeros of the records up to the layer: the next one; written out, so that scalar instructions alone write it)
                    const unsigned long long r = __ballot((uint32_t)(rec >> (k & 32)) & (1u << (k & 31)));
                    unsigned long long upto;
                    asm("s_lshr_b64 %1, -1, %0\n s_and_b64 %1, %1, %2\n s_flbit_i32_b64 %0, %1" : "+s"(up), "=&s"(upto) : "s"(r) : "scc");
                    asm("v_writelane_b32 %0, %1, %2" : "+v"(chosen) : "s"(up), "n"(k));
                }
            }
        }
        if (j0 + lane < n) f[j0 + lane] = 63 - chosen;
    }
}

// Runs of 512 or 256 entries per workgroup, and workgroups along the entries: one per CU as soon as there are that many
// runs (the LDS of eight waves allows no second).
// Few runs go out half as long: a SIMD then has one wave's logarithms and products to do instead of two.  (2 x 3 layers
// of 400 entries 10.0 us instead of 11.9, 8 x 12 of 512 9.6 and 10.9, 4 x 40 of 8192 10.9 and 14.4.)
struct KlPlan { int waves, iters, chunks, gi, gj; };
KlPlan kl_plan(int m, int n, int64_t per_layer, int64_t most_chunks)
{
    KlPlan p;
    p.gi = (m + KL_TI - 1) / KL_TI;
    p.gj = (n + KL_TJ - 1) / KL_TJ;
    int64_t run = KL_WAVES * KL_WAVE_K, want = cu_count() / ((int64_t)p.gi * p.gj);
    p.waves = KL_WAVES;
    if (2 * ((per_layer + run - 1) / run) <= want) { p.waves = KL_FEW_WAVES; run = KL_FEW_WAVES * KL_WAVE_K; }
    const int64_t runs = (per_layer + run - 1) / run;
    want = want > most_chunks ? most_chunks : want;
    want = want < 1 ? 1 : want;
    p.iters = (int)((runs + want - 1) / want);
    p.chunks = (int)((runs + p.iters - 1) / p.iters);
    return p;
}

// Chunks a call is accepted with at least: what fills the chip with one workgroup per layer pair and chunk of 4096 terms
// or more.  (A workspace between that and the full size takes fewer, longer chunks.)
int64_t kl_least_chunks(int m, int n, int64_t per_layer)
{
    const int64_t pairs = (int64_t)m * n, want = (4 * (int64_t)cu_count() + pairs - 1) / pairs, most = (per_layer + 4095) / 4096;
    const int64_t least = want < most ? want : most;
    return least < 1 ? 1 : (least > 1024 ? 1024 : least);
}

bool bad_dims(int m, int n, int rows, int L)
{
    return m <= 0 || n <= 0 || rows <= 0 || L <= 0 || (int64_t)m * n > 65535 || (int64_t)rows * L > ((int64_t)1 << 40);
}

}  // namespace

// The LDS sizes of the similarity and of the alignment in one wave, set once per device.
specattn_status layer_map_configure()
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static bool done[MAX_DEVICES] = {false};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        set_error("no current device");
        return SPECATTN_EHIP;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (done[dev]) return SPECATTN_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&layer_kl_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kl_lds_bytes(KL_WAVES)) != hipSuccess) {
        (void)hipGetLastError();
        set_error("cannot reserve %d bytes of LDS", kl_lds_bytes(KL_WAVES));
        return SPECATTN_EHIP;
    }
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&layer_map_wave_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)wave_lds_bytes(WAVE_MOST, WAVE_RECORDS / WAVE_MOST * 64)) != hipSuccess) {
        (void)hipGetLastError();
        set_error("cannot reserve %zu bytes of LDS", wave_lds_bytes(WAVE_MOST, WAVE_RECORDS / WAVE_MOST * 64));
        return SPECATTN_EHIP;
    }
    done[dev] = true;
    return SPECATTN_OK;
}

}  // namespace specattn

using namespace specattn;

extern "C" {

size_t specattn_layer_similarity_workspace_size(int32_t m, int32_t n, int32_t rows, int32_t L)
{
    if (bad_dims(m, n, rows, L)) return 0;
    const size_t bytes = (size_t)m * n * kl_plan(m, n, (int64_t)rows * L, INT64_MAX).chunks * sizeof(double);
    return (bytes + 255) & ~(size_t)255;
}

specattn_status specattn_layer_similarity(const float *attn_draft, const float *attn_verifier, int32_t m, int32_t n,
                                          int32_t rows, int32_t L, double *S, void *workspace, size_t workspace_bytes,
                                          void *stream)
{
    clear_error();
    if (!attn_draft || !attn_verifier || !S) { set_error("attn_draft, attn_verifier and S must not be NULL"); return SPECATTN_EINVAL; }
    if (m <= 0 || n <= 0 || rows <= 0 || L <= 0) { set_error("m, n, rows and L must be positive"); return SPECATTN_EINVAL; }
    if (bad_dims(m, n, rows, L)) { set_error("at most 65535 layer pairs and 2^40 entries per layer"); return SPECATTN_ESHAPE; }
    const int pairs = m * n;
    const int64_t per_layer = (int64_t)rows * L, least = kl_least_chunks(m, n, per_layer);
    size_t need = specattn_layer_similarity_workspace_size(m, n, rows, L);
    const size_t least_bytes = ((size_t)pairs * least * sizeof(double) + 255) & ~(size_t)255;
    need = need < least_bytes ? need : least_bytes;
    if (!workspace) { set_error("workspace is NULL, %zu bytes needed", need); return SPECATTN_EWORKSPACE; }
    if (reinterpret_cast<uintptr_t>(workspace) % 256) { set_error("workspace must be 256-byte aligned"); return SPECATTN_EWORKSPACE; }
    if (workspace_bytes < need) { set_error("workspace has %zu bytes, %zu needed", workspace_bytes, need); return SPECATTN_EWORKSPACE; }
    const KlPlan plan = kl_plan(m, n, per_layer, (int64_t)(workspace_bytes / ((size_t)pairs * sizeof(double))));
    specattn_status st = layer_map_configure();
    if (st != SPECATTN_OK) return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    double *partial = static_cast<double *>(workspace);
    hipLaunchKernelGGL(layer_kl_kernel, dim3(plan.chunks, plan.gi, plan.gj), dim3(plan.waves * 64), kl_lds_bytes(plan.waves), hs, attn_draft, attn_verifier,
                       m, n, per_layer, plan.iters, partial);
    st = check_launch("layer_kl_kernel");
    if (st != SPECATTN_OK) return st;
    hipLaunchKernelGGL(layer_kl_finish_kernel, dim3((pairs + 7) / 8), dim3(512), 0, hs, partial, m, n, plan.chunks, (double)rows,
                       attn_draft, attn_verifier, per_layer, S);
    return check_launch("layer_kl_finish_kernel");
}

size_t specattn_layer_map_workspace_size(int32_t m, int32_t n)
{
    if (m <= 0 || n <= 0 || m > MAP_THREADS || n > 65535) return 0;
    return (((size_t)m * n * sizeof(int32_t)) + 255) & ~(size_t)255;
}

specattn_status specattn_layer_map(const double *S, int32_t m, int32_t n, int32_t *f, double *total, void *workspace,
                                   size_t workspace_bytes, void *stream)
{
    clear_error();
    if (!S || !f || !total) { set_error("S, f and total must not be NULL"); return SPECATTN_EINVAL; }
    if (m <= 0 || n <= 0) { set_error("m and n must be positive"); return SPECATTN_EINVAL; }
    if (m > MAP_THREADS || n > 65535) { set_error("at most %d draft layers and 65535 verifier layers", MAP_THREADS); return SPECATTN_ESHAPE; }
    const size_t need = specattn_layer_map_workspace_size(m, n);
    if (!workspace) { set_error("workspace is NULL, %zu bytes needed", need); return SPECATTN_EWORKSPACE; }
    if (reinterpret_cast<uintptr_t>(workspace) % 256) { set_error("workspace must be 256-byte aligned"); return SPECATTN_EWORKSPACE; }
    if (workspace_bytes < need) { set_error("workspace has %zu bytes, %zu needed", workspace_bytes, need); return SPECATTN_EWORKSPACE; }
    hipStream_t hs = static_cast<hipStream_t>(stream);
    int32_t *back = static_cast<int32_t *>(workspace);
    if (m <= WAVE_MOST) {
        const specattn_status st = layer_map_configure();
        if (st != SPECATTN_OK) return st;
        hipLaunchKernelGGL(layer_map_wave_kernel, dim3(1), dim3(WAVE_THREADS), wave_lds_bytes(m, n), hs, S, m, n, back, f, total);
    } else {
        hipLaunchKernelGGL(layer_map_kernel, dim3(1), dim3((m + 63) / 64 * 64), 0, hs, S, m, n, back, f, total);
    }
    return check_launch("layer_map_kernel");
}

}  // extern "C"
