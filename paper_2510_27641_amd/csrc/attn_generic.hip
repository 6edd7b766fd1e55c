// Sparse decode attention over a selected index list (Section 3.1.2, Eq. 2-3; Section 3.5): the variant that
// computes both contractions in fp32, for every element type - fp32 inputs, and what the 16-bit matrix-core kernel
// does not take (more than 512 kv heads; at d = 64 short lists, workspaces too small for its partials and strides beyond its offsets).
//
// Work split: one workgroup of eight waves per (row, split); a split is a contiguous run of the row's kept positions
// and tile k of 16 positions goes to wave k mod 8.  Each wave keeps the running softmax state (max m, sum l,
// un-normalised output o) of all G*T query rows of the kv head; the eight states are combined in LDS in wave order.
// A row with one split is finished there; otherwise the split leaves one partial (m, l, o) and merge_kernel combines
//   O = sum_s 2^(m_s - m) o_s / sum_s 2^(m_s - m) l_s,  lse = ln 2 * (m + log2(sum_s 2^(m_s - m) l_s)).
//
// Both products run on the fp32 matrix cores (v_mfma_f32_16x16x4: full fp32 operands and sums, the rate of the vector
// ALU but one operand fetch per 16 products), with no layout change anywhere between memory and the cores:
//   S^T = K Q^T   : lane (p = lane % 16, g = lane / 16) loads elements 16j + 4g .. + 3 of key p with one 16-byte load
//                   (64 contiguous bytes of each of 16 rows per instruction); k-step (j, i) contracts the elements
//                   16j + 4g + i, an order of the head dimension that the Q fragments share.
//   O^T += V^T P^T: lane (m = lane % 16, g) loads elements 4m .. 4m + 3 of value row 4g + c - four whole rows per
//                   instruction - and component i is row m of the output tile of dv = 4m + i.  The weights of positions
//                   4g + c are what the score product left in this very lane.
// What bounds it: small calls, latency (list word -> K and V rows -> eight states); large ones, HBM or, from two
// query tiles on, the fp32 matrix rate.  The kernel before it fed the vector ALU from LDS, four barriers per 32 positions:
// selection and attention of 8 rows of 1024 positions (d = 64, 5 tokens) 26.9 us then, 13.9 us now (12.5 with the
// selection as it has become); 32 rows of 424 (d =
// 128, 28 query rows) 67 and 22 us; 8 rows of 5039 (d = 64) 54 and 22 us; error against 64 bits 2.4e-7 .. 4.5e-7 then,
// 1.7e-7 .. 2.7e-7 now.
#include "common.h"

#include <algorithm>
#include <mutex>

namespace specattn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int GEN_WAVES = 8;
constexpr int GEN_THREADS = GEN_WAVES * 64;
constexpr int GEN_TILE = 16;          // positions
constexpr int MAX_QT = 64;            // G*T query rows per kv head handled here
constexpr float RESCALE_SLACK = 8.0f; // log2 units the running max may exceed the reference by

// four consecutive elements as fp32
template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ f32x4 ld4(const void *p, int64_t i) { return *reinterpret_cast<const f32x4 *>(static_cast<const float *>(p) + i); }
};
template <> struct Elem<_Float16> {
    static __device__ __forceinline__ f32x4 ld4(const void *p, int64_t i)
    {
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        return __builtin_convertvector(*reinterpret_cast<const f16x4 *>(static_cast<const _Float16 *>(p) + i), f32x4);
    }
};
template <> struct Elem<uint16_t> {   // bf16
    static __device__ __forceinline__ f32x4 ld4(const void *p, int64_t i)
    {
        const uint2 u = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(p) + i);
        return (f32x4){__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u)};
    }
};

// element offset of position/slot `idx` of (b, h) inside k or v
struct KvMap {
    int64_t base;            // b / h part (contiguous) or h part (paged)
    int64_t stride_n, stride_page;
    const int32_t *ptab;     // this sequence's page table row, or null
    int page_shift;
    bool physical;
    template <bool PLAIN> __device__ __forceinline__ int64_t off(int idx) const
    {
        if (PLAIN || (!ptab && !physical)) return base + (int64_t)idx * stride_n;
        const int mask = (1 << page_shift) - 1;
        const int page = physical ? (idx >> page_shift) : ptab[idx >> page_shift];
        return base + (int64_t)page * stride_page + (int64_t)(idx & mask) * stride_n;
    }
};

template <bool PLAIN> __device__ __forceinline__ KvMap make_map(const AttnLaunch &a, int b, int h)
{
    KvMap m;
    const bool paged = !PLAIN && (a.page_table != nullptr || a.indices_are_physical);
    m.base = paged ? (int64_t)h * a.kv_stride_h : (int64_t)b * a.kv_stride_b + (int64_t)h * a.kv_stride_h;
    m.stride_n = a.kv_stride_n;
    m.stride_page = a.kv_stride_page;
    m.ptab = (a.page_table && !a.indices_are_physical) ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    m.page_shift = a.page_shift;
    m.physical = a.indices_are_physical != 0;
    return m;
}

// LDS, in floats: the Q tile and a state of every wave for one query tile, rows padded by one 16-byte chunk so that
// 16 rows at one column fall on different banks; (m, l) of every wave and query row; scores of the new tokens.
template <int D> struct Lds {
    static constexpr int ROW = D + 4;
    static constexpr int q_floats(int nqt) { return nqt * 16 * ROW; }
    static constexpr int O_FLOATS = GEN_WAVES * 16 * ROW;
    static constexpr int ML_FLOATS = GEN_WAVES * MAX_QT * 2;
    static constexpr int TAIL_FLOATS = MAX_QT * SPECATTN_MAX_T;
    static constexpr size_t bytes(int nqt) { return sizeof(float) * (size_t)(q_floats(nqt) + O_FLOATS + ML_FLOATS + TAIL_FLOATS); }
};

struct F32Plan {
    int n_splits, group;          // splits of a row; query heads per kv head
    FastDivisor per_split, per_h;
    uint32_t per_t;               // 2^16 / T, rounded up: q / T for q < 2^12, T < 2^4
    float *part_o, *part_ml;
};

// PLAIN: contiguous keys and values, lists of single positions, no new tokens.  A launch starts with cold instruction caches, and what it does not
// need is jumped over and held in registers all the same.  One form for all calls / two, us: selection and attention of 8 rows of 1024 11.4 / 10.8;
// attention of 8 rows of 8192 11.4 / 10.9, 32 of 6000 with 32 query rows (d = 128) 27.8 / 26.1, 16 of 4000 with 6 (d = 128) 10.5 / 9.7.
// Not with four query tiles of 128: either form spills there, this one 112 bytes per lane, the other 84.  PLAIN / the other, attention alone: 64 query
// rows, 8 rows of 512 kept positions 22.9 / 22.5, 16 of 1024 28.3 / 27.2, 64 of 320 47.3 / 45.6, 8 of 4000 56.7 / 54.3; but three tiles 17.0 / 17.5, and
// four of 64 (16 of 1024) 31.4 / 31.9.
constexpr bool plain_form(int d, int nqt) { return !(d == 128 && nqt == 4); }
// Two workgroups to a CU where 128 registers will do (d = 64, up to two query tiles): the form for single positions took 132 for two tiles, and with one
// workgroup 64 rows of 600 kept positions of 2000 with 32 query rows 17.1 us instead of 13.9, of 1500 of 6000 (32 rows) 18.1 instead of 16.0.
template <typename T, int D, int NQT, bool PLAIN>
__global__ __launch_bounds__(GEN_THREADS, D == 64 && NQT <= 2 ? 4 : 1) void attn_f32_kernel(AttnLaunch a, F32Plan plan)
{
    SPECATTN_PRELOAD(a.q); SPECATTN_PRELOAD(a.k); SPECATTN_PRELOAD(a.v); SPECATTN_PRELOAD(a.H_q); SPECATTN_PRELOAD(a.H_kv); SPECATTN_PRELOAD(a.T);
    SPECATTN_PRELOAD(a.sm_scale); SPECATTN_PRELOAD(a.q_stride_b); SPECATTN_PRELOAD(a.q_stride_h); SPECATTN_PRELOAD(a.q_stride_t); SPECATTN_PRELOAD(a.kv_stride_b);
    SPECATTN_PRELOAD(a.kv_stride_h); SPECATTN_PRELOAD(a.kv_stride_n); SPECATTN_PRELOAD(a.indices);
    SPECATTN_PRELOAD(a.idx_stride); SPECATTN_PRELOAD(a.counts); SPECATTN_PRELOAD(a.idx_capacity);
    SPECATTN_PRELOAD(a.out); SPECATTN_PRELOAD(a.out_lowp); SPECATTN_PRELOAD(a.lse);
    if (!PLAIN) {
        SPECATTN_PRELOAD(a.n_max); SPECATTN_PRELOAD(a.page_table); SPECATTN_PRELOAD(a.page_shift); SPECATTN_PRELOAD(a.indices_are_physical); SPECATTN_PRELOAD(a.dense);
        SPECATTN_PRELOAD(a.chunk_shift); SPECATTN_PRELOAD(a.k_new); SPECATTN_PRELOAD(a.seq_lens);
    }
    SPECATTN_PRELOAD(plan.n_splits); SPECATTN_PRELOAD(plan.per_split.mul); SPECATTN_PRELOAD(plan.per_split.shift); SPECATTN_PRELOAD(plan.per_h.mul);
    SPECATTN_PRELOAD(plan.per_h.shift); SPECATTN_PRELOAD(plan.group); SPECATTN_PRELOAD(plan.per_t); SPECATTN_PRELOAD(plan.part_o); SPECATTN_PRELOAD(plan.part_ml);
    extern __shared__ __attribute__((aligned(16))) float smem[];
    typedef Lds<D> L;
    constexpr int KJ = D / 16;            // 16-byte loads per key and lane
    constexpr int DH = D / 64;            // value loads per row and lane
    float *Qs = smem;
    float *Os = Qs + L::q_floats(NQT);
    float *ml = Os + L::O_FLOATS;         // [wave][query row][2]
    float *tail = ml + L::ML_FLOATS;      // [query row][new token]

    const int n_splits = plan.n_splits;
    const int r = plan.per_split.divide(blockIdx.x), s = blockIdx.x - r * n_splits;
    const int b = plan.per_h.divide(r), h = r - b * a.H_kv;
    const int G = plan.group, QT = G * a.T;
    auto head_of = [&](int q) { return (int)(((uint32_t)q * plan.per_t) >> 16); };      // q / T
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const float scale2 = a.sm_scale * 1.4426950408889634f;            // scores in log2 units
    // Q first: it waits for nothing but the arguments, and loads come back in order.  (Behind the first keys and values, with arguments in several
    // turns and divisions / now, us with the selection: 8 rows of 1024 11.8 / 11.7, of 1024 with d = 128 14.8 / 14.2, 32 of 8192 with 32 query rows
    // 26.4 / 25.1, 16 of 8192 with d = 128 and 24 query rows 34.2 / 32.1.  The barrier behind the loads instead: 32 of 2000 15.5 / 16.0.)
    constexpr int Q_PER = (NQT * 16 * (D / 4) + GEN_THREADS - 1) / GEN_THREADS;
    f32x4 qv[Q_PER];
#pragma unroll
    for (int k = 0; k < Q_PER; ++k) {
        const int e = k * GEN_THREADS + tid, qi = e / (D / 4), ch = e - qi * (D / 4);
        qv[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (qi < QT) {
            const int gh = head_of(qi), tt = qi - gh * a.T;
            qv[k] = Elem<T>::ld4(a.q, (int64_t)b * a.q_stride_b + (int64_t)(h * G + gh) * a.q_stride_h + (int64_t)tt * a.q_stride_t + 4 * ch);
        }
    }
    const int count = PLAIN ? min(max(a.counts[r], 0), a.idx_capacity) : attn_row_count(a, r, b);
    const int tiles = (count + GEN_TILE - 1) / GEN_TILE;
    const int per = (tiles + n_splits - 1) / n_splits;
    const int t_end = (s + 1) * per < tiles ? (s + 1) * per : tiles;
    const int32_t *idx = !PLAIN && a.dense ? nullptr : a.indices + (int64_t)r * a.idx_stride;
    const KvMap map = make_map<PLAIN>(a, b, h);

    // Element offset of the position whose key this lane helps to load; ranks past the end repeat the last one.
    auto tile_off = [&](int t) -> int64_t {
        const int jj = t * GEN_TILE + l16, rank = jj < count ? jj : count - 1;
        return map.off<PLAIN>(PLAIN ? idx[rank] : attn_list_pos(a, idx, rank));
    };
    f32x4 kf[KJ], vf[4][DH];
    auto load_k = [&](int64_t off) {
#pragma unroll
        for (int j = 0; j < KJ; ++j) kf[j] = Elem<T>::ld4(a.k, off + 16 * j + 4 * g);
    };
    auto load_v = [&](int64_t off) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t row = __shfl(off, 4 * g + c, 64);
#pragma unroll
            for (int u = 0; u < DH; ++u) vf[c][u] = Elem<T>::ld4(a.v, row + 64 * u + 4 * l16);
        }
    };
    int t = s * per + wave;
    int64_t off_next = 0;
    int64_t off = 0;
    if (t < t_end) off = tile_off(t);
#pragma unroll
    for (int k = 0; k < Q_PER; ++k) {
        const int e = k * GEN_THREADS + tid, qi = e / (D / 4), ch = e - qi * (D / 4);
        if (e < NQT * 16 * (D / 4)) *reinterpret_cast<f32x4 *>(Qs + qi * L::ROW + 4 * ch) = qv[k];
    }
    // Q and the list words have arrived, also for threads without a part of Q.  The compiler only sees that those have not waited, takes the
    // registers that the first keys share with Q for still on their way, and waits for the values as well ahead of every tile's scores.
    // (Without / with, us: 8 query rows and more of d = 64 in the form for all calls, 64 dense rows of 2000 29.3 / 27.0, 128 rows of 2000 in chunks
    // 14.7 / 13.4, with new tokens 16.6 / 15.0.)
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __syncthreads();                      // (ahead of the loads of keys and values: all waves' start together)
    if (t < t_end) {
        load_k(off);
        load_v(off);
        if (t + GEN_WAVES < t_end) off_next = tile_off(t + GEN_WAVES);
    }

    f32x4 o[NQT][DH][4];                  // [query tile][64 u +][i]: dv = 64 u + 16 g + 4 x + i in component x
    float m_ref[NQT], l_sum[NQT];
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        m_ref[qt] = -INFINITY;
        l_sum[qt] = 0.0f;
#pragma unroll
        for (int u = 0; u < DH; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[qt][u][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    int q_at = l16 * L::ROW + 4 * g;
    // Scores of the 16 positions in kf against query tile qt: lane (q = l16, g) gets positions 4 g + i.  (Two chains:
    // half the depth of dependent products, and of rounded sums.)
    auto scores = [&](int qt) -> f32x4 {
        f32x4 acc[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const f32x4 qf = *reinterpret_cast<const f32x4 *>(Qs + q_at + qt * 16 * L::ROW + 16 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][i], qf[i], acc[i & 1], 0, 0, 0);
        }
        return acc[0] + acc[1];
    };
    for (; t < t_end; t += GEN_WAVES) {
        asm volatile("" : "+v"(q_at));    // (Q is read from LDS again for every tile: held, it would spill)
        const bool has_next = t + GEN_WAVES < t_end;
        const int remaining = count - t * GEN_TILE;
        f32x4 p[NQT];
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) p[qt] = scores(qt);
        const int64_t off = off_next;
        if (has_next) {                   // (uniform) the key registers are free again
            load_k(off);
            if (t + 2 * GEN_WAVES < t_end) off_next = tile_off(t + 2 * GEN_WAVES);
        }
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            f32x4 x = p[qt];
            if (remaining < GEN_TILE) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * g + i >= remaining) x[i] = -INFINITY;
            }
            const float mloc = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])) * scale2;
            if (__any(mloc > m_ref[qt] + RESCALE_SLACK)) {             // first tile, then rare
                float mx = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                const float mnew = fmaxf(m_ref[qt], mx);
                const float alpha = (m_ref[qt] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m_ref[qt] - mnew);
                l_sum[qt] *= alpha;
#pragma unroll
                for (int u = 0; u < DH; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[qt][u][i] *= alpha;
                m_ref[qt] = mnew;
            }
            const float mr = (m_ref[qt] == -INFINITY) ? 0.0f : m_ref[qt];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                p[qt][i] = __builtin_amdgcn_exp2f(fmaf(x[i], scale2, -mr));
                l_sum[qt] += p[qt][i];
            }
        }
        if (remaining < GEN_TILE) {       // a weight of zero must not meet an infinite value
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int u = 0; u < DH; ++u)
                    if (4 * g + c >= remaining) vf[c][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int u = 0; u < DH; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int qt = 0; qt < NQT; ++qt)
                        o[qt][u][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][u][i], p[qt][c], o[qt][u][i], 0, 0, 0);
        if (has_next) load_v(off);
    }

    // ---- scores of the new tokens behind the cache (first split): wave qt takes query tile qt ----------------
    const bool with_tail = !PLAIN && a.k_new != nullptr && s == 0;     // uniform
    const int64_t noff = ((int64_t)b * a.H_kv + h) * a.T * D;
    if (with_tail && wave < NQT) {
        const int row = l16 < a.T ? l16 : a.T - 1;
#pragma unroll
        for (int j = 0; j < KJ; ++j) kf[j] = Elem<T>::ld4(a.k_new, noff + (int64_t)row * D + 16 * j + 4 * g);
        const f32x4 x = scores(wave);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * g + i < a.T) tail[(wave * 16 + l16) * SPECATTN_MAX_T + 4 * g + i] = x[i] * scale2;
    }

    // ---- combine the eight states, one query tile per round ---------------------------------------------------
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        float l = l_sum[qt];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (g == 0) {
            ml[(wave * MAX_QT + qt * 16 + l16) * 2] = m_ref[qt];
            ml[(wave * MAX_QT + qt * 16 + l16) * 2 + 1] = l;
        }
        if (qt) __syncthreads();          // the round before has been read out
#pragma unroll
        for (int u = 0; u < DH; ++u)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                *reinterpret_cast<f32x4 *>(Os + (wave * 16 + l16) * L::ROW + 64 * u + 16 * g + 4 * x) =
                    (f32x4){o[qt][u][0][x], o[qt][u][1][x], o[qt][u][2][x], o[qt][u][3][x]};
        __syncthreads();
        const int ql = tid / (D / 4), dv = 4 * (tid & (D / 4 - 1)), q = qt * 16 + ql;
        if (ql < 16 && q < QT) {
            const int gh = head_of(q), tt = q - gh * a.T;
            float m = -INFINITY;
#pragma unroll
            for (int w = 0; w < GEN_WAVES; ++w) m = fmaxf(m, ml[(w * MAX_QT + q) * 2]);
            if (with_tail)
                for (int p = 0; p <= tt; ++p) m = fmaxf(m, tail[q * SPECATTN_MAX_T + p]);
            f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
            float lt = 0.0f;
#pragma unroll
            for (int w = 0; w < GEN_WAVES; ++w) {
                const float mw = ml[(w * MAX_QT + q) * 2];
                const float f = (mw == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mw - m);
                lt += f * ml[(w * MAX_QT + q) * 2 + 1];
                acc += f * *reinterpret_cast<const f32x4 *>(Os + (w * 16 + ql) * L::ROW + dv);
            }
            if (with_tail)
                for (int p = 0; p <= tt; ++p) {
                    const float f = __builtin_amdgcn_exp2f(tail[q * SPECATTN_MAX_T + p] - m);
                    lt += f;
                    acc += f * Elem<T>::ld4(a.v_new, noff + (int64_t)p * D + dv);
                }
            if (n_splits == 1) {
                const int64_t orow = ((int64_t)b * a.H_q + (h * G + gh)) * a.T + tt;
                const f32x4 res = lt > 0.0f ? acc / lt : (f32x4){0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<f32x4 *>(a.out + orow * D + dv) = res;
                if (a.out_lowp) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) st_lowp(a.out_lowp, orow * D + dv + i, res[i], a.dtype);
                }
                if (a.lse && dv == 0) a.lse[orow] = lt > 0.0f ? (m + log2f(lt)) * 0.6931471805599453f : -INFINITY;
            } else {
                const int64_t slot = ((int64_t)r * n_splits + s) * QT + q;
                *reinterpret_cast<f32x4 *>(plan.part_o + slot * D + dv) = acc;
                if (dv == 0) { plan.part_ml[2 * slot] = m; plan.part_ml[2 * slot + 1] = lt; }
            }
        }
    }
}

// One workgroup per (row, query row): combine the partials of all splits in split order, eight per round trip.
__global__ void merge_kernel(AttnLaunch a, int n_splits, const float *part_o, const float *part_ml)
{
    const int G = a.H_q / a.H_kv;
    const int QT = G * a.T;
    const int r = blockIdx.x / QT, qi = blockIdx.x - r * QT;
    const int b = r / a.H_kv, h = r - b * a.H_kv;
    const int D = a.d, dv = threadIdx.x;
    float m = -INFINITY, l = 0.0f, o = 0.0f;
    for (int s0 = 0; s0 < n_splits; s0 += 8) {
        float ms[8], ls[8], os[8], mx = m;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool ok = s0 + k < n_splits;
            const int64_t slot = ((int64_t)r * n_splits + (ok ? s0 + k : 0)) * QT + qi;
            ms[k] = ok ? part_ml[2 * slot] : -INFINITY;
            ls[k] = ok ? part_ml[2 * slot + 1] : 0.0f;
            os[k] = ok ? part_o[slot * D + dv] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) mx = fmaxf(mx, ms[k]);
        const float fa = (m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m - mx);
        l *= fa;
        o *= fa;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float f = (ms[k] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(ms[k] - mx);
            l += f * ls[k];
            o += f * os[k];
        }
        m = mx;
    }
    const int g = qi / a.T, t = qi - g * a.T;
    const int64_t orow = ((int64_t)b * a.H_q + (h * G + g)) * a.T + t;
    const float res = l > 0.0f ? o / l : 0.0f;
    a.out[orow * D + dv] = res;
    if (a.out_lowp) st_lowp(a.out_lowp, orow * D + dv, res, a.dtype);
    if (a.lse && dv == 0) a.lse[orow] = l > 0.0f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

template <typename T, int D, bool PLAIN> const void *variant(int nqt)
{
    switch (nqt) {
    case 1: return reinterpret_cast<const void *>(&attn_f32_kernel<T, D, 1, PLAIN>);
    case 2: return reinterpret_cast<const void *>(&attn_f32_kernel<T, D, 2, PLAIN>);
    case 3: return reinterpret_cast<const void *>(&attn_f32_kernel<T, D, 3, PLAIN>);
    case 4: return reinterpret_cast<const void *>(&attn_f32_kernel<T, D, 4, PLAIN && plain_form(D, 4)>);
    }
    return nullptr;
}
template <bool PLAIN> const void *variant(int dtype, int d, int nqt)
{
    if (d != 64 && d != 128) return nullptr;
    if (dtype == SPECATTN_F32) return d == 64 ? variant<float, 64, PLAIN>(nqt) : variant<float, 128, PLAIN>(nqt);
    if (dtype == SPECATTN_BF16) return d == 64 ? variant<uint16_t, 64, PLAIN>(nqt) : variant<uint16_t, 128, PLAIN>(nqt);
    if (dtype == SPECATTN_F16) return d == 64 ? variant<_Float16, 64, PLAIN>(nqt) : variant<_Float16, 128, PLAIN>(nqt);
    return nullptr;
}
size_t lds_bytes(int d, int nqt) { return d == 64 ? Lds<64>::bytes(nqt) : Lds<128>::bytes(nqt); }
static_assert(Lds<128>::bytes(4) <= 160 * 1024, "the tables must fit");

// Splits of a row in this kernel, never more than attn_num_splits (which sizes the workspace).  A row whose list is
// short is finished by one workgroup: the second launch costs more (4.5 us) than the rounds saved, a round of eight
// tiles being about a microsecond of latency per query tile and 64 elements of head dimension.  The line, both sides
// measured: 12 rows of 1214 (d = 64) 16.4 us with one split and 18.5 us with several, 32 rows of 1948 (d = 64) 17.0
// and 18.7 us, but 32 rows of 1617 (d = 128, two query tiles) 31 and 22 us.  Otherwise two workgroups per CU, which evens
// out rows of different counts.
int splits(int rows, int capacity, int nqt, int d)
{
    if ((int64_t)capacity * nqt * (d / 64) <= 2048) return 1;
    const int most = attn_num_splits(rows, capacity), want = (2 * cu_count() + rows - 1) / rows;
    return want < most ? want : most;
}

}  // namespace

// The LDS size of every variant, set once per device (not on a variant's first launch: a first call may be
// recorded in a graph, and a process may use several devices).
specattn_status attn_generic_configure()
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
    for (int k = 0; k < 3 * 2 * 4; ++k) {
        const int dtype = k % 3, d = k / 3 % 2 ? 128 : 64, nqt = k / 6 + 1;
        for (const void *fn : {variant<false>(dtype, d, nqt), variant<true>(dtype, d, nqt)})
            if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes(d, nqt)) != hipSuccess) {
                (void)hipGetLastError();
                set_error("cannot reserve %zu bytes of LDS", lds_bytes(d, nqt));
                return SPECATTN_EHIP;
            }
    }
    done[dev] = true;
    return SPECATTN_OK;
}

int attn_num_splits(int rows, int idx_capacity)
{
    const int want = 4 * cu_count();                          // workgroups in flight to aim for
    int s = (want + rows - 1) / rows;
    const int max_s = (idx_capacity + 255) / 256;             // at least 256 positions per split
    if (s > max_s) s = max_s;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    return s;
}

static size_t generic_bytes(int rows, int G, int T, int d, int idx_capacity)
{
    const size_t ns = (size_t)attn_num_splits(rows, idx_capacity);
    const size_t bytes = (size_t)rows * ns * (size_t)G * T * (size_t)(d + 2) * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}
// the 16-bit variant may take any shape (the size does not depend on the element type)
size_t attn_workspace_bytes(int rows, int G, int T, int d, int idx_capacity)
{
    return std::max(generic_bytes(rows, G, T, d, idx_capacity), attn_mfma_workspace_bytes(rows, G, T, d));
}
size_t attn_workspace_min_bytes(int rows, int G, int T, int d, int idx_capacity)
{
    return std::max(generic_bytes(rows, G, T, d, idx_capacity), attn_mfma_workspace_min_bytes(rows, G, T, d));
}
size_t attn_workspace_accepted_bytes(int rows, int G, int T, int d, int idx_capacity)
{
    const size_t bytes = generic_bytes(rows, G, T, d, idx_capacity);
    return d == 64 ? bytes : std::max(bytes, attn_mfma_workspace_narrow_bytes(rows, G, T, d));
}

// d = 64 on the 16-bit kernel: its partials have to fit the workspace (a call is accepted with one that holds this file's
// partials only), and the row offsets 32 bits: in pools in units of 128 bytes, contiguous rows in units of 16.  Lists of at most
// 128 positions are finished here, by one workgroup per row in one launch (us, 16-bit kernel / here, without and with new tokens:
// 8 rows of 128 with 20 query rows 10.6 / 8.2 and 14.8 / 9.9, 1024 rows of 20 with 4 20.4 / 8.6 and 25.0 / 10.3, of 128 22.0 / 15.4
// and 26.9 / 16.9; 64 rows with 64 query rows, of 128 13.6 / 13.0 and 21.3 / 17.5, but of 256 13.8 / 18.3 without new tokens).
constexpr int SHORT_64 = 128;
static bool attn_mfma_takes_64(const AttnLaunch &a)
{
    if (((int64_t)a.idx_capacity << a.chunk_shift) <= SHORT_64) return false;
    if (a.workspace_bytes < attn_mfma_workspace_min_bytes(a.B * a.H_kv, a.H_q / a.H_kv, a.T, a.d)) return false;
    if (a.page_table || a.indices_are_physical) return a.kv_stride_n % 64 == 0 && a.kv_stride_page % 64 == 0;
    return a.kv_stride_n <= ((int64_t)1 << 35) / a.n_max;
}

specattn_status launch_attn(const AttnLaunch &a, hipStream_t stream)
{
    const int rows = a.B * a.H_kv;
    const int G = a.H_q / a.H_kv;
    if (attn_mfma_supported(a) && (a.d == 128 || attn_mfma_takes_64(a))) return launch_attn_mfma(a, stream);
    const int QT = G * a.T, nqt = (QT + 15) / 16;
    int ns = splits(rows, a.idx_capacity << a.chunk_shift, nqt, a.d);
    const bool plain = plain_form(a.d, nqt) && !a.dense && !a.chunk_shift && !a.page_table && !a.indices_are_physical && !a.k_new;
    const void *fn = plain ? variant<true>(a.dtype, a.d, nqt) : variant<false>(a.dtype, a.d, nqt);
    if (!fn) { set_error("no attention kernel for dtype %d, d %d", a.dtype, a.d); return SPECATTN_EUNSUPPORTED; }
    specattn_status st = attn_generic_configure();
    if (st != SPECATTN_OK) return st;
    float *part_o = static_cast<float *>(a.workspace);
    float *part_ml = part_o + (size_t)rows * ns * QT * a.d;
    F32Plan plan{ns, G, FastDivisor(ns), FastDivisor(a.H_kv), (65536u + a.T - 1) / a.T, part_o, part_ml};
    void *kargs[] = {const_cast<AttnLaunch *>(&a), &plan};
    if (hipLaunchKernel(fn, dim3(rows * ns), dim3(GEN_THREADS), kargs, lds_bytes(a.d, nqt), stream) != hipSuccess) {
        set_error("attn_f32_kernel: launch failed");
        (void)hipGetLastError();
        return SPECATTN_EHIP;
    }
    st = check_launch("attn_f32_kernel");
    if (st != SPECATTN_OK || ns == 1) return st;
    hipLaunchKernelGGL(merge_kernel, dim3(rows * QT), dim3(a.d), 0, stream, a, ns, part_o, part_ml);
    return check_launch("merge_kernel");
}

}  // namespace specattn
