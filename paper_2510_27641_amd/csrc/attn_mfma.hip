// Host side of the matrix-core attention route and the merge of its partials; the kernel itself is in
// attn_mfma_kernel.h, its variants in four translation units of their own.
#include "attn_mfma_kernel.h"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace specattn {
namespace {

// Sum of v over the wave, in every lane.
__device__ __forceinline__ float wave_sum(float v)
{
#define SPECATTN_SUM_STEP(CTRL, RM) v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, RM, 0xf, false))
    SPECATTN_SUM_STEP(0x111, 0xf);    // row_shr:1
    SPECATTN_SUM_STEP(0x112, 0xf);    // row_shr:2
    SPECATTN_SUM_STEP(0x114, 0xf);    // row_shr:4
    SPECATTN_SUM_STEP(0x118, 0xf);    // row_shr:8
    SPECATTN_SUM_STEP(0x142, 0xa);    // row_bcast:15 into rows 1 and 3
    SPECATTN_SUM_STEP(0x143, 0xc);    // row_bcast:31 into rows 2 and 3
#undef SPECATTN_SUM_STEP
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 63));
}

// What the merge needs of a launch only in the end; with the new tokens, also what those need.  What its first requests need are the
// leading arguments, scalars of 14 words in all: those come in registers with the launch (the build asks for it), without a trip to memory.
// All arguments from memory in one batch / so, us, with what goes before: 8 rows of 8192 19.3 / 19.1, 64 of 13001 (40 query rows each)
// 45.2 / 44.6, 16 layers of 64 rows of 32768 776.5 / 772.8.  (The main kernel's arguments the same way, with the counts requested ahead of
// the rest: 8 rows of 8192 19.5 / 19.8, 16 layers 778 / 784.)
struct MergeArgs {
    float *out, *lse;
    void *out_lowp;
    // the new tokens behind the cache
    float sm_scale;
    const uint16_t *q, *k_new, *v_new;
    int64_t q_stride_b, q_stride_h, q_stride_t;
};

// After the main kernel, one workgroup per (query row, row): rows shared by several workgroups get
// their partials (r, w) combined; rows without any kept position get out = 0, lse = -inf.  When the
// caller gave the new tokens behind the cache (TAIL), every row goes through here (the main kernel then
// leaves partials only) and query t also attends to new tokens 0..t.
// Bound by latency: the row's shares, then a trip to memory and two chains of sums per sixteen partials.  Head dimension and element type
// are constants, the host hands divisors over as reciprocals, and every load of a trip is requested before the first partial is used; a
// short rest asks for two, five or eight, since sixteen are a chain too long there (rows of 9 to 16 parts in two trips of eight / one: 8
// rows of 8192 19.2 / 19.0 us).  What the new tokens need is requested ahead of the shares, in one go (with the element type tested at each
// of those loads, one waited for the other, and partials joined one by one: 32 rows of 2044 in chunks with new tokens 20.0 / 17.7).
// A partial's (m, l) is the same for all threads, so the compiler takes scalar loads for it: eight of them, which come back in any order
// and are waited for together, cost 0.12 us more per trip than vector loads that are asked for ahead of the outputs (one row of 270 tiles
// among 31 empty ones, 268 partials, 31.3 / 27.2 us; over 440 calls of few rows 4 % on average, none slower).
template <int D, bool F16, bool TAIL>
__global__ __launch_bounds__(D) void merge_partials_kernel(const uint32_t *row_parts, const float *part_ml, const float *part_o, uint32_t per_h, uint32_t per_t, int H_q,
                                                           int H_kv, int T, int heads, int g_first, int qtp, MergeArgs a)
{
    __shared__ float red[2 * SPECATTN_MAX_T];
    const int q = blockIdx.x, r = blockIdx.y;
    const uint32_t parts = row_parts[r];
    SPECATTN_PRELOAD(a.out); SPECATTN_PRELOAD(a.lse); SPECATTN_PRELOAD(a.out_lowp);
    if (TAIL) {
        SPECATTN_PRELOAD(a.sm_scale); SPECATTN_PRELOAD(a.q); SPECATTN_PRELOAD(a.k_new); SPECATTN_PRELOAD(a.v_new);
        SPECATTN_PRELOAD(a.q_stride_b); SPECATTN_PRELOAD(a.q_stride_h); SPECATTN_PRELOAD(a.q_stride_t);
    }
    const int b = (int)__umulhi((uint32_t)r << 1, per_h), h = r - b * H_kv;              // (div_h, div_t)
    const int gh = (int)(((uint32_t)q * per_t) >> 16), t = q - gh * T;
    const int head = h * heads + g_first + gh;
    const int64_t orow = ((int64_t)b * H_q + head) * T + t;
    const int dv = threadIdx.x;
    auto value = [](uint16_t x) { return F16 ? (float)__builtin_bit_cast(_Float16, x) : __uint_as_float((uint32_t)x << 16); };
    uint16_t qe = 0, ke[SPECATTN_MAX_T], ve[SPECATTN_MAX_T];
    if constexpr (TAIL) {
        const uint16_t *kn = a.k_new + (int64_t)r * T * D + dv, *vn = a.v_new + (int64_t)r * T * D + dv;
        qe = a.q[(int64_t)b * a.q_stride_b + (int64_t)head * a.q_stride_h + (int64_t)t * a.q_stride_t + dv];
#pragma unroll
        for (int p = 0; p < SPECATTN_MAX_T; ++p) {              // (tokens past t: t's again, not used)
            ke[p] = kn[(p < t ? p : t) * D];
            ve[p] = vn[(p < t ? p : t) * D];
        }
    }
    Merge acc;
    if (parts != ROW_EMPTY) {
        const int w0 = parts & 0xffffu, w1 = parts >> 16;
        if (w0 == w1 && !TAIL) return;              // finished by its only workgroup
        auto trip = [&](int wb, auto most) {        // partials wb .. w1, at most N
            constexpr int N = decltype(most)::value;
            float mw[N], lw[N], ow[N];
            uint32_t s[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {           // (behind the last share: that one's again)
                s[k] = (uint32_t)((min(wb + k, w1) + r) * qtp + q);
                if (N >= 8) asm("" : "+v"(s[k]));   // (the same in all lanes, but no scalar loads: above; the short rest does not care)
                const float2 ml = reinterpret_cast<const float2 *>(part_ml)[s[k]];
                mw[k] = ml.x;
                lw[k] = ml.y;
            }
            __builtin_amdgcn_sched_barrier(0);      // the weights first: they are used first
#pragma unroll
            for (int k = 0; k < N; ++k) ow[k] = part_o[s[k] * D + dv];
            __builtin_amdgcn_sched_barrier(0);      // all requested before the first is used
#pragma unroll
            for (int k = 0; k < N; ++k) {           // (a weight of zero must not meet an infinite value)
                mw[k] = wb + k <= w1 ? mw[k] : -INFINITY;
                ow[k] = wb + k <= w1 ? ow[k] : 0.0f;
            }
            acc.add_all(mw, lw, ow);
        };
        int wb = w0;
        for (; wb + 15 <= w1; wb += 16) trip(wb, std::integral_constant<int, 16>{});
        const int left = w1 - wb + 1;
        if (left > 8) trip(wb, std::integral_constant<int, 16>{});
        else if (left > 5) trip(wb, std::integral_constant<int, 8>{});
        else if (left > 2) trip(wb, std::integral_constant<int, 5>{});
        else if (left > 0) trip(wb, std::integral_constant<int, 2>{});
    }
    if constexpr (TAIL) {
        // scores of the query row against new tokens 0..t, over all threads of the workgroup
        const int lane = dv & 63, wave = dv >> 6;
#pragma unroll
        for (int p = 0; p < SPECATTN_MAX_T; ++p) {
            if (p > t) break;                       // (uniform)
            const float x = wave_sum(value(qe) * value(ke[p]));
            if (lane == 0) red[wave * SPECATTN_MAX_T + p] = x;
        }
        __syncthreads();
        const float scale2 = a.sm_scale * 1.4426950408889634f;       // m is in log2 units
        float mw[SPECATTN_MAX_T], lw[SPECATTN_MAX_T], ow[SPECATTN_MAX_T];
#pragma unroll
        for (int p = 0; p < SPECATTN_MAX_T; ++p) {
            mw[p] = p <= t ? (red[p] + (D > 64 ? red[SPECATTN_MAX_T + p] : 0.0f)) * scale2 : -INFINITY;
            lw[p] = p <= t ? 1.0f : 0.0f;
            ow[p] = p <= t ? value(ve[p]) : 0.0f;
        }
        acc.add_all(mw, lw, ow);
    }
    const float res = acc.l > 0.0f ? acc.o / acc.l : 0.0f;
    a.out[orow * D + dv] = res;
    if (a.out_lowp) st_lowp(a.out_lowp, orow * D + dv, res, F16 ? SPECATTN_F16 : SPECATTN_BF16);
    // m is in log2 units of the scaled scores
    if (a.lse && dv == 0) a.lse[orow] = acc.l > 0.0f ? (acc.m + log2f(acc.l)) * 0.6931471805599453f : -INFINITY;
}

template <int D> auto merge_variant(bool f16, bool tail)
{
    return f16 ? tail ? merge_partials_kernel<D, true, true> : merge_partials_kernel<D, true, false>
               : tail ? merge_partials_kernel<D, false, true> : merge_partials_kernel<D, false, false>;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

bool attn_mfma_supported(const AttnLaunch &a)
{
    // any number of query heads per kv head: groups of more than 64 query rows run as several launches
    return (a.dtype == SPECATTN_BF16 || a.dtype == SPECATTN_F16) && (a.d == 128 || a.d == 64) && a.T <= SPECATTN_MAX_T && a.H_kv <= MAX_ROWS;
}

int attn_mfma_workgroups() { return cu_count() * WG_PER_CU; }

static const void *attn_mfma_variant(int d, int src, int form, int nqt, int layout, bool f16)
{
    if (src == MASK) return d == 128 && form != FEW_ANY ? attn_mfma_mask(form, nqt, layout, f16) : nullptr;
    return form == FEW_POSITIONS ? attn_mfma_few_positions(d, nqt, layout, f16) : form == FEW_ANY ? attn_mfma_few_any(d, nqt, layout, f16) : attn_mfma_many(d, nqt, layout, f16);
}

// The kernels use more LDS than the default limit: raise it for every variant, once per device.
specattn_status attn_mfma_configure()
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
    for (int k = 0; k < 3 * 4 * 3 * 2 * 3; ++k) {
        const void *fn = attn_mfma_variant(k % 3 == 2 ? 64 : 128, k % 3 == 1 ? MASK : LIST, k / 72, k / 3 % 4 + 1, k / 12 % 3, k / 36 % 2 != 0);
        if (fn && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(MASK)) != hipSuccess) {
            (void)hipGetLastError();
            set_error("cannot reserve %d bytes of LDS", lds_bytes(MASK));
            return SPECATTN_EHIP;
        }
    }
    done[dev] = true;
    return SPECATTN_OK;
}

// Query rows per launch of a group of G heads x T tokens: groups of more than `limit` query rows are cut into equal
// shares of heads.
static int heads_per_launch(int G, int T, int limit)
{
    const int most = limit / T;                              // T <= 8 <= limit
    const int shares = (G + most - 1) / most;
    return (G + shares - 1) / shares;
}
static int query_tiles(int G, int T, int limit) { return (heads_per_launch(G, T, limit) * T + 15) / 16; }
constexpr int WIDE = 64, WIDE_MASK = 48, NARROW = 32;        // query rows a launch takes: four tiles (the mask source three),
                                                             // or two where the workspace holds no more

static size_t workspace_for(int rows, int nqt, int d)
{
    const size_t slots = (size_t)attn_mfma_workgroups() + rows;
    size_t bytes = align256(((size_t)rows + 1) * sizeof(int32_t));                        // the rows' shares (and a word to spare)
    bytes += slots * nqt * 16 * (d + 2) * sizeof(float);
    return align256(bytes);
}
// larger batches run as several launches over the same workspace
size_t attn_mfma_workspace_bytes(int rows, int G, int T, int d)
{
    const int nqt = query_tiles(G, T, WIDE), most = launch_rows(nqt, d);
    const size_t wide = workspace_for(rows < most ? rows : most, nqt, d), least = attn_mfma_workspace_min_bytes(rows, G, T, d);
    return wide > least ? wide : least;
}
size_t attn_mfma_workspace_narrow_bytes(int rows, int G, int T, int d)
{
    return workspace_for(rows < MAX_ROWS_LIST ? rows : MAX_ROWS_LIST, query_tiles(G, T, NARROW), d);
}
size_t attn_mfma_workspace_min_bytes(int rows, int G, int T, int d)
{
    return workspace_for(rows < MAX_ROWS ? rows : MAX_ROWS, query_tiles(G, T, NARROW), d);
}

// Calls of up to 64 rows with few tiles in all: every share is `unit` tiles (3, 4, 6, 8, 12, ... 32) of one row, so that no workgroup
// starts twice or holds a row's start alone, and a call's time is that of one share.  How many shares: fewer tiles in each are fewer to
// wait for, and spread a call's bytes over more CUs; but every sixteen parts of a row are one more trip of the merge, which from about 48
// on costs more than that saves, and with nearly all CUs taken the last shares come late.  So the least unit that leaves 218 of 256
// workgroups a share (fewer where rounding rows up could take the others) and a row 48 parts; three tiles where that is one tile per wave
// and few partials.  Longer ones, whose shares are many rounds of tiles, are cut from the line.
// Measured, rows x tiles (d = 128, 20 query rows): the line / units, the rule's in brackets, us for both launches:
//   1 x 50 10.4 / [3] 8.9, 4 8.8, 8 9.6;  1 x 200 18.0 / 4 11.0, [6] 11.2, 12 11.9;  1 x 573 21.6 / 8 14.4, [12] 13.5, 16 14.4
//   4 x 24 9.3 / [3] 8.45, 4 8.5;  4 x 150 12.6 / 3 12.2, [4] 11.5, 8 12.0;  4 x 500 16.2 / 8 16.1, [12] 15.0, 16 15.0;  4 x 1500 24.9 / 28 24.7, [32] 24.0
//   8 x 25 9.9 / 3 9.3, [4] 9.0, 6 9.9;  8 x 87 11.2 / 3 11.3, [4] 10.9, 6 11.0, 8 11.6;  8 x 154 12.5 / [6] 12.4, 8 12.7;  8 x 300 15.2 / [12] 14.8, 16 15.0;
//   8 x 457 19.0 / 16 18.5, [20] 17.7, 24 18.4;  8 x 640 22.2 / 20 21.4, [24] 21.2, 28 21.0
//   32 x 28 11.1 / 4 10.7, [6] 11.1, 8 11.7;  32 x 56 13.4 / 8 13.2, [12] 13.0;  32 x 160 21.2 / 20 20.9, [24] 20.5
//   64 x 9 10.5 / 3 10.0, [4] 10.2;  64 x 19 12.4 / 6 12.0, [8] 12.3, 12 12.3;  64 x 37 14.3 / 12 14.1, [16] 14.7;  64 x 48 15.8 / 12 15.6, [16] 15.7
//   d = 64: 4 x 128 11.8 / 3 11.0, [4] 10.4, 6 11.4;  64 x 25 13.2 / 8 12.8, [12] 13.2;  64 x 45 15.6 / 12 15.0, [16] 15.8
// Rows alone or in twos with more than 900 tiles would do with more than 48 parts: 1 x 1200 22.8 / 12 16.8, 16 16.4, [28] 18.3;
// 1 x 1530 23.5 / 16 17.4, 24 18.1, [32] 19.6; 2 x 1530 20.7 / 20 19.1, [32] 20.7.  (64 parts for all of them: 2 x 450 13.6 / 14.2.)
static void share_units(Plan &plan, int rows)
{
    const int goal = std::min({plan.n_wg * 218 / 256, plan.n_wg - rows, 48 * rows});
    plan.unit_line = rows > FEW_ROWS || goal <= 1 ? -1 : (rows > 32 ? 16 : rows > 4 ? 24 : 32) * goal;
    plan.per_share = goal <= 1 ? 0 : (uint32_t)((((uint64_t)1 << 32) + goal - 1) / goal);
}

static specattn_status launch_chunk(const AttnLaunch &a, hipStream_t stream)
{
    const int rows = a.B * a.H_kv;
    const int G = a.g_count ? a.g_count : a.H_q / a.H_kv;
    const int QT = G * a.T;
    const int nqt = (QT + 15) / 16, qtp = nqt * 16;
    Plan plan;
    plan.n_wg = attn_mfma_workgroups();
    share_units(plan, rows);
    plan.heads = a.H_q / a.H_kv;
    plan.group = G;
    plan.per_h = (uint32_t)((((uint64_t)1 << 31) + a.H_kv - 1) / a.H_kv);
    plan.per_t = (65536u + a.T - 1) / a.T;
    const size_t slots = (size_t)plan.n_wg + rows;
    // every workgroup may leave a partial in slot (workgroup + row): never launch over a workspace that cannot hold them
    if (!a.workspace || a.workspace_bytes < workspace_for(rows, nqt, a.d)) {
        set_error("attention workspace has %zu bytes, %zu needed", a.workspace_bytes, workspace_for(rows, nqt, a.d));
        return SPECATTN_EWORKSPACE;
    }
    char *ws = static_cast<char *>(a.workspace);
    plan.row_parts = reinterpret_cast<uint32_t *>(ws);
    ws += align256(((size_t)rows + 1) * sizeof(int32_t));
    plan.part_ml = reinterpret_cast<float *>(ws);
    plan.part_o = plan.part_ml + slots * qtp * 2;
    const int layout = a.indices_are_physical ? PHYSICAL : (a.page_table ? PAGE_TABLE : CONTIGUOUS);
    const int src = a.kept_mask ? MASK : LIST;
    const bool f16 = a.dtype == SPECATTN_F16;
    // (The form for single positions spills six registers more at four query tiles of 128: 64 rows of 13001 positions with 64 query rows 43.0 one form for
    // all, 44.0 that one, 42.5 the form for lists of any kind.)
    const bool any = src == LIST && (a.dense || a.chunk_shift || (nqt == 4 && a.d == 128));
    const int form = rows > FEW_ROWS ? MANY : any ? FEW_ANY : FEW_POSITIONS;
    const void *fn = attn_mfma_variant(a.d, src, form, nqt, layout, f16);
    if (!fn) { set_error("the fused path takes logical positions, not pool slots"); return SPECATTN_EUNSUPPORTED; }
    specattn_status st = attn_mfma_configure();
    if (st != SPECATTN_OK) return st;
    void *kargs[] = {const_cast<AttnLaunch *>(&a), &plan};
    if (hipLaunchKernel(fn, dim3(plan.n_wg), dim3(THREADS), kargs, lds_bytes(src), stream) != hipSuccess) {
        set_error("attn_mfma_kernel: launch failed");
        (void)hipGetLastError();
        return SPECATTN_EHIP;
    }
    st = check_launch("attn_mfma_kernel");
    if (st != SPECATTN_OK) return st;
    const MergeArgs m = {a.out, a.lse, a.out_lowp, a.sm_scale, static_cast<const uint16_t *>(a.q), static_cast<const uint16_t *>(a.k_new), static_cast<const uint16_t *>(a.v_new),
                         a.q_stride_b, a.q_stride_h, a.q_stride_t};
    const auto merge = a.d == 64 ? merge_variant<64>(f16, a.k_new != nullptr) : merge_variant<128>(f16, a.k_new != nullptr);
    hipLaunchKernelGGL(merge, dim3(QT, rows), dim3(a.d), 0, stream, plan.row_parts, plan.part_ml, plan.part_o, plan.per_h, plan.per_t, a.H_q, a.H_kv, a.T, plan.heads,
                       a.g_first, qtp, m);
    return check_launch("merge_partials_kernel");
}

// Batches with more rows than the kernel's LDS tables hold go out as several launches over
// consecutive sequences (rows are independent; the workspace is reused, the stream orders them).
// Likewise the query heads of a kv head: at most 64 query rows (heads x T) fit one launch, larger groups
// are cut into equal shares of heads, each streaming the kept K/V again.
static specattn_status launch_batch(const AttnLaunch &a, int cap, hipStream_t stream);

// Rows per launch of `nqt` query tiles that the workspace has room for: as many as the kernel's tables hold, or - when it
// was sized for less (the built-in scratch buffer) - what is left of that, at least one sequence; 0 if not even that fits.
static int rows_per_launch(const AttnLaunch &a, int nqt)
{
    const int rows = a.B * a.H_kv, most = launch_rows(nqt, a.d);
    for (int cap = rows < most ? rows : most;; cap = cap > MAX_ROWS ? MAX_ROWS : cap / 2) {
        if (cap < a.H_kv) return 0;
        if (a.workspace_bytes >= workspace_for(cap, nqt, a.d)) return cap;
    }
}

specattn_status launch_attn_mfma(const AttnLaunch &a, hipStream_t stream)
{
    const int G = a.H_q / a.H_kv;
    int limit = a.kept_mask ? WIDE_MASK : WIDE, cap = rows_per_launch(a, query_tiles(G, a.T, limit));
    if (cap == 0) { limit = NARROW; cap = rows_per_launch(a, query_tiles(G, a.T, NARROW)); }
    if (cap == 0) cap = a.H_kv;                             // (launch_chunk refuses what its workspace cannot hold)
    const int heads = heads_per_launch(G, a.T, limit);
    if (heads >= G) return launch_batch(a, cap, stream);
    for (int g0 = 0; g0 < G; g0 += heads) {
        AttnLaunch c = a;
        c.g_first = g0;
        c.g_count = (G - g0) < heads ? (G - g0) : heads;
        const specattn_status st = launch_batch(c, cap, stream);
        if (st != SPECATTN_OK) return st;
    }
    return SPECATTN_OK;
}

static specattn_status launch_batch(const AttnLaunch &a, int cap, hipStream_t stream)
{
    const int b_max = cap / a.H_kv;
    if (a.B <= b_max) return launch_chunk(a, stream);
    const int es = 2;                                       // bf16 or fp16
    for (int b0 = 0; b0 < a.B; b0 += b_max) {
        AttnLaunch c = a;
        c.B = (a.B - b0) < b_max ? (a.B - b0) : b_max;
        const int64_t r0 = (int64_t)b0 * a.H_kv;
        c.q = static_cast<const char *>(a.q) + (int64_t)b0 * a.q_stride_b * es;
        const bool paged = a.page_table != nullptr || a.indices_are_physical;
        if (!paged) {
            c.k = static_cast<const char *>(a.k) + (int64_t)b0 * a.kv_stride_b * es;
            c.v = static_cast<const char *>(a.v) + (int64_t)b0 * a.kv_stride_b * es;
        }
        if (a.page_table) c.page_table = a.page_table + (int64_t)b0 * a.max_pages;
        if (a.indices) c.indices = a.indices + r0 * a.idx_stride;
        if (a.counts) c.counts = a.counts + r0;
        c.out = a.out + (int64_t)b0 * a.H_q * a.T * a.d;
        if (a.out_lowp) c.out_lowp = static_cast<char *>(a.out_lowp) + (int64_t)b0 * a.H_q * a.T * a.d * es;
        if (a.lse) c.lse = a.lse + (int64_t)b0 * a.H_q * a.T;
        if (a.seq_lens) c.seq_lens = a.seq_lens + b0;
        if (a.k_new) {
            c.k_new = static_cast<const char *>(a.k_new) + r0 * a.T * a.d * es;
            c.v_new = static_cast<const char *>(a.v_new) + r0 * a.T * a.d * es;
        }
        if (a.kept_mask) {
            c.kept_mask = a.kept_mask + r0 * a.blocks_per_row * (SEL_BLOCK / 32);
            c.block_counts = a.block_counts + r0 * a.blocks_per_row;
        }
        const specattn_status st = launch_chunk(c, stream);
        if (st != SPECATTN_OK) return st;
    }
    return SPECATTN_OK;
}

}  // namespace specattn
