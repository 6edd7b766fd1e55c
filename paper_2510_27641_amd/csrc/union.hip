// Algorithm 2 as a whole (Section 3.4): the draft model's attention row of every speculative step
// (and of every draft head that feeds a kv head) is cut at its own exact top-p threshold, and the
// union of the kept sets is emitted as one ascending list per (sequence, kv head).
//
// Two launches: the selection kernel over all member rows, which leaves every row's kept set as one bit per position
// while the row is still in its registers; then a pass over those bits alone (a thirty-second of the rows) in which every
// workgroup combines the members' words of one segment of a row and numbers its kept positions.
//
// Rows whose thresholds come from elsewhere (the bisection), rows that the selection does not hold in registers, and unions
// with a workspace that does not hold the members' bits, take a mask pass that compares the rows with their thresholds again
// and a compaction pass over its ballots.
#include <hip/hip_runtime.h>

#include "common.h"

#include <type_traits>

namespace specattn {
namespace {

constexpr int U_THREADS = 256;
constexpr int U_WAVES = U_THREADS / 64;
constexpr int U_ITERS = 4;                                  // float4 loads per thread and member row
constexpr int U_BLOCK = U_THREADS * 4 * U_ITERS;            // 4096 positions per workgroup
constexpr int U_WORDS = U_ITERS * U_WAVES * 4;              // ballots per block: [iter][wave][component]

typedef float f32x4a __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load from any float's address

struct UnionLaunch {
    const float *probs;
    int64_t stride_b, stride_m;     // elements between sequences / between consecutive member rows
    int B, H_kv, M, n_max;          // M member rows per (sequence, kv head), consecutive
    const int32_t *seq_lens;
    const float *tau;               // [B * H_kv * M] thresholds of the member rows
    const int32_t *mcounts;         // [B * H_kv * M] kept counts of the member rows (0 = contributes nothing)
    const uint32_t *mflags;         // [B * H_kv * M]
    int32_t *block_counts;          // [rows][blocks]
    unsigned long long *ballots;    // [rows][blocks][U_WORDS]
    int blocks;
    int32_t *indices;
    int64_t idx_stride;
    int idx_capacity;
    int32_t *counts;
    uint32_t *row_flags;
    const int32_t *page_table;
    int page_shift, max_pages, emit_physical;
};

// one workgroup per (row, block): kept bits of positions [blk * U_BLOCK, (blk + 1) * U_BLOCK) of row r.
// Position of (iter, thread, component): blk * U_BLOCK + iter * U_THREADS * 4 + thread * 4 + component.
template <int U_MEMBERS> __global__ __launch_bounds__(U_THREADS) void union_mask_kernel(UnionLaunch a)
{
    __shared__ int wave_cnt[U_WAVES];
    const int r = blockIdx.x / a.blocks, blk = blockIdx.x - r * a.blocks;
    const int b = r / a.H_kv, h = r - b * a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int len = a.seq_lens ? a.seq_lens[b] : a.n_max;
    len = len < 0 ? 0 : (len > a.n_max ? a.n_max : len);
    const float *rows = a.probs + (int64_t)b * a.stride_b + (int64_t)h * a.M * a.stride_m;
    const int64_t m0 = (int64_t)r * a.M;
    unsigned keep[U_ITERS] = {0u, 0u, 0u, 0u};                // 4 bits per iteration
    // compared as integers, like the selection itself: non-negative floats order like their bit
    // patterns; -0.0 (the only signed value a valid row can hold) counts as zero
    auto bits = [](float f) { const int i = __float_as_int(f); return i == (int)0x80000000 ? 0 : i; };
    auto compare = [&](int it, const f32x4a &v, int t) {
        const int x = bits(v.x), y = bits(v.y), z = bits(v.z), w = bits(v.w);
        keep[it] |= (x >= t ? 1u : 0u) | (y >= t ? 2u : 0u) | (z >= t ? 4u : 0u) | (w >= t ? 8u : 0u);
    };
    const bool whole = (blk + 1) * U_BLOCK <= len;             // uniform
    for (int mc = 0; mc < a.M; mc += 64) {
        const int ms = a.M - mc < 64 ? a.M - mc : 64;
        // lane m: the threshold of member mc + m, negative where it keeps nothing.  (Exact thresholds are above 0; a
        // bisection's may be 0 and keeps zeros, too.)
        const int64_t at = m0 + mc + (lane < ms ? lane : 0);
        const int tau = a.mcounts[at] > 0 ? __float_as_int(a.tau[at]) : -1;
        const float *first = rows + (int64_t)mc * a.stride_m;
        int m = 0;
        if (whole) {
            // four members at a time: their thresholds are here and all of their loads in flight together (one after the
            // other, with a trip for each threshold, 8 rows of 66000 with 24 members each took 91 us, now 59)
            for (; m + U_MEMBERS <= ms; m += U_MEMBERS) {
                f32x4a v[U_MEMBERS][U_ITERS];
#pragma unroll
                for (int k = 0; k < U_MEMBERS; ++k)
#pragma unroll
                    for (int it = 0; it < U_ITERS; ++it)
                        v[k][it] = *reinterpret_cast<const f32x4a *>(first + (m + k) * a.stride_m + blk * U_BLOCK + it * U_THREADS * 4 + tid * 4);
#pragma unroll
                for (int k = 0; k < U_MEMBERS; ++k) {
                    const int t = __builtin_amdgcn_readlane(tau, m + k);
                    if (t < 0) continue;                      // (uniform) an invalid row's entries may compare anyhow
#pragma unroll
                    for (int it = 0; it < U_ITERS; ++it) compare(it, v[k][it], t);
                }
            }
        }
        for (; m < ms; ++m) {
            const int t = __builtin_amdgcn_readlane(tau, m);
            if (t < 0) continue;
            const float *row = first + m * a.stride_m;
#pragma unroll
            for (int it = 0; it < U_ITERS; ++it) {
                const int p = blk * U_BLOCK + it * U_THREADS * 4 + tid * 4;
                f32x4a v = {-1.f, -1.f, -1.f, -1.f};          // positions past the row's end: below any threshold
                if (p + 3 < len) {
                    v = *reinterpret_cast<const f32x4a *>(row + p);
                } else {
                    if (p < len) v.x = row[p];
                    if (p + 1 < len) v.y = row[p + 1];
                    if (p + 2 < len) v.z = row[p + 2];
                    if (p + 3 < len) v.w = row[p + 3];
                }
                compare(it, v, t);
            }
        }
    }
    unsigned long long *words = a.ballots + ((int64_t)r * a.blocks + blk) * U_WORDS;
    int cnt = 0;
#pragma unroll
    for (int it = 0; it < U_ITERS; ++it) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned long long w = __ballot((keep[it] >> c) & 1u);
            cnt += __popcll(w);
            if (lane == 0) words[(it * U_WAVES + wave) * 4 + c] = w;
        }
    }
    if (lane == 0) wave_cnt[wave] = cnt;
    __syncthreads();
    if (tid == 0) {
        int total = 0;
        for (int w = 0; w < U_WAVES; ++w) total += wave_cnt[w];
        a.block_counts[(int64_t)r * a.blocks + blk] = total;
    }
}

// flags of row r, whose union holds `total` positions
__device__ __forceinline__ uint32_t union_flags(const UnionLaunch &a, int r, int total)
{
    uint32_t any_valid = 0, near = 0;
    for (int m = 0; m < a.M; ++m) {
        const uint32_t f = a.mflags[(int64_t)r * a.M + m];
        if (!(f & SPECATTN_ROW_INVALID)) { any_valid = 1; near |= f & SPECATTN_ROW_NEAR_BOUNDARY; }
    }
    uint32_t f = any_valid ? near : SPECATTN_ROW_INVALID;
    if (total > a.idx_capacity) f |= SPECATTN_ROW_OVERFLOW;
    return f;
}

// one workgroup per (row, block): writes the positions of its block at their rank in the row's list.
__global__ __launch_bounds__(U_THREADS) void union_compact_kernel(UnionLaunch a)
{
    __shared__ int part[U_WAVES][2];
    __shared__ unsigned long long words[U_WORDS];
    __shared__ int group_base[U_ITERS * U_WAVES];
    const int r = blockIdx.x / a.blocks, blk = blockIdx.x - r * a.blocks;
    const int b = r / a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // kept before this block, and in the whole row
    int before = 0, total = 0;
    for (int k = tid; k < a.blocks; k += U_THREADS) {
        const int c = a.block_counts[(int64_t)r * a.blocks + k];
        total += c;
        if (k < blk) before += c;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        before += __shfl_xor(before, off, 64);
        total += __shfl_xor(total, off, 64);
    }
    if (lane == 0) { part[wave][0] = before; part[wave][1] = total; }
    if (tid < U_WORDS) words[tid] = a.ballots[((int64_t)r * a.blocks + blk) * U_WORDS + tid];
    __syncthreads();
    before = total = 0;
#pragma unroll
    for (int w = 0; w < U_WAVES; ++w) { before += part[w][0]; total += part[w][1]; }
    if (tid == 0) {                                           // list position of every (iter, wave) group
        int run = before;
        for (int gidx = 0; gidx < U_ITERS * U_WAVES; ++gidx) {
            group_base[gidx] = run;
            for (int c = 0; c < 4; ++c) run += __popcll(words[gidx * 4 + c]);
        }
    }
    if (blk == 0 && tid == 0) {
        a.counts[r] = total;
        if (a.row_flags) a.row_flags[r] = union_flags(a, r, total);
    }
    __syncthreads();
    int32_t *out = a.indices + (int64_t)r * a.idx_stride;
    const int32_t *ptab = (a.emit_physical && a.page_table) ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int it = 0; it < U_ITERS; ++it) {
        const unsigned long long *w = words + (it * U_WAVES + wave) * 4;
        int o = group_base[it * U_WAVES + wave] +
                __popcll(w[0] & below) + __popcll(w[1] & below) + __popcll(w[2] & below) + __popcll(w[3] & below);
        const int p = blk * U_BLOCK + it * U_THREADS * 4 + tid * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if ((w[c] >> lane) & 1ull) {
                if (o < a.idx_capacity) {
                    const int pos = p + c;
                    out[o] = ptab ? ((ptab[pos >> a.page_shift] << a.page_shift) | (pos & ((1 << a.page_shift) - 1))) : pos;
                }
                ++o;
            }
        }
    }
}

// ---- from the members' kept bits ------------------------------------------------------------------------------
constexpr int W_SEGMENTS = 16;                              // per row, at most
constexpr int W_LEAST = 4096;                               // positions per segment, at least
constexpr int W_MOST = (SPECATTN_MAX_N + W_SEGMENTS - 1) / W_SEGMENTS;     // ... and at most

struct WordsLaunch {
    const uint32_t *masks;          // [rows * M][words]
    int words;                      // 32-bit words per member row (a multiple of SEL_BLOCK / 32)
    int segments, seg_words;        // workgroups per row; 32-bit words of each (a multiple of 4)
};

// one workgroup per (row, segment).  It counts the row's kept positions ahead of its segment by itself, from the words of
// all segments before (on average half the row's words: 16 segments read 8 / 32 = a quarter of what the rows weigh, from
// L2), which costs less than a launch of its own or a pass over the rows: 64 rows of 32768 positions, 16 members each,
// 8.5 us behind a selection of 58 us (without the bits: selection 48 us, mask pass over the rows 44 us, compaction 6.5 us).
// Bound by its chain of trips: the arguments come in one batch, up to 16 members' words are requested together, the segments that read most start
// first, and all segments of a row go to one XCD (where the rows are a multiple of eight), whose L2 then fetches the row's words once.
// (Before / so, us, with the selection: 64 rows of 16 members of 32768 46.0 / 41.4, of 10 of 30000 38.2 / 35.6, of 2 of 32768 17.5 / 16.9, 16 rows
// of 6 of 8192 11.8 / 10.7.)
__global__ __launch_bounds__(U_THREADS) void union_words_kernel(UnionLaunch a, WordsLaunch w)
{
    __shared__ uint4 words4[W_MOST / 128];
    __shared__ int wave_sum[2][U_WAVES];
    __shared__ int base_of[W_MOST / 64];                      // kept in the segment before each 64-bit word
    SPECATTN_PRELOAD(w.masks); SPECATTN_PRELOAD(w.words); SPECATTN_PRELOAD(w.segments); SPECATTN_PRELOAD(w.seg_words); SPECATTN_PRELOAD(a.M); SPECATTN_PRELOAD(a.H_kv);
    SPECATTN_PRELOAD(a.counts); SPECATTN_PRELOAD(a.row_flags); SPECATTN_PRELOAD(a.indices); SPECATTN_PRELOAD(a.idx_stride); SPECATTN_PRELOAD(a.idx_capacity);
    SPECATTN_PRELOAD(a.emit_physical); SPECATTN_PRELOAD(a.page_table); SPECATTN_PRELOAD(a.page_shift); SPECATTN_PRELOAD(a.max_pages);
    const int r = blockIdx.x, seg = w.segments - 1 - (int)blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row4 = w.words >> 2, seg4 = w.seg_words >> 2;
    const int q0 = seg * seg4;
    int q1 = q0 + seg4;
    q1 = q1 < row4 ? q1 : row4;
    const uint4 *masks = reinterpret_cast<const uint4 *>(w.masks) + (int64_t)r * a.M * row4;
    int before = 0;
    for (int q = tid; q < q1; q += U_THREADS) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        auto members = [&](int m0, auto most) {                // (behind the last member: that one again)
            constexpr int N = decltype(most)::value;
            uint4 u[N];
#pragma unroll
            for (int k = 0; k < N; ++k) u[k] = masks[(int64_t)min(m0 + k, a.M - 1) * row4 + q];
#pragma unroll
            for (int k = 0; k < N; ++k) { v.x |= u[k].x; v.y |= u[k].y; v.z |= u[k].z; v.w |= u[k].w; }
        };
        int m = 0;
        for (; m + 8 < a.M; m += 16) members(m, std::integral_constant<int, 16>{});
        if (m < a.M) members(m, std::integral_constant<int, 8>{});
        if (q >= q0) words4[q - q0] = v;
        else before += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    before = wave_inclusive_sum(before);
    if (lane == 63) wave_sum[0][wave] = before;
    __syncthreads();
    before = 0;
#pragma unroll
    for (int k = 0; k < U_WAVES; ++k) before += wave_sum[0][k];
    // prefix over the segment's 64-bit words, U_THREADS of them per round
    const unsigned long long *words = reinterpret_cast<const unsigned long long *>(words4);
    const int n64 = (q1 - q0) * 2;
    int run = 0;
    for (int k0 = 0; k0 < n64; k0 += U_THREADS) {
        const int k = k0 + tid, c = k < n64 ? __popcll(words[k]) : 0;
        const int inc = wave_inclusive_sum(c);
        if (k0) __syncthreads();                              // the round before has been read out
        if (lane == 63) wave_sum[1][wave] = inc;
        __syncthreads();
        int base = run;
#pragma unroll
        for (int j = 0; j < U_WAVES; ++j) {
            const int t = wave_sum[1][j];
            if (j < wave) base += t;
            run += t;
        }
        if (k < n64) base_of[k] = base + inc - c;
    }
    if (seg == w.segments - 1 && tid == 0) {
        const int total = before + run;
        a.counts[r] = total;
        if (a.row_flags) a.row_flags[r] = union_flags(a, r, total);
    }
    __syncthreads();
    int32_t *out = a.indices + (int64_t)r * a.idx_stride;
    const int32_t *ptab = (a.emit_physical && a.page_table) ? a.page_table + (int64_t)(r / a.H_kv) * a.max_pages : nullptr;
    for (int k = wave; k < n64; k += U_WAVES) {               // lane i: position i of the word
        const unsigned long long v = words[k];
        const int o = before + base_of[k] + __popcll(v & ((1ull << lane) - 1ull));
        if (((v >> lane) & 1ull) && o < a.idx_capacity) {
            const int pos = q0 * 128 + k * 64 + lane;
            // (a streaming store, as the selection writes its lists: 1024 members with attention 176.8 us without, 174.8 with)
            __builtin_nontemporal_store(ptab ? ((ptab[pos >> a.page_shift] << a.page_shift) | (pos & ((1 << a.page_shift) - 1))) : pos, out + o);
        }
    }
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t union_blocks(int n_max) { return ((size_t)n_max + U_BLOCK - 1) / U_BLOCK; }

size_t union_workspace_bytes(int B, int H_kv, int M, int n_max)
{
    const size_t rows = (size_t)B * H_kv, members = rows * M, blocks = union_blocks(n_max);
    return 3 * align256(members * 4) + align256(rows * blocks * 4) + align256(rows * blocks * U_WORDS * 8);
}

// The passes behind the selection, for rows whose member thresholds are known: over the members' kept bits where there
// are any, else over the rows.
specattn_status launch_threshold_union(const float *probs, int64_t stride_b, int64_t stride_m, int B, int H_kv, int M,
                                       int n_max, const int32_t *seq_lens, const float *tau, const int32_t *mcounts,
                                       const uint32_t *mflags, void *scratch, int32_t *indices, int64_t idx_stride,
                                       int idx_capacity, int32_t *counts, uint32_t *row_flags,
                                       const int32_t *page_table, int page_size, int max_pages, int emit_physical,
                                       const uint32_t *masks, hipStream_t stream)
{
    const size_t rows = (size_t)B * H_kv, blocks = union_blocks(n_max);
    char *ws = static_cast<char *>(scratch);
    UnionLaunch a{};
    a.probs = probs; a.stride_b = stride_b; a.stride_m = stride_m;
    a.B = B; a.H_kv = H_kv; a.M = M; a.n_max = n_max;
    a.seq_lens = seq_lens;
    a.tau = tau; a.mcounts = mcounts; a.mflags = mflags;
    a.block_counts = reinterpret_cast<int32_t *>(ws);
    a.ballots = reinterpret_cast<unsigned long long *>(ws + align256(rows * blocks * 4));
    a.blocks = (int)blocks;
    a.indices = indices; a.idx_stride = idx_stride; a.idx_capacity = idx_capacity;
    a.counts = counts; a.row_flags = row_flags;
    a.page_table = page_table; a.max_pages = max_pages; a.emit_physical = emit_physical;
    a.page_shift = 0;
    if (page_table) while ((1 << a.page_shift) < page_size) ++a.page_shift;
    if (masks) {
        const int blocks1k = (n_max + SEL_BLOCK - 1) / SEL_BLOCK;
        WordsLaunch w{};
        w.masks = masks;
        w.words = blocks1k * (SEL_BLOCK / 32);
        int seg = (n_max + W_SEGMENTS - 1) / W_SEGMENTS;
        seg = seg < W_LEAST ? W_LEAST : seg;
        w.seg_words = (seg + 127) / 128 * 4;
        w.segments = (w.words + w.seg_words - 1) / w.seg_words;
        hipLaunchKernelGGL(union_words_kernel, dim3((unsigned)rows, (unsigned)w.segments), dim3(U_THREADS), 0, stream, a, w);
        return check_launch("union_words_kernel");
    }
    const dim3 grid((unsigned)(blocks * rows));
    if (M >= 8) hipLaunchKernelGGL(union_mask_kernel<4>, grid, dim3(U_THREADS), 0, stream, a);
    else if (M >= 2) hipLaunchKernelGGL(union_mask_kernel<2>, grid, dim3(U_THREADS), 0, stream, a);
    else hipLaunchKernelGGL(union_mask_kernel<1>, grid, dim3(U_THREADS), 0, stream, a);
    specattn_status st = check_launch("union_mask_kernel");
    if (st != SPECATTN_OK) return st;
    hipLaunchKernelGGL(union_compact_kernel, grid, dim3(U_THREADS), 0, stream, a);
    return check_launch("union_compact_kernel");
}

// Kept bits of all member rows, behind union_workspace_bytes.  Only of rows that stay in the selection's registers: a longer
// row's bits take the selection a fourth pass over it, with one workgroup, where the mask pass reads it with the whole chip
// (us, with bits / without: 8 members of 131072 72 / 50, of 400000 209 / 126, 768 of 66000 168 / 150).
size_t union_masks_bytes(int B, int H_kv, int M, int n_max)
{
    return align256((size_t)B * H_kv * M * ((n_max + SEL_BLOCK - 1) / SEL_BLOCK) * (SEL_BLOCK / 32) * sizeof(uint32_t));
}

// workspace: [member tau][member counts][member flags][block counts][ballots], then the members' kept bits if there is room
specattn_status launch_union(const specattn_union_args *u, void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    const int per = u->H_draft / u->H_kv, M = per * u->S;
    const size_t members = (size_t)u->B * u->H_kv * M;
    char *ws = static_cast<char *>(workspace);
    const size_t before_masks = union_workspace_bytes(u->B, u->H_kv, M, u->n_max);
    const bool room = workspace_bytes >= before_masks + union_masks_bytes(u->B, u->H_kv, M, u->n_max);
    uint32_t *masks = u->n_max <= SELECT_RESIDENT && room ? reinterpret_cast<uint32_t *>(ws + before_masks) : nullptr;
    float *tau = u->member_thresholds ? u->member_thresholds : reinterpret_cast<float *>(ws);
    ws += align256(members * 4);
    int32_t *mcounts = u->member_counts ? u->member_counts : reinterpret_cast<int32_t *>(ws);
    ws += align256(members * 4);
    uint32_t *mflags = reinterpret_cast<uint32_t *>(ws);
    ws += align256(members * 4);

    SelectLaunch s{};                                         // every member row on its own: threshold and kept bits
    s.probs = u->probs;
    s.stride_b = u->probs_stride_b;
    s.stride_h = u->probs_stride_row;
    s.B = u->B;
    s.H_kv = u->H_draft * u->S;
    s.n_max = u->n_max;
    s.n_tokens = u->n_max;
    s.seq_lens = u->seq_lens;
    s.top_p = u->top_p;
    s.counts = mcounts;
    s.thresholds = tau;
    s.row_flags = mflags;
    s.kept_mask = masks;
    s.blocks_per_row = (u->n_max + SEL_BLOCK - 1) / SEL_BLOCK;
    const specattn_status st = launch_select(s, stream);
    if (st != SPECATTN_OK) return st;
    return launch_threshold_union(u->probs, u->probs_stride_b, u->probs_stride_row, u->B, u->H_kv, M, u->n_max,
                                  u->seq_lens, tau, mcounts, mflags, ws, u->indices, u->idx_stride_row, u->idx_capacity,
                                  u->counts, u->row_flags, u->page_table, u->page_size, u->max_pages_per_seq,
                                  u->emit_physical, masks, stream);
}

}  // namespace specattn
