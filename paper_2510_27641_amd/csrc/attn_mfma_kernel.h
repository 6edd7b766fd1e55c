// Sparse decode attention over a selected index list or kept-position mask (Section 3.1.2, Eq. 2-3;
// Section 3.5), bf16 or fp16, d = 128 or 64, up to 64 query rows per kv head and launch: the gfx950
// matrix-core variant.
//
// Work split ("stream-K" over kept positions): the kept positions of all rows, in tiles of 8 KiB of keys
// (32 positions of 128, 64 positions of 64), form one line; the line is cut into one share per workgroup (one workgroup of eight waves
// per CU), so the split is balanced by the *kept* count whatever the per-row counts are: equal shares, long ones a few per cent
// larger on even XCDs (make_share), or, in calls of up to 64 rows with few tiles, a few tiles of one row each (share_units).  A fixed
// permutation of the workgroup numbers puts the owners of consecutive shares on different XCDs.  A share
// that crosses row boundaries yields one partial (m, l, o) per (row, workgroup); partial (r, w) lives in
// slot w + r.  merge_partials_kernel combines a row's partials, in workgroup order.  Inside a share tile k goes
// to wave k mod 8, over the mask wave w takes the w-th eighth of the tiles, so every sum is taken in a fixed order and the outputs are
// bit-identical from run to run.
// Measured and dropped: waves claiming the tiles of a share from an LDS counter as their data arrives (no
// faster on any workload, 1.3 us slower on the 32K layer, and it gives the fixed summation order up); tiles of
// a row claimed by all of its workgroups from a counter in memory (a device-scope atomic takes about as long
// as a tile under load - 5 us - and claims made that far ahead leave as much unbalanced work at the end as they
// remove); the merge folded into this kernel (last arriver per row: write-through stores, an atomic and
// device-scope loads in a row cost 14 us after the last tile, against 8 us for the wrap-up plus the second
// launch).
//
// Data path per wave and tile: the gathered K rows and V rows (32 of 256 B, or 64 of 128 B) go from HBM
// straight into LDS (global_load_lds: 16 or 8 lanes fetch one full row, 1 KiB per instruction,
// XOR-swizzled chunk order).  Each wave owns one K buffer and one V buffer; the next tile's K is
// requested as soon as this tile's K fragments are in registers, the next V as soon as this tile's
// V has been consumed.  The list words of a tile (or the words of the kept mask) are fetched the same way,
// by LDS-DMA into two small slots per wave, one iteration ahead of the gathers that need them: nothing a
// tile needs is waited for when its turn comes, and no barrier separates the tiles of a share.
//   S^T = K Q^T    : mfma 16x16x32, A = K fragment (ds_read_b128), B = Q fragment (Q tile in LDS)
//   softmax        : running reference max per query row, rescaled only when a tile leaves its range (Half)
//   O^T += V^T P^T : A = V^T fragment (ds_read_b64_tr_b16), B = P split into parts of the element type (two, at d = 64 three)
// Query rows come in tiles of 16, up to four per launch: a kept K/V row is fetched once for all of them.  (Groups of
// more than 32 query rows used to take a launch per 32 and fetch everything again: 8 heads x 5 tokens, 64 rows x 4500
// kept positions, 69 us of attention against 40 us.)  d = 64 keeps bytes per tile, requests in flight and the
// schedule of d = 128; only the fragment geometry differs (32 heads over 4 kv heads, 4 x 8192 positions: 15 us against
// 71 us on the vector ALU).
// The mfma output layout puts each query row in a fixed lane, so scores, weights and output
// accumulators of that row never leave the lane.
#pragma once

#include "common.h"

namespace specattn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// The two 16-bit element types the matrix cores take here.  Both contractions use the 16x16x32 shape;
// the softmax weights are handed over as a high part (the weight rounded to the element type) and a low
// part (the rounding error, rounded again), so that the type's short significand costs no accuracy.
// A tile's weights are taken in units of 2^ref, its query row's running reference: the largest weight of a tile lies between
// 2^LO and 2^HI of them, and a reference chosen anew puts it at 2^HEAD.  bf16 has the exponents of fp32, so its reference only
// has to follow the maximum up.  fp16 ends at 2^-24: there the reference follows it down as well, or the weights that lie far
// below a row's one large one (an attention sink) would be lost to the products but not to the sum of the weights.
template <bool F16> struct Half;
template <> struct Half<false> {
    static constexpr float HEAD = 0.0f, HI = 8.0f;
    typedef bf16x8 x8;
    typedef bf16x2 x2;
    static __device__ __forceinline__ f32x4 mfma(x8 a, x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct Half<true> {
    static constexpr float HEAD = 12.0f, HI = 15.0f, LO = 8.0f;
    typedef f16x8 x8;
    typedef f16x2 x2;
    static __device__ __forceinline__ f32x4 mfma(x8 a, x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))
#define GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void *)(p))

constexpr int NW = ATTN_MFMA_WAVES;   // waves per workgroup
constexpr int THREADS = NW * 64;
constexpr int WG_PER_CU = 8 / NW;     // eight waves per CU in all
constexpr int TILE_BYTES = 8192;      // of one tensor
constexpr int WAVE_LDS = 2 * TILE_BYTES;              // K buffer, V buffer
// Geometry of a tile for head dimension D.
template <int D> struct Geo {
    static constexpr int ROW_BYTES = D * 2;           // one K or V row
    static constexpr int TILE = TILE_BYTES / ROW_BYTES;   // positions per tile
    static constexpr int LPR = ROW_BYTES / 16;        // lanes that fetch one row
    static constexpr int RPI = 64 / LPR;              // rows per gather instruction
    static constexpr int PT = TILE / 16;              // 16-position tiles of the score product
    static constexpr int KS = D / 32;                 // its k-steps
    static constexpr int PB = TILE / 32;              // k-steps of the value product
    static constexpr int DT = D / 16;                 // 16-wide tiles of the output
    // 16-byte chunk c of row `row` is stored in slot c ^ swz(row): makes both the K fragment reads
    // (16 rows x one chunk) and the V transpose reads (8 rows x 32 B) spread over all banks.
    static __device__ __forceinline__ int swz(int row)
    {
        return D == 128 ? ((row & 7) << 1) | ((row >> 3) & 1) : (((row >> 1) & 3) << 1) | ((row >> 3) & 1);
    }
};
constexpr int MAX_ROWS = ATTN_MFMA_MAX_ROWS;          // rows whose cost prefix fits the LDS table
constexpr int SLOT_BYTES = 256;       // one wave-wide LDS-DMA of 4 bytes per lane
constexpr int KV_AUX = 2;             // cache policy of the K/V gathers: non-temporal (each row is used once)
constexpr int SEG_COST = 12;          // cost of picking a row up, in tiles

// dynamic LDS, in bytes from the start
constexpr int OFF_WSUM = NW * WAVE_LDS;                         // int[NW]
constexpr int OFF_MISC = OFF_WSUM + NW * 4;                     // int[4]: spare
constexpr int OFF_SLOT = (OFF_MISC + 16 + 255) & ~255;          // [NW][2][SLOT_BYTES] list / mask words in flight;
                                                                // a wave's (m, l) table of the wave merge uses them afterwards
constexpr int OFF_SCAT = OFF_SLOT + NW * 2 * SLOT_BYTES;        // list: row offsets between two gathers; mask: uint[NW][POS_CAP] positions of a wave's next tiles
constexpr int POS_CAP = 240;                                    // (what the LDS leaves)
constexpr int MAX_ROWS_LIST = ATTN_MFMA_MAX_ROWS_LIST;
constexpr int FEW_ROWS = 64;                                    // rows a single wave scans by itself
// Where the kept positions of a row come from: an index list in memory (also chunk lists and dense calls, which
// have no list at all), or the kept-position mask and per-block counts of the selection (fused call).
enum Source { LIST = 0, MASK = 1 };
// What a kernel is built for: up to FEW_ROWS rows with lists of single positions (or the mask), as many rows with chunk lists or no
// lists, any number of rows.  A launch starts with cold instruction caches, and what it does not need is jumped over and held in
// registers all the same.  One form for all calls / these three, us, with the selection: 8 rows of 8192 18.6 / 18.2, 16 of 8192 (d = 64) 18.3 /
// 17.7, 64 of 13001 44.3 / 43.6, 32 of 2044 in chunks with new tokens 17.8 / 17.4, 16 layers of 64 rows of 32768 777 / 770, over the mask 835 / 830; 512
// ragged rows 548.3 / 547.9.
enum Form { FEW_POSITIONS = 0, FEW_ANY = 1, MANY = 2 };
constexpr int off_q(int src) { return OFF_SCAT + NW * (src == MASK ? POS_CAP * 4 : 256); }   // Q tile [NQT * 16 rows], chunks swizzled like K
constexpr int lds_bytes(int src) { return 157956 + off_q(src) - off_q(LIST); }
// Rows a launch of NQT query tiles can take: what the LDS leaves for the row tables behind the Q tile.
constexpr int launch_rows(int nqt, int d) { return d == 128 && nqt == 3 ? 1024 : d == 128 && nqt == 4 ? ATTN_MFMA_MAX_ROWS : MAX_ROWS_LIST; }
// Behind Q: the row tables (cost prefix and kept counts of up to ROWS rows).  Calls of up to 64 rows hold their rows in registers; with three and four query tiles, copies of them lie in the first kilobyte.
// The mask source then uses the rest of the region for the block counts of all rows.
template <int NQT, int D, int SRC> struct Tables {
    static constexpr int Q_BYTES = NQT <= 2 ? 8192 : NQT * 16 * Geo<D>::ROW_BYTES;
    static constexpr int ROWS = launch_rows(NQT, D);
    static constexpr int OFF_TAB = off_q(SRC) + Q_BYTES;
    static constexpr int TAB_BYTES = (2 * ROWS + 1) * 4;        // int[rows + 1] cost prefix, int[rows] kept counts, clamped
    static constexpr int OFF_BC = OFF_TAB + 1024;               // int[BC_ALL] block counts of all rows (mask source, <= FEW_ROWS rows)
    static constexpr int BC_ALL = (TAB_BYTES - 1024) / 4 / THREADS * THREADS < 2048 ? (TAB_BYTES - 1024) / 4 / THREADS * THREADS : 2048;
    static_assert((2 * FEW_ROWS + 1) * 4 <= 1024 && BC_ALL > 0, "the block counts must fit behind the tables of a small call");
    static_assert(OFF_TAB + TAB_BYTES <= lds_bytes(SRC), "the tables must fit");
};
static_assert(4 * 16 * 2 * 4 <= 2 * SLOT_BYTES, "a wave's (m, l) table must fit its slots");
static_assert(lds_bytes(MASK) * WG_PER_CU <= 160 * 1024 && lds_bytes(LIST) <= lds_bytes(MASK), "the workgroups of a CU must fit its LDS");

// Where the gathered rows live.  A list entry is a logical position (contiguous layout) or a pool
// slot page * page_size + offset (paged layouts; logical positions are mapped through the page
// table when the tile's row offsets are formed).
enum Layout { CONTIGUOUS = 0, PAGE_TABLE = 1, PHYSICAL = 2 };

// Row offsets are held in 32 bits, in units of 2^unit_shift bytes.  Rows of 64 elements in pools: whole rows of 128 bytes
// (512 GiB, more than a GPU has); the host sends strides that are no multiple of a row to the fp32 kernel.
template <int D, int LAYOUT> constexpr int unit_shift() { return D == 64 && LAYOUT != CONTIGUOUS ? 7 : 4; }

struct KvMap {
    int64_t base, stride_n, stride_page;
    const int32_t *ptab;
    int page_shift;
    // row offsets (units of 2^UNIT bytes, relative to `base`) of N positions, the page-table loads (if any) in flight together.
    // (Strides are whole units, so 32-bit products give the offsets' 32 bits: an eighth of the instructions of 64-bit ones.)
    template <int LAYOUT, int UNIT, int N> __device__ __forceinline__ void rel_n(const int (&idx)[N], uint32_t (&off)[N]) const
    {
        const uint32_t step = (uint32_t)(stride_n >> (UNIT - 1));
        if (LAYOUT == CONTIGUOUS) {
#pragma unroll
            for (int i = 0; i < N; ++i) off[i] = (uint32_t)idx[i] * step;
            return;
        }
        const uint32_t page_step = (uint32_t)(stride_page >> (UNIT - 1));
        const int mask = (1 << page_shift) - 1;
        int page[N];
#pragma unroll
        for (int i = 0; i < N; ++i) page[i] = LAYOUT == PAGE_TABLE ? ptab[idx[i] >> page_shift] : (idx[i] >> page_shift);
#pragma unroll
        for (int i = 0; i < N; ++i) off[i] = (uint32_t)page[i] * page_step + (uint32_t)(idx[i] & mask) * step;
    }
};

template <int LAYOUT> __device__ __forceinline__ KvMap make_map(const AttnLaunch &a, int b, int h)
{
    KvMap m;
    m.base = LAYOUT == CONTIGUOUS ? (int64_t)b * a.kv_stride_b + (int64_t)h * a.kv_stride_h : (int64_t)h * a.kv_stride_h;
    m.stride_n = a.kv_stride_n;
    m.stride_page = a.kv_stride_page;
    m.ptab = LAYOUT == PAGE_TABLE ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    m.page_shift = a.page_shift;
    return m;
}

// LDS reads are issued by hand, each batch together with its wait in one asm block: the compiler
// then neither adds waits for the gathers still in flight (it cannot tell them from the data being
// read) nor touches a result register before the data has arrived.
// Fragments of a tile's keys: 16-row tile pt, k-step c (32 elements) at address base ^ (64 c), 16-row tiles
// 4096 (d = 128) or 2048 bytes apart.
template <int D> struct KFrags { u32x4 f[Geo<D>::PT][Geo<D>::KS]; };
__device__ __forceinline__ void lds_read_k(KFrags<128> &k, uint32_t base)
{
    asm volatile(
        "ds_read_b128 %0, %8\n ds_read_b128 %1, %9\n ds_read_b128 %2, %10\n ds_read_b128 %3, %11\n"
        "ds_read_b128 %4, %8 offset:4096\n ds_read_b128 %5, %9 offset:4096\n"
        "ds_read_b128 %6, %10 offset:4096\n ds_read_b128 %7, %11 offset:4096\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(k.f[0][0]), "=&v"(k.f[0][1]), "=&v"(k.f[0][2]), "=&v"(k.f[0][3]),
          "=&v"(k.f[1][0]), "=&v"(k.f[1][1]), "=&v"(k.f[1][2]), "=&v"(k.f[1][3])
        : "v"(base), "v"(base ^ 64u), "v"(base ^ 128u), "v"(base ^ 192u)
        : "memory");
}
__device__ __forceinline__ void lds_read_k(KFrags<64> &k, uint32_t base)
{
    asm volatile(
        "ds_read_b128 %0, %8\n ds_read_b128 %1, %9\n"
        "ds_read_b128 %2, %8 offset:2048\n ds_read_b128 %3, %9 offset:2048\n"
        "ds_read_b128 %4, %8 offset:4096\n ds_read_b128 %5, %9 offset:4096\n"
        "ds_read_b128 %6, %8 offset:6144\n ds_read_b128 %7, %9 offset:6144\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(k.f[0][0]), "=&v"(k.f[0][1]), "=&v"(k.f[1][0]), "=&v"(k.f[1][1]),
          "=&v"(k.f[2][0]), "=&v"(k.f[2][1]), "=&v"(k.f[3][0]), "=&v"(k.f[3][1])
        : "v"(base), "v"(base ^ 64u)
        : "memory");
}
// The Q fragments of 16-row query tile QT from the Q tile staged in LDS.
template <int D> struct QFrags { u32x4 f[Geo<D>::KS]; };
template <int QT> __device__ __forceinline__ void lds_read_q(QFrags<128> &q, uint32_t base)
{
    asm volatile(
        "ds_read_b128 %0, %4 offset:%8\n ds_read_b128 %1, %5 offset:%8\n ds_read_b128 %2, %6 offset:%8\n ds_read_b128 %3, %7 offset:%8\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(q.f[0]), "=&v"(q.f[1]), "=&v"(q.f[2]), "=&v"(q.f[3])
        : "v"(base), "v"(base ^ 64u), "v"(base ^ 128u), "v"(base ^ 192u), "i"(QT * 4096)
        : "memory");
}
template <int QT> __device__ __forceinline__ void lds_read_q(QFrags<64> &q, uint32_t base)
{
    asm volatile(
        "ds_read_b128 %0, %2 offset:%4\n ds_read_b128 %1, %3 offset:%4\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(q.f[0]), "=&v"(q.f[1])
        : "v"(base), "v"(base ^ 64u), "i"(QT * 2048)
        : "memory");
}
// Transposing reads: within each group of 16 lanes, lane i receives element i%4 of the four 8-byte
// rows addressed by lanes i/4, i/4+4, i/4+8 and i/4+12.  One batch of a tile's values: four dv tiles (addresses
// base ^ (32 t)), both 16-row halves of 32 positions.  d = 128: batch b holds dv tiles 4 b .. 4 b + 3; d = 64: batch b
// holds positions 32 b .. 32 b + 31.
struct VFrags { u32x2 f[4][2]; };     // [dv tile][half]
template <int LO, int HI> __device__ __forceinline__ void lds_read_v(VFrags &v, uint32_t base)
{
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%12\n ds_read_b64_tr_b16 %1, %8 offset:%13\n"
        "ds_read_b64_tr_b16 %2, %9 offset:%12\n ds_read_b64_tr_b16 %3, %9 offset:%13\n"
        "ds_read_b64_tr_b16 %4, %10 offset:%12\n ds_read_b64_tr_b16 %5, %10 offset:%13\n"
        "ds_read_b64_tr_b16 %6, %11 offset:%12\n ds_read_b64_tr_b16 %7, %11 offset:%13\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v.f[0][0]), "=&v"(v.f[0][1]), "=&v"(v.f[1][0]), "=&v"(v.f[1][1]),
          "=&v"(v.f[2][0]), "=&v"(v.f[2][1]), "=&v"(v.f[3][0]), "=&v"(v.f[3][1])
        : "v"(base), "v"(base ^ 32u), "v"(base ^ 64u), "v"(base ^ 96u), "i"(LO), "i"(HI)
        : "memory");
}
template <int D, int B> __device__ __forceinline__ void lds_read_v_batch(VFrags &v, uint32_t base)
{
    if constexpr (D == 128) lds_read_v<0, 4096>(v, base ^ (uint32_t)(B * 128));
    else lds_read_v<B * 4096, B * 4096 + 2048>(v, base);
}
// The 8 words a lane needs of a tile's: words addr/4, addr/4 + STEP, ...
template <int STEP> __device__ __forceinline__ void lds_read_entries(uint32_t (&e)[8], uint32_t addr)
{
    asm volatile(
        "ds_read_b32 %0, %8\n ds_read_b32 %1, %8 offset:%9\n ds_read_b32 %2, %8 offset:%10\n"
        "ds_read_b32 %3, %8 offset:%11\n ds_read_b32 %4, %8 offset:%12\n ds_read_b32 %5, %8 offset:%13\n"
        "ds_read_b32 %6, %8 offset:%14\n ds_read_b32 %7, %8 offset:%15\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(e[0]), "=&v"(e[1]), "=&v"(e[2]), "=&v"(e[3]), "=&v"(e[4]), "=&v"(e[5]), "=&v"(e[6]), "=&v"(e[7])
        : "v"(addr), "i"(4 * STEP), "i"(8 * STEP), "i"(12 * STEP), "i"(16 * STEP), "i"(20 * STEP), "i"(24 * STEP), "i"(28 * STEP)
        : "memory");
}
template <int STEP> __device__ __forceinline__ void lds_write_entries(const uint32_t (&e)[8], uint32_t addr)
{
    asm volatile(
        "ds_write_b32 %8, %0\n ds_write_b32 %8, %1 offset:%9\n ds_write_b32 %8, %2 offset:%10\n"
        "ds_write_b32 %8, %3 offset:%11\n ds_write_b32 %8, %4 offset:%12\n ds_write_b32 %8, %5 offset:%13\n"
        "ds_write_b32 %8, %6 offset:%14\n ds_write_b32 %8, %7 offset:%15"
        :: "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]),
           "v"(addr), "i"(4 * STEP), "i"(8 * STEP), "i"(12 * STEP), "i"(16 * STEP), "i"(20 * STEP), "i"(24 * STEP), "i"(28 * STEP)
        : "memory");
}
__device__ __forceinline__ uint32_t lds_read_word(uint32_t addr)
{
    uint32_t v;
    asm volatile("ds_read_b32 %0, %1\n s_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(addr) : "memory");
    return v;
}
__device__ __forceinline__ void lds_write_word(uint32_t addr, uint32_t v)
{
    asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// One word from global memory, waited for on the spot.  Written out because a load the compiler tracks makes it wait
// for everything in flight (the gathers included) wherever the loaded value may be used, taken or not.
__device__ __forceinline__ uint32_t global_read_word(const uint32_t *p)
{
    uint32_t r;
    asm volatile("global_load_dword %0, %1, off\n s_waitcnt vmcnt(0)" : "=&v"(r) : "v"(p) : "memory");
    return r;
}
// Index of the k-th set bit of x (k = 0 is the lowest; k must be below the number of set bits).
__device__ __forceinline__ int kth_set_bit(uint32_t x, int k)
{
    int r = 0, c;
    c = __popc(x & 0xffffu); if (k >= c) { k -= c; r = 16; x >>= 16; }
    c = __popc(x & 0xffu);   if (k >= c) { k -= c; r += 8; x >>= 8; }
    c = __popc(x & 0xfu);    if (k >= c) { k -= c; r += 4; x >>= 4; }
    c = __popc(x & 0x3u);    if (k >= c) { k -= c; r += 2; x >>= 2; }
    c = (int)(x & 1u);       if (k >= c) { r += 1; }
    return r;
}
// Workgroup barrier for data handed over through LDS only: waits for this wave's LDS operations, not for its
// outstanding global loads (a plain __syncthreads() also waits for every gather and prefetch still in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory"); }

// Waits on the vector-memory counter with a run-time count (the instruction takes an immediate).
__device__ __forceinline__ void vm_wait(int n)
{
    switch (n) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 9: asm volatile("s_waitcnt vmcnt(9)" ::: "memory"); break;
    case 16: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
    case 17: asm volatile("s_waitcnt vmcnt(17)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

// What a launch hands to both kernels.  The divisors are known on the host, so the divisions by them are multiplications here.
struct Plan {
    float *part_ml;           // [slots][16 * NQT][2]
    float *part_o;            // [slots][16 * NQT][d]
    uint32_t *row_parts;      // [rows] in the workspace: the shares that hold a row's first (low half) and last tile, or ROW_EMPTY
    int n_wg;
    int unit_line;            // calls of up to so many tiles are cut into shares of single rows (share_units), or -1
    uint32_t per_share;       // 2^32 / (their number to aim for), rounded up
    int heads, group;         // query heads per kv head: in all, and in this launch
    uint32_t per_h, per_t;    // 2^31 / H_kv and 2^16 / T, rounded up
};
constexpr uint32_t ROW_EMPTY = 0xffffffffu;
// r / H_kv for r < 2^20, H_kv < 2^11, and q / T for q < 2^12, T < 2^4 (the rounding of the reciprocal stays below one part)
__device__ __forceinline__ int div_h(const Plan &p, int r) { return (int)__umulhi((uint32_t)r << 1, p.per_h); }
__device__ __forceinline__ int div_t(const Plan &p, int q) { return (int)(((uint32_t)q * p.per_t) >> 16); }

// Cost of a row on the line the workgroups share out: its tiles, plus SEG_COST for picking the row up
// (fresh Q, partial write), so that workgroups holding many short rows get fewer tiles.
template <int TILE> __device__ __forceinline__ int row_cost(int count) { return count > 0 ? (count + TILE - 1) / TILE + SEG_COST : 0; }

// The positions row r of sequence b attends to; PLAIN: as many as its list or mask has.
template <bool PLAIN> __device__ __forceinline__ int row_positions(const AttnLaunch &a, int r, int b)
{
    return PLAIN ? min(max(a.counts[r], 0), a.idx_capacity) : attn_row_count(a, r, b);
}

// Exclusive prefix of the row costs into pre[0..rows], every workgroup for itself (more than FEW_ROWS rows).
template <int TILE, int TABLE_ROWS> __device__ __forceinline__ void cost_prefix(const AttnLaunch &a, const Plan &plan, int rows, int *pre, int *cnt, int *wsum)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Many rows: THREADS rows per round (the counts of all rounds are requested at once), a wave-wide scan, the
    // wave totals through LDS, the rounds before carried along.
    constexpr int ROUNDS = (TABLE_ROWS + THREADS - 1) / THREADS;
    int c[ROUNDS];
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        const int rr = k * THREADS + tid;
        c[k] = rr < rows ? attn_row_count(a, rr, div_h(plan, rr)) : 0;
    }
    int carry = 0;
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        if (k * THREADS >= rows) break;                  // (uniform)
        const int rr = k * THREADS + tid;
        const int cost = row_cost<TILE>(c[k]);
        const int inc = wave_inclusive_sum(cost);
        if (rr < rows) cnt[rr] = c[k];
        if (lane == 63) wsum[wave] = inc;
        lds_barrier();
        int base = carry, all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int s = wsum[w];
            if (w < wave) base += s;
            all += s;
        }
        if (rr < rows) pre[rr] = base + inc - cost;
        carry += all;
        lds_barrier();                                   // the wave totals are rewritten by the next round
    }
    if (tid == 0) pre[rows] = carry;
    lds_barrier();
}

// The share [c0, c1) of the cost line a workgroup takes, and where a row's tiles fall inside it: tile k of
// row r sits at pre[r] + SEG_COST + k.
template <int TILE> struct Share {
    int c0, c1;
    // local tile range of row r inside the share; empty when lt_begin >= lt_end
    __device__ __forceinline__ void seg_range(const int *pre, const int *cnt, int r, int &lt_begin, int &lt_end) const
    {
        const int tiles = (cnt[r] + TILE - 1) / TILE;
        const int lo = c0 - pre[r] - SEG_COST, hi = c1 - pre[r] - SEG_COST;
        lt_begin = lo < 0 ? 0 : (lo > tiles ? tiles : lo);
        lt_end = hi < 0 ? 0 : (hi > tiles ? tiles : hi);
    }
    // first row at or after r with work for this workgroup, or `rows`
    __device__ __forceinline__ int next_seg(const int *pre, const int *cnt, int rows, int r) const
    {
        for (; r < rows && pre[r] < c1; ++r) {
            int lb, le;
            seg_range(pre, cnt, r, lb, le);
            if (lb < le) return r;
        }
        return rows;
    }
    // first row with work for this workgroup, or `rows`
    __device__ __forceinline__ int first_seg(const int *pre, const int *cnt, int rows) const
    {
        int lo = 0, hi = rows;                      // row holding cost c0: pre[r] <= c0 < pre[r+1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= c0) lo = mid; else hi = mid;
        }
        return next_seg(pre, cnt, rows, lo);
    }
};
// floor(a / b) for 0 <= a < 2^52, 0 < b < 2^31 in one fp64 division instead of the long 64-bit integer division
// sequence: both operands are exact in fp64, the correctly rounded quotient can only reach the next integer from
// below when a / b is within 2^-53 of it, and a true quotient that is no integer lies at least 1 / b below it.
__host__ __device__ __forceinline__ int floor_div(int64_t a, int b)
{
    return (int)floor((double)a / (double)b);
}

// The first n = min(n_wg, total) workgroups share the line.  Equal shares: workgroup w takes [w * total / n, (w + 1) * total / n), which
// differ by one unit at most.  None is empty, tilted ones neither (every workgroup between the first and the last of a row therefore holds
// tiles of that row, which the merge relies on).
// Long shares are tilted (TILT_FROM): while all XCDs read, those of odd number mostly stream more slowly, and with equal shares their
// workgroups end 4 to 7 % later (the rest of the spread has no fixed place; a plain read of 1 GiB in equal parts: even XCDs 132 us, odd
// ones 150).  So the shares of even XCDs are TILT / 128 larger than the mean, those of odd ones as much smaller: of the four shares of a
// team (share_index) two are of either kind, so boundaries 2 k stay where they are and the others move by TILT / 128 of a share.
// TILT 0 / 4 / 6 / 8 / 12, us: 16 layers of 64 rows of 32768 with their selection 799 / 787 / 786 / 789 / 798 (mask source 834 / 817 / 817 /
// 821 / 833), dense rows of up to 32768 109.6 / 108.4 / 108.2 / 108.1 / 110.0.  TILT 0 / 5 / -5: 16 layers 786 / 772 / 788, 512 ragged rows
// 512 / 508 / 520.  It does not help every call: over 40 of one layer (32 to 320 rows, 38 to 122 units a share) it gives 0.6 % on average,
// from 2.7 faster to 1.6 slower, the slower ones 128 rows with shares of 50 units and 256 rows with 65 to 80; rows of random
// positions have taken up to 2.5 % longer.
constexpr int TILT = 5;
// Lines whose shares are tilted: of TILT_FROM tiles a share or more, as little as moved boundaries cost (equal / tilted, us: 64 rows of 120
// tiles, 30 a share, 30.5 / 31.0, of 15 times 256 tiles in 768 rows of five 31.5 / 32.8, 128 of 60 32.9 / 33.1; 64 rows of 20011 positions, 35
// a share, 31.0 / 30.5; the mean of TILT 4 and 6, 64 rows of 59 tiles a share 46.8 / 46.1, of 94 67.8 / 67.6).  Not where rows are so many that
// equal counts make every share whole rows: there a moved boundary costs a partial (256 rows of 30 tiles 30.4 / 33.6, of 60 48.8 / 52.7,
// 512 of 60 91.4 / 95.3).  Whole shares make the line a multiple of their number, and that is what is tested: it keeps the shares of
// other lines of that length equal too, one in 256 of those of uneven rows, which costs them what the tilt gives.
constexpr int TILT_FROM = 32;
// ... and only with the workgroups of a whole GPU, 32 on each of eight XCDs: on a partition of it a share's parity says nothing about an
// XCD that is known to be slower (with one XCD all shares are on the same one), and the shares stay equal.
constexpr int TILT_WORKGROUPS = 256;
template <int TILE> __host__ __device__ __forceinline__ Share<TILE> make_share(int total, int n_wg, int rows, int w)
{
    // (This is on the way to a workgroup's first request: no branches, and the usual numbers of workgroups are powers of two, for which a
    // shift gives the same floor as the division.)
    int move = ((w >> 1) ^ (w >> 2)) & 1 ? -TILT : TILT;       // of boundary w or w + 1, whichever is odd
    move = (n_wg == TILT_WORKGROUPS) & (total - SEG_COST * rows >= TILT_FROM * n_wg) & ((rows * 2 <= n_wg) | ((total & (n_wg - 1)) != 0)) ? move : 0;
    const int64_t from = (int64_t)(w * 128 + ((w & 1) ? move : 0)) * total, to = (int64_t)(w * 128 + 128 + ((w & 1) ? 0 : move)) * total;
    Share<TILE> s;
    s.c0 = (int)(from >> (38 - __builtin_clz(n_wg)));
    s.c1 = (int)(to >> (38 - __builtin_clz(n_wg)));
    if (__builtin_expect((n_wg & (n_wg - 1)) != 0, 0)) {       // (equal shares: share_index deals these to XCDs as they come)
        s.c0 = floor_div((int64_t)w * total, n_wg);
        s.c1 = floor_div((int64_t)(w + 1) * total, n_wg);
    }
    const bool units = total < n_wg;                           // fewer units than shares: one each
    s.c0 = min(units ? w : s.c0, total);
    s.c1 = min(units ? w + 1 : s.c1, total);
    return s;
}
// Which share of the line a workgroup takes.  The hardware deals workgroup i to XCD i mod 8; the owners of
// four consecutive shares (the usual team of a row) are four workgroups on four different XCDs, and the sets
// {x, x+1, x+3, x+6} rotate from team to team, so that every XCD serves half of the teams and a difference in
// speed between XCDs is spread over all rows.  (A bijection of 0 .. n_wg - 1 when n_wg is a multiple of 32.)
__host__ __device__ __forceinline__ int share_index(int wg, int n_wg)
{
    if (n_wg & 31) return wg;
    const int x = wg & 7, c = wg >> 3, m = c & 3;
    const int off = (0x6310 >> (4 * m)) & 7;
    const int team = ((c >> 2) << 3) | ((x - off) & 7);
    return (team << 2) | m;
}

// body(integral_constant<int, 0>) ... body(integral_constant<int, N - 1>)
template <int I> struct IntConst { static constexpr int value = I; };
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F &&body)
{
    if constexpr (I < N) {
        body(IntConst<I>{});
        static_for<N, I + 1>(body);
    }
}

// A row's partials (m, l, o) as they are joined, m in log2 units.
struct Merge {
    float m = -INFINITY, l = 0.0f, o = 0.0f;
    // N of them: their largest first, then weights that wait for nothing else, and sums in two chains.
    template <int N> __device__ __forceinline__ void add_all(const float (&mw)[N], const float (&lw)[N], const float (&ow)[N])
    {
        float top[N];
#pragma unroll
        for (int k = 0; k < N; ++k) top[k] = mw[k];
#pragma unroll
        for (int step = 1; step < N; step *= 2)
#pragma unroll
            for (int k = 0; k + step < N; k += 2 * step) top[k] = fmaxf(top[k], top[k + step]);
        const float mn = fmaxf(m, top[0]), ref = mn == -INFINITY ? 0.0f : mn;
        float f[N];
#pragma unroll
        for (int k = 0; k < N; ++k) f[k] = __builtin_amdgcn_exp2f(mw[k] - ref);
        const float fa = __builtin_amdgcn_exp2f(m - ref);
        float l2[2] = {l * fa, 0.0f}, o2[2] = {o * fa, 0.0f};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            l2[k & 1] = fmaf(f[k], lw[k], l2[k & 1]);
            o2[k & 1] = fmaf(f[k], ow[k], o2[k & 1]);
        }
        l = l2[0] + l2[1];
        o = o2[0] + o2[1];
        m = mn;
    }
};
// Sum and largest over the four lanes l, l + 16, l + 32, l + 48, in each of them (exchanged on the vector ALU, not through LDS).
template <typename F> __device__ __forceinline__ float over_rows(float x, F &&join)
{
    const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = join(__uint_as_float(v[0]), __uint_as_float(v[1]));
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return join(__uint_as_float(w[0]), __uint_as_float(w[1]));
}
__device__ __forceinline__ float sum_of_rows(float x) { return over_rows(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float max_of_rows(float x) { return over_rows(x, [](float a, float b) { return fmaxf(a, b); }); }

template <int D, int NQT, int LAYOUT, int SRC, bool F16, int FORM>
__global__ __launch_bounds__(THREADS, WG_PER_CU) void attn_mfma_kernel(AttnLaunch a, Plan plan)
{
    typedef typename Half<F16>::x8 h16x8;
    typedef typename Half<F16>::x2 h16x2;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    static_assert(D == 128 || SRC == LIST, "the mask source is built for 32-position tiles");
    typedef Geo<D> GEO;
    typedef Tables<NQT, D, SRC> TAB;
    constexpr int TILE = GEO::TILE, ROW_BYTES = GEO::ROW_BYTES, LPR = GEO::LPR, RPI = GEO::RPI, PT = GEO::PT, KS = GEO::KS, PB = GEO::PB, DT = GEO::DT;
    constexpr int UNIT = unit_shift<D, LAYOUT>();
    constexpr int QTP = NQT * 16;
    constexpr int QCH = NQT * 16 * LPR;                                 // 16-byte chunks of the Q tile
    constexpr int QROUNDS = (QCH + THREADS - 1) / THREADS;              // chunks per thread
    // Parts the softmax weights are handed over in: 16 significant bits with two of bf16, 22 with two of fp16, 24 with three
    // (d = 64, where the products have time to spare).
    constexpr int NP = D == 64 ? 3 : 2;
    constexpr bool TIGHT = NQT >= 3;                                    // registers are short: what the tile loop can fetch again is not held
    constexpr bool FOLD = !TIGHT && UNIT == 4;                          // a lane's chunk of a row is part of the row offset it holds
    constexpr int QG = NQT <= 2 ? NQT : 1;                              // query tiles whose scores are held at a time
    constexpr bool few_rows = FORM != MANY;                             // the launch has at most FEW_ROWS rows
    constexpr bool PLAIN = FORM == FEW_POSITIONS || SRC == MASK;        // ranks are single positions of a list or mask
    const bool dense = !PLAIN && a.dense;
    const int chunk_shift = PLAIN ? 0 : a.chunk_shift;
    const int rows = a.B * a.H_kv;
    int *pre = reinterpret_cast<int *>(smem + TAB::OFF_TAB);
    int *cnt_lds = pre + ((few_rows ? FEW_ROWS : TAB::ROWS) + 1);
    int *wsum = reinterpret_cast<int *>(smem + OFF_WSUM);
    char *q_lds = smem + off_q(SRC);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int l16 = lane & 15, g = lane >> 4;
    char *wave_lds = smem + wave * WAVE_LDS;
    char *slot_lds = smem + OFF_SLOT + wave * 2 * SLOT_BYTES;
    float *mlw = reinterpret_cast<float *>(smem + OFF_SLOT);            // wave w's (m, l): [w * 128 + q * 2 * NQT + ...]
    const uint32_t ks_addr = (uint32_t)(uintptr_t)LDS_PTR(char, wave_lds);
    const uint32_t vs_addr = ks_addr + TILE_BYTES;
    const uint32_t slot_addr = (uint32_t)(uintptr_t)LDS_PTR(char, slot_lds);
    const uint32_t scat_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem + OFF_SCAT + wave * (SRC == MASK ? POS_CAP * 4 : 256));
    const uint32_t q_addr = (uint32_t)(uintptr_t)LDS_PTR(char, q_lds);
    // K fragment of k-step c: row l16 (+16 per position tile), 16-byte chunk 4c + g - address k_off ^ (64 c)
    uint32_t k_off = ks_addr + (uint32_t)(l16 * ROW_BYTES + ((g ^ GEO::swz(l16)) << 4));
    // Q fragment of k-step c: same pattern on the Q tile (row = query row l16, +16 per query tile)
    uint32_t q_off = q_addr + (k_off - ks_addr);
    // V^T fragment of dv tile t: source lane points at row 4g + l16/4 (+16 per half), 4 values from
    // column 16t + 4*(l16%4) - address v_off ^ (32 t)
    uint32_t v_off;
    {
        const int row = 4 * g + (l16 >> 2);
        v_off = vs_addr + (uint32_t)(row * ROW_BYTES + ((((l16 & 3) >> 1) ^ GEO::swz(row)) << 4) + ((l16 & 1) << 3));
    }
    // gather instruction i moves rows RPI*i ...; this lane fetches a chunk of row RPI*i + lrow: chunk (lane % LPR) ^ swz(row).
    // swz depends on i only through bits that i has to itself, so the byte offset is lane_chunk ^ (a constant of i).
    int lrow = lane / LPR;
    uint32_t lane_chunk = (uint32_t)(((lane & (LPR - 1)) ^ GEO::swz(lrow)) << 4);
    auto chunk_flip = [](int i) -> uint32_t { return D == 128 ? ((i & 1) << 7) | ((i & 2) << 3) : (i & 1) << 4; };

    // Every kernel argument the main path uses, in one batch.
    SPECATTN_PRELOAD(a.q); SPECATTN_PRELOAD(a.k); SPECATTN_PRELOAD(a.v);
    SPECATTN_PRELOAD(a.B); SPECATTN_PRELOAD(a.H_q); SPECATTN_PRELOAD(a.H_kv); SPECATTN_PRELOAD(a.T);
    SPECATTN_PRELOAD(a.sm_scale);
    SPECATTN_PRELOAD(a.q_stride_b); SPECATTN_PRELOAD(a.q_stride_h); SPECATTN_PRELOAD(a.q_stride_t);
    SPECATTN_PRELOAD(a.kv_stride_b); SPECATTN_PRELOAD(a.kv_stride_h); SPECATTN_PRELOAD(a.kv_stride_n);
    SPECATTN_PRELOAD(a.counts); SPECATTN_PRELOAD(a.idx_capacity);
    if (!PLAIN) { SPECATTN_PRELOAD(a.dense); SPECATTN_PRELOAD(a.chunk_shift); }
    SPECATTN_PRELOAD(a.g_first); SPECATTN_PRELOAD(a.k_new);
    SPECATTN_PRELOAD(a.out); SPECATTN_PRELOAD(a.out_lowp); SPECATTN_PRELOAD(a.lse);
    SPECATTN_PRELOAD(plan.part_ml); SPECATTN_PRELOAD(plan.part_o); SPECATTN_PRELOAD(plan.row_parts);
    SPECATTN_PRELOAD(plan.n_wg); SPECATTN_PRELOAD(plan.unit_line); SPECATTN_PRELOAD(plan.per_share); SPECATTN_PRELOAD(plan.heads); SPECATTN_PRELOAD(plan.group); SPECATTN_PRELOAD(plan.per_h); SPECATTN_PRELOAD(plan.per_t);
    if (LAYOUT != CONTIGUOUS) { SPECATTN_PRELOAD(a.page_table); SPECATTN_PRELOAD(a.page_shift); SPECATTN_PRELOAD(a.max_pages); SPECATTN_PRELOAD(a.kv_stride_page); }
    if (SRC == LIST) { SPECATTN_PRELOAD(a.indices); SPECATTN_PRELOAD(a.idx_stride); }
    if (SRC == MASK) { SPECATTN_PRELOAD(a.kept_mask); SPECATTN_PRELOAD(a.block_counts); SPECATTN_PRELOAD(a.blocks_per_row); SPECATTN_PRELOAD(a.n_max); }
    // Mask source, small calls: the per-block kept counts of all rows are requested together with the counts (the row
    // this workgroup starts in is not known yet), so that its first segment need not go to memory for them again.
    constexpr int BC_PT = TAB::BC_ALL / THREADS;
    int *bc_lds = reinterpret_cast<int *>(smem + TAB::OFF_BC);
    const bool bc_all = SRC == MASK && few_rows && rows * a.blocks_per_row <= TAB::BC_ALL;
    int bc_pf[BC_PT];
    if (bc_all) {
#pragma unroll
        for (int k = 0; k < BC_PT; ++k) {
            const int j = tid + k * THREADS;
            bc_pf[k] = a.block_counts[j < rows * a.blocks_per_row ? j : 0];
        }
    }
    // Every workgroup finds the cost line by itself.  Up to 64 rows, lane i of every wave holds row i: counts, prefix, share and
    // every row's local tile range without a table, a barrier or a search; more rows go through tables in LDS.
    int row_lo = 0, row_cnt = 0, total;                  // few rows: cost prefix and kept count of row `lane`
    int unit = 0;                                        // tiles of a share that is a part of one row, or 0: a share of the line
    if constexpr (few_rows) {
        row_cnt = lane < rows ? row_positions<PLAIN>(a, lane, div_h(plan, lane)) : 0;
        const int cost = row_cost<TILE>(row_cnt), inc = wave_inclusive_sum(cost);
        row_lo = inc - cost;
        total = __builtin_amdgcn_readlane(inc, 63);      // (lanes past the last row add nothing)
        // Few tiles in all: shares of `unit` tiles of one row each (share_units)
        const int tiles = total - SEG_COST * (int)__popcll(__ballot(row_cnt > 0));
        if (tiles <= plan.unit_line) {                   // (uniform)
            const int least = (int)__umulhi((uint32_t)(tiles > 0 ? tiles - 1 : 0), plan.per_share) + 1;
            unit = ((least <= 3) & (tiles > 4 * rows) & (tiles <= 128)) ? 3 : least <= 4 ? 4 : least <= 6 ? 6 : (least + 3) & ~3;
            // (exact: fewer than 2^16 tiles, and half a tile is more than the reciprocal is off)
            const int parts = (int)(((float)((row_cnt + TILE - 1) / TILE + unit - 1) + 0.5f) * __builtin_amdgcn_rcpf((float)unit));
            const int parts_inc = wave_inclusive_sum(parts);
            row_lo = (parts_inc - parts) * unit;
            total = __builtin_amdgcn_readlane(parts_inc, 63) * unit;
        }
        if (TIGHT) { pre[lane] = row_lo; cnt_lds[lane] = row_cnt; }     // (every wave the same values, and a wave reads behind its own)
        if (blockIdx.x == 0 && tid < rows && row_cnt == 0) plan.row_parts[tid] = ROW_EMPTY;
    } else {
        cost_prefix<TILE, TAB::ROWS>(a, plan, rows, pre, cnt_lds, wsum);
        total = pre[rows];
        if (blockIdx.x == 0)
            for (int rr = tid; rr < rows; rr += THREADS)
                if (cnt_lds[rr] == 0) plan.row_parts[rr] = ROW_EMPTY;
    }
    if (bc_all) {
#pragma unroll
        for (int k = 0; k < BC_PT; ++k) bc_lds[tid + k * THREADS] = bc_pf[k];   // (read behind the first segment's barrier)
    }
    // Everything loaded so far has arrived, which the compiler does not see where the block counts are requested and used under a condition each: it
    // would wait for the first gathers before it gives those registers to others.
    if (SRC == MASK) __builtin_amdgcn_s_waitcnt(0x0f70);             // vmcnt(0)
    const int QT = plan.group * a.T;
    const float scale2 = a.sm_scale * 1.4426950408889634f;            // scores in log2 units

    // The Q tile of a segment goes straight into LDS: wave w fetches 16-byte slots 64 w .. of it (and of its second 8 KiB), swizzled like
    // K rows.  Query rows past the last one repeat it: their results are not written.
    auto load_q = [&](int rr) {
        const int b = div_h(plan, rr), h = rr - b * a.H_kv;
#pragma unroll
        for (int k = 0; k < QROUNDS; ++k) {
            if (k * THREADS + wave * 64 >= QCH) break;   // (uniform over the wave)
            const int row = k * (THREADS / LPR) + tid / LPR, qi = min(row, QT - 1);
            const int gh = div_t(plan, qi), tt = qi - gh * a.T;
            const uint16_t *qp = static_cast<const uint16_t *>(a.q) + (int64_t)b * a.q_stride_b +
                                 (int64_t)attn_query_head(a, plan.heads, h, gh) * a.q_stride_h + (int64_t)tt * a.q_stride_t;
            __builtin_amdgcn_global_load_lds(GLOBAL_PTR(qp + ((tid & (LPR - 1)) ^ GEO::swz(row & 15)) * 8),
                                             LDS_PTR(void, q_lds + (k * THREADS + wave * 64) * 16), 16, 0, 0);
        }
    };
    const int n_q = wave * 64 >= QCH ? 0 : (QROUNDS == 1 || THREADS + wave * 64 >= QCH) ? 1 : 2;    // such loads of this wave

    // This workgroup's share of the cost line, and the rows of which it holds tiles
    const int my_share = __builtin_amdgcn_readfirstlane(share_index(blockIdx.x, plan.n_wg));
    total = __builtin_amdgcn_readfirstlane(total);
    Share<TILE> sh;
    sh.c0 = min(my_share * unit, total);
    sh.c1 = min(sh.c0 + unit, total);
    if (unit == 0) sh = make_share<TILE>(total, plan.n_wg, rows, my_share);
    const int seg_cost = unit ? 0 : SEG_COST;
    const int c0 = sh.c0, c1 = sh.c1;
    if (c0 >= c1) return;                                // more workgroups than units of work
    int my_lb = 0, my_le = 0;                            // few rows: local tile range of row `lane`
    unsigned long long seg_mask = 0;                     // few rows: the rows with tiles in this share
    auto local_tiles = [&]() {
        const int tiles = (row_cnt + TILE - 1) / TILE;
        const int lo = c0 - row_lo - seg_cost, hi = c1 - row_lo - seg_cost;
        my_lb = lo < 0 ? 0 : (lo > tiles ? tiles : lo);
        my_le = hi < 0 ? 0 : (hi > tiles ? tiles : hi);
    };
    if (few_rows) {
        local_tiles();
        seg_mask = __ballot(lane < rows && my_lb < my_le);
    }
    auto seg_range = [&](int r, int &lt_begin, int &lt_end) {
        if (few_rows) {
            const int ru = __builtin_amdgcn_readfirstlane(r);
            lt_begin = __builtin_amdgcn_readlane(my_lb, ru);
            lt_end = __builtin_amdgcn_readlane(my_le, ru);
        } else {
            sh.seg_range(pre, cnt_lds, r, lt_begin, lt_end);
        }
    };
    // first row at or after r with work for this workgroup, or `rows`
    auto next_seg = [&](int r) {
        if (few_rows) {
            const unsigned long long m = r < 64 ? (seg_mask >> r) << r : 0ull;
            return m ? (int)__ffsll((long long)m) - 1 : rows;
        }
        return sh.next_seg(pre, cnt_lds, rows, r);
    };
    int r = __builtin_amdgcn_readfirstlane(few_rows ? next_seg(0) : sh.first_seg(pre, cnt_lds, rows));

    bool first_seg = true;
    // The list words of the wave's first two tiles, ahead of everything else: the first gathers wait for them (counts -> list words ->
    // K/V rows are three dependent trips to memory), and what the compiler computes ahead of the loop then runs while they fly.
    auto row_count = [&](int r) { return few_rows ? __builtin_amdgcn_readlane(row_cnt, __builtin_amdgcn_readfirstlane(r)) : cnt_lds[r]; };
    // (ranks past the row's end read the last word again)
    auto request_words = [&](const int32_t *idx_row, int count, int t, int s) {
        int jj = t * TILE + (lane & (TILE - 1));
        jj = jj < count ? jj : count - 1;
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(idx_row + (jj >> chunk_shift)), LDS_PTR(void, slot_lds + s * SLOT_BYTES), 4, 0, 0);
    };
    if (r < rows) {
        if (SRC == LIST && !dense) {
            int lt_begin, lt_end;
            seg_range(r, lt_begin, lt_end);
            if (lt_begin + wave < lt_end) {
                const int32_t *idx_row = a.indices + (int64_t)r * a.idx_stride;
                request_words(idx_row, row_count(r), lt_begin + wave, 0);
                request_words(idx_row, row_count(r), lt_begin + wave + NW, 1);
            }
        }
        if (SRC == LIST) load_q(r);
    }

    while (r < rows) {
        int lt_begin, lt_end;
        if (TIGHT && few_rows && !first_seg) {           // (not held in registers through the tile loop)
            row_lo = pre[lane];
            row_cnt = cnt_lds[lane];
            local_tiles();
        }
        seg_range(r, lt_begin, lt_end);
        if (SRC == MASK) { lt_begin = __builtin_amdgcn_readfirstlane(lt_begin); lt_end = __builtin_amdgcn_readfirstlane(lt_end); }
        const int r_next = __builtin_amdgcn_readfirstlane(next_seg(r + 1));
        const int b = div_h(plan, r), h = r - b * a.H_kv;
        const int count = SRC == MASK ? __builtin_amdgcn_readfirstlane(row_count(r)) : row_count(r);
        const int tiles = (count + TILE - 1) / TILE;
        const KvMap map = make_map<LAYOUT>(a, b, h);
        const char *kbh = static_cast<const char *>(a.k) + map.base * 2;
        const char *vbh = static_cast<const char *>(a.v) + map.base * 2;
        const int32_t *idx_row = (SRC == LIST && !dense) ? a.indices + (int64_t)r * a.idx_stride : nullptr;
        const uint32_t *mask_row = SRC == MASK ? a.kept_mask + (int64_t)r * a.blocks_per_row * (SEL_BLOCK / 32) : nullptr;
        const int n_idx = (SRC == MASK || !dense) ? 1 : 0;            // LDS-DMA instructions per tile for list / mask words

        // ---- the wave's tiles --------------------------------------------------------------------------
        // list: tile k of the share goes to wave k mod NW; mask: every wave takes a run of tiles, whose positions it finds by itself
        constexpr int STEP = SRC == MASK ? 1 : NW;
        const int run = lt_end - lt_begin;
        const int t_first = lt_begin + (SRC == MASK ? run * wave / NW : wave);
        const int tile_end = SRC == MASK ? lt_begin + run * (wave + 1) / NW : lt_end;
        int t_cur = t_first, t_nxt = t_cur + STEP, t_nn = t_nxt + STEP;
        // Mask source.  A wave turns mask words into positions as it needs them, a few tiles' worth at a time: 64 words travel to LDS by
        // LDS-DMA an iteration ahead, lane w takes word w, a prefix sum over the bit counts gives its first rank, and its bits go one
        // after the other to their places in the wave's buffer.  As many words are taken as fit there.
        // Before, every tile was located and decoded by itself, with one rank to a lane, and a row's block prefix was a table behind two barriers: a
        // verify step of 16 layers x 64 rows of 32768 835.4 / 830.0 us, 12 x 8 rows of 30000 231.0 / 226.0, 8 x 24 rows of 12345 175.3 / 171.0, 4 x 192
        // rows of 16384 301.5 / 300.0.  Runs of tiles cost some of what they save, since a wave's rows then lie far from the other waves' (the list
        // source with such runs: 781 / 794 us); the tiles in turns, with the positions of a whole share found by the workgroup at once: 2 barriers
        // more ahead of the first gathers, 0.6 % slower than this.
        int p_at = 0, p_have = 0;                                       // the buffer holds the next p_have positions from entry p_at on
        int p_word = 0, p_skip = 0;                                     // the first word not taken yet; kept positions in it and behind to be passed over
        const int nw = SRC == MASK ? a.blocks_per_row * (SEL_BLOCK / 32) : 0;
        // Where the wave's first tile starts: the block that holds its first rank, and the block's kept positions ahead of it.
        auto mask_locate = [&](int t) {
            const int rank = t * TILE, nb = a.blocks_per_row;
            const int32_t *bc = a.block_counts + (int64_t)r * nb;
            int before = 0;
            for (int base = 0;; base += 64) {
                const int at = min(base + lane, nb - 1);
                int c = bc_all ? bc_lds[r * nb + at] : bc[at];
                c = base + lane < nb ? c : 0;
                const int inc = before + wave_inclusive_sum(c), all = __builtin_amdgcn_readlane(inc, 63);
                if (all > rank || base + 64 >= nb) {
                    const int ahead = min((int)__popcll(__ballot(inc <= rank)), min(63, nb - 1 - base));    // blocks that end ahead of it
                    p_skip = max(rank - __builtin_amdgcn_readlane(inc - c, ahead), 0);
                    p_word = (base + ahead) * (SEL_BLOCK / 32);
                    return;
                }
                before = all;
            }
        };
        // Requests what the wave's next gathers need (one LDS-DMA instruction): tile t's list words into slot s (tiles past the end: the
        // last tile's), or the next 64 mask words.
        auto request = [&](int t, int s) {
            if (SRC == MASK) {
                const int w = p_word + lane;
                __builtin_amdgcn_global_load_lds(GLOBAL_PTR(mask_row + (w < nw ? w : nw - 1)), LDS_PTR(void, slot_lds), 4, 0, 0);
            } else if (!dense) {
                request_words(idx_row, count, t < tiles ? t : tiles - 1, s);
            }
        };
        // Makes sure that the buffer holds the positions of tile t, which start at p_at.  `fresh`: the slot has the words from p_word on (requested
        // there, and arrived but for the newest 16 requests).  Rows so sparse that those do not hold the tile take further words from memory.
        auto positions = [&](int t, bool fresh) {
            const int need = (count - t * TILE) < TILE ? (count - t * TILE) : TILE;
            if (p_have < need) {
                if (p_at > 0) {                                         // what is left goes to the front
                    if (lane < p_have) lds_write_word(scat_addr + (uint32_t)lane * 4, lds_read_word(scat_addr + (uint32_t)(p_at + lane) * 4));
                    p_at = 0;
                }
                uint32_t bits;
                if (fresh) {
                    vm_wait(16);
                    bits = lds_read_word(slot_addr + (uint32_t)(lane * 4));
                }
                while (p_have < need && p_word < nw) {
                    if (!fresh) bits = global_read_word(mask_row + (p_word + lane < nw ? p_word + lane : nw - 1));
                    fresh = false;
                    if (p_word + lane >= nw) bits = 0u;
                    const int pc = __popc(bits), inc = wave_inclusive_sum(pc), skip = inc - pc - p_skip;
                    // whole words, as many as fit (the first one does, and 31 entries are left for the padding below)
                    const int taken = (int)__popcll(__ballot(inc - p_skip <= POS_CAP - (TILE - 1) - p_have));
                    const int got = __builtin_amdgcn_readlane(inc, taken - 1) - p_skip;
                    if (lane >= taken) bits = 0u;
                    if (p_skip > 0 && skip < 0) bits = -skip < pc ? bits & (~0u << kth_set_bit(bits, -skip < pc ? -skip : 0)) : 0u;
                    uint32_t at = scat_addr + (uint32_t)(p_have + (skip > 0 ? skip : 0)) * 4;
                    const int first = (p_word + lane) * 32;
                    while (bits) {
                        lds_write_word(at, (uint32_t)(first + __ffs((int)bits) - 1));
                        at += 4;
                        bits &= bits - 1;
                    }
                    p_have += got > 0 ? got : 0;
                    p_skip = got < 0 ? -got : 0;
                    p_word += taken;
                }
            }
            // (no wait: the buffer is read by this wave's own later LDS reads, which the LDS unit serves in order)
            if (need < TILE) {                                          // ranks past the end repeat the last kept position
                lds_wait();
                const uint32_t last_pos = lds_read_word(scat_addr + (uint32_t)(p_at + (need > 0 ? need : 1) - 1) * 4);
                if (lane >= need && lane < TILE) lds_write_word(scat_addr + (uint32_t)(p_at + lane) * 4, last_pos);
            }
        };
        // Row offsets (in units) of the 8 rows this lane helps to fetch for tile t, whose list words are in slot s (or whose positions
        // are the buffer's next, which are used up with this).
        auto entries = [&](int t, int s, uint32_t (&ent)[8]) {
            int pos[8];
            auto rank = [&](int i) -> int {                             // ranks past the end repeat the last kept position
                const int jj = t * TILE + RPI * i + lrow;
                return jj < count ? jj : count - 1;
            };
            if (SRC == MASK) {
                uint32_t e[8];
                lds_read_entries<RPI>(e, scat_addr + (uint32_t)((p_at + lrow) * 4));
                p_at += TILE;
                p_have = p_have > TILE ? p_have - TILE : 0;
                // (a mask that does not hold `count` bits would leave entries unwritten: stay inside the row)
#pragma unroll
                for (int i = 0; i < 8; ++i) pos[i] = e[i] < (uint32_t)a.n_max ? (int)e[i] : a.n_max - 1;
            } else if (dense) {
#pragma unroll
                for (int i = 0; i < 8; ++i) pos[i] = rank(i);
            } else {
                uint32_t e[8];
                lds_read_entries<RPI>(e, slot_addr + (uint32_t)(s * SLOT_BYTES + lrow * 4));
                const int cs = chunk_shift, low = (1 << cs) - 1;
#pragma unroll
                for (int i = 0; i < 8; ++i) pos[i] = (int)e[i];
                if (cs) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) pos[i] = (int)(e[i] << cs) | (rank(i) & low);
                }
            }
            map.rel_n<LAYOUT, UNIT>(pos, ent);
            if constexpr (FOLD) {
#pragma unroll
                for (int i = 0; i < 8; ++i) ent[i] += (lane_chunk ^ chunk_flip(i)) >> 4;
            }
        };
        // Where a tile's row offsets wait for the V gathers when they are not held in registers (the mask source has one slot to spare).
        auto stash_addr = [&]() { return (SRC == LIST ? scat_addr : slot_addr + (uint32_t)SLOT_BYTES) + (uint32_t)(lrow * 4); };
        // gather a tile's rows of one tensor into this wave's buffer: 8 instructions of 1 KiB
        auto issue = [&](const char *base, char *buf, const uint32_t (&ent)[8]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const char *src = base + ((int64_t)ent[i] << UNIT) + (FOLD ? 0u : lane_chunk ^ chunk_flip(i));
                __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src), LDS_PTR(void, buf + i * 1024), 16, 0, KV_AUX);
            }
        };

        // ---- start of the segment: the words of the wave's first two tiles are requested before anything else the
        //      segment needs, since the first gathers wait for them (counts -> list words -> K/V rows are three
        //      dependent trips to memory); then Q goes into LDS ---------------------------------------------------
        if (!first_seg) lds_barrier();           // the previous segment's readers of the wave buffers, slots and Q are done
        if (SRC == MASK && first_seg && bc_all) lds_barrier();          // the block counts of all rows are in LDS
        if (SRC == MASK || !first_seg) {
            if (t_cur < tile_end) {
                if (SRC == MASK) mask_locate(t_cur);
                request(t_cur, 0);
                if (SRC == LIST) request(t_nxt, 1);
            }
            load_q(r);
        }

        f32x4 o[NQT][DT];                    // O^T[dv = 16t + 4g + i][q = l16]
        float m_ref[NQT], l_sum[NQT];        // reference max (log2 units) and sum of weights
#pragma unroll
        for (int qt = 0; qt < NQT; ++qt) {
            m_ref[qt] = -INFINITY;
            l_sum[qt] = 0.0f;
#pragma unroll
            for (int t = 0; t < DT; ++t) o[qt][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }

        // The gathers and word requests are not tracked by the compiler's wait insertion; every wait on them is written out.  Order
        // of issue per wave and iteration: K(next) ... V(next) words(third).  The first gathers go out as soon as the list words are
        // there; Q, which the first product waits for, is waited for and shared behind them.  (Q through registers and a barrier ahead of the
        // gathers: 0.2 to 0.6 us more per launch.)
        uint32_t ent[8];
        if (t_cur < tile_end) {
            vm_wait(n_q);                                               // the words of the first two tiles are there
            if (SRC == MASK) positions(t_cur, true);
            entries(t_cur, 0, ent);
            issue(kbh, wave_lds, ent);
            issue(vbh, wave_lds + TILE_BYTES, ent);
            if (SRC == MASK && t_nxt < tile_end) positions(t_nxt, false);
            request(t_nn, 0);
            vm_wait(16 + n_idx);                                        // this wave's part of Q is there
        } else {
            vm_wait(0);
        }
        lds_barrier();
        if (t_cur < tile_end) {
            int s_nxt = 1;                                              // slot with the words of t_nxt; t_nn's is the other
            while (t_cur < tile_end) {
                const bool has_next = t_nxt < tile_end;
                // (keeps what is derived from these from being computed ahead of the loop and held)
                if (TIGHT) asm volatile("" : "+v"(lane_chunk), "+v"(k_off), "+v"(q_off), "+v"(v_off), "+v"(l16), "+v"(g), "+v"(lrow));
                vm_wait(8 + n_idx);                                     // K(cur) landed; V(cur) and the last request may be in flight

                h16x8 p_part[NP][NQT][PB];
                const int remaining = count - t_cur * TILE;            // > 0; < TILE only on a row's last tile
                {
                    KFrags<D> kf;
                    lds_read_k(kf, k_off);
                    if (has_next) {                                    // the K buffer is free again
                        entries(t_nxt, s_nxt, ent);
                        issue(kbh, wave_lds, ent);
                        if (TIGHT) lds_write_entries<RPI>(ent, stash_addr());
                    }
                    static_for<NQT / QG>([&](auto grp) {
                        constexpr int Q0 = decltype(grp)::value * QG;
                        // ---- S^T[pos][q] = K Q^T -------------------------------------------------------
                        f32x4 s[QG][PT];
                        static_for<QG>([&](auto sub) {
                            constexpr int qq = decltype(sub)::value;
                            QFrags<D> qf;
                            lds_read_q<Q0 + qq>(qf, q_off);
#pragma unroll
                            for (int pt = 0; pt < PT; ++pt) {
                                f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                for (int c = 0; c < KS; ++c)
                                    acc = Half<F16>::mfma(__builtin_bit_cast(h16x8, kf.f[pt][c]),
                                                          __builtin_bit_cast(h16x8, qf.f[c]), acc);
                                s[qq][pt] = acc;
                            }
                        });
                        // ---- softmax weights; lane (q = l16, g) holds positions 16pt + 4g + i -----------
#pragma unroll
                        for (int qq = 0; qq < QG; ++qq) {
                            const int qt = Q0 + qq;
                            constexpr int NE = 4 * PT;
                            float x[NE];
#pragma unroll
                            for (int e = 0; e < NE; ++e) x[e] = s[qq][e >> 2][e & 3];
                            if (remaining < TILE) {
#pragma unroll
                                for (int e = 0; e < NE; ++e)
                                    if (16 * (e >> 2) + 4 * g + (e & 3) >= remaining) x[e] = -INFINITY;
                            }
                            float mloc = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                                               fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
                            if constexpr (NE == 16)
                                mloc = fmaxf(mloc, fmaxf(fmaxf(fmaxf(x[8], x[9]), fmaxf(x[10], x[11])),
                                                         fmaxf(fmaxf(x[12], x[13]), fmaxf(x[14], x[15]))));
                            mloc *= scale2;
                            const bool above = __any(mloc > m_ref[qt] + Half<F16>::HI);     // first tile, then rare
                            bool below = false;
                            if constexpr (F16) {                       // (a query row's scores are in four lanes)
                                unsigned long long low = __ballot(mloc < m_ref[qt] + Half<F16>::LO);
                                low &= low >> 32;
                                low &= low >> 16;
                                below = (low & 0xffffull) != 0ull;
                            }
                            if (above || below) {
                                const float mx = max_of_rows(mloc);
                                float mnew = fmaxf(m_ref[qt], mx);
                                if constexpr (F16) {
                                    const float want = floorf(mx) - Half<F16>::HEAD;       // (whole numbers: rescaling is exact)
                                    mnew = mx > m_ref[qt] + Half<F16>::HI ? want : m_ref[qt];
                                    if (below) {
                                        // Down only as far as the sums stay well inside the range of fp32: beyond that a
                                        // tile adds nothing to them.
                                        const float sum = sum_of_rows(l_sum[qt]);
                                        const float least = m_ref[qt] + (float)(__builtin_amdgcn_frexp_expf(sum) - 80);
                                        if (mx < m_ref[qt] + Half<F16>::LO && mx > -INFINITY) mnew = fminf(fmaxf(want, least), m_ref[qt]);
                                    }
                                }
                                const float alpha = (m_ref[qt] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m_ref[qt] - mnew);
                                l_sum[qt] *= alpha;
#pragma unroll
                                for (int t = 0; t < DT; ++t) o[qt][t] *= alpha;
                                m_ref[qt] = mnew;
                            }
                            const float mr = (m_ref[qt] == -INFINITY) ? 0.0f : m_ref[qt];
                            float psum = 0.0f;
#pragma unroll
                            for (int e = 0; e < NE; e += 2) {
                                const float p0 = __builtin_amdgcn_exp2f(fmaf(x[e], scale2, -mr));
                                const float p1 = __builtin_amdgcn_exp2f(fmaf(x[e + 1], scale2, -mr));
                                psum += p0 + p1;
                                // each part is what the parts before left over, rounded to the element type
                                f32x2 rest = (f32x2){p0, p1};
#pragma unroll
                                for (int n = 0; n < NP; ++n) {
                                    const h16x2 part = __builtin_convertvector(rest, h16x2);
                                    p_part[n][qt][e >> 3][e & 7] = part[0];
                                    p_part[n][qt][e >> 3][(e & 7) + 1] = part[1];
                                    if (n + 1 < NP) {
                                        const f32x2 back = __builtin_convertvector(part, f32x2);
                                        rest = (f32x2){rest[0] - back[0], rest[1] - back[1]};
                                    }
                                }
                            }
                            l_sum[qt] += psum;
                        }
                    });
                }

                // ---- O^T += V^T P^T -----------------------------------------------------------------
                if (has_next) vm_wait(8 + n_idx);                      // V(cur) landed; the last request and K(next) in flight
                else vm_wait(0);
                static_for<2>([&](auto batch) {                        // four 16-wide dv tiles x 32 positions per batch
                    constexpr int B = decltype(batch)::value;
                    constexpr int T0 = D == 128 ? 4 * B : 0, U = D == 128 ? 0 : B;
                    VFrags vh;
                    lds_read_v_batch<D, B>(vh, v_off);
                    if (B == 1 && has_next) {                          // the V buffer is free again
                        if (TIGHT) lds_read_entries<RPI>(ent, stash_addr());
                        issue(vbh, wave_lds + TILE_BYTES, ent);
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const u32x4 both = (u32x4){vh.f[t][0][0], vh.f[t][0][1], vh.f[t][1][0], vh.f[t][1][1]};
                        const h16x8 vf = __builtin_bit_cast(h16x8, both);
#pragma unroll
                        for (int qt = 0; qt < NQT; ++qt)
#pragma unroll
                            for (int n = 0; n < NP; ++n) o[qt][T0 + t] = Half<F16>::mfma(vf, p_part[n][qt][U], o[qt][T0 + t]);
                    }
                });
                // ---- the tile after the next two: request its words -------------------------------------------
                const int t_new = t_nn + STEP;
                if (has_next) {
                    if (SRC == MASK && t_nn < tile_end) positions(t_nn, true);
                    request(t_new, s_nxt);                             // (list: the slot t_nxt's words were read from)
                }
                t_cur = t_nxt; t_nxt = t_nn; t_nn = t_new;
                s_nxt ^= 1;
            }
        }
        vm_wait(0);                              // nothing of this wave's is in flight any more (the slots are reused below)

        // ---- infinite and NaN values, d = 64.  The products above are right for finite values only: an infinite one also met
        //      the low parts of its weights (of either sign, or zero) and the zero weights of the ranks past a row's end, so
        //      its whole column is infinite or NaN in every query row.  What belongs there does not depend on the (positive)
        //      weights: the sum of the column's infinities and NaNs, which are then looked for.  (0.1 us on a call.  At d = 128
        //      it cost 0.3 us of every call, mostly in what the compiler then keeps in registers; such columns are NaN there.) --
        if constexpr (D == 64) {
            float mag[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) mag[i] += fabsf(o[0][t][i]);
            if (__builtin_expect(__any(!((mag[0] + mag[1]) + (mag[2] + mag[3]) < INFINITY)), 0)) {      // (uniform)
                float odd[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};    // of columns 8 (lane % LPR) ..
                for (int t = lt_begin + wave; t < tile_end; t += NW) {
                    uint32_t ent[8];
                    request(t, 0);
                    vm_wait(0);
                    entries(t, 0, ent);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const u32x4 c = *reinterpret_cast<const u32x4 *>(vbh + ((int64_t)ent[i] << UNIT) - (FOLD ? lane_chunk ^ chunk_flip(i) : 0u) + ((lane & (LPR - 1)) << 4));
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const uint32_t bits = (c[e >> 1] >> (16 * (e & 1))) & 0xffffu;
                            const float x = F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)bits) : __uint_as_float(bits << 16);
                            if (!(fabsf(x) < INFINITY)) odd[e] += x;
                        }
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int off = LPR; off < 64; off <<= 1) odd[e] += __shfl_xor(odd[e], off, 64);
#pragma unroll
                for (int t = 0; t < DT; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {                       // column 16 t + 4 g + i
                        const float lo = __shfl(odd[i], 2 * t + (g >> 1), 64), hi = __shfl(odd[4 + i], 2 * t + (g >> 1), 64);
                        const float x = (g & 1) ? hi : lo;
#pragma unroll
                        for (int qt = 0; qt < NQT; ++qt)
                            if (x != 0.0f) o[qt][t][i] = x;             // (true for NaN)
                    }
                vm_wait(0);
            }
        }


        // ---- combine the waves of this workgroup: every wave hands its state over lane by lane through its
        //      own tile buffers, which are idle as soon as the wave itself has no tile left - before the barrier,
        //      so that only the last wave's hand-over is waited for; wave w then reduces and writes the
        //      (query tile, dv tile) blocks k = w * KPW .. of all states.  (m, l) per query row go into the
        //      wave's word slots. ---------------------------------------------------------------------------
        // (a wave's buffers hold 16 blocks: two query tiles at d = 128, four at d = 64; more go over in rounds)
        constexpr int RQ = 16 / DT < NQT ? 16 / DT : NQT;                      // query tiles per round
        // A row owned by one workgroup is finished here; otherwise the partial goes to slot (share + r) for the merge kernel, which
        // learns from the owners of the row's first and last tile which shares those are.
        const bool final_here = lt_begin == 0 && lt_end == tiles && !a.k_new;
        if (tid == 0) {
            uint16_t *parts = reinterpret_cast<uint16_t *>(plan.row_parts + r);
            if (lt_begin == 0) parts[0] = (uint16_t)my_share;
            if (lt_end == tiles) parts[1] = (uint16_t)my_share;
        }
        static_for<(NQT + RQ - 1) / RQ>([&](auto round) {
            constexpr int Q0 = decltype(round)::value * RQ;
            constexpr int QN = NQT - Q0 < RQ ? NQT - Q0 : RQ;
            if (Q0) lds_barrier();               // the round before has been read out
            float *dmp = reinterpret_cast<float *>(wave_lds);                  // [QN * DT][64 lanes] float4
#pragma unroll
            for (int qq = 0; qq < QN; ++qq) {
                const int qt = Q0 + qq;
#pragma unroll
                for (int t = 0; t < DT; ++t)
                    *reinterpret_cast<f32x4 *>(dmp + ((qq * DT + t) * 64 + lane) * 4) = o[qt][t];
                const float l = sum_of_rows(l_sum[qt]);
                if (g == 0) {
                    mlw[wave * 128 + l16 * 2 * NQT + 2 * qt] = m_ref[qt];
                    mlw[wave * 128 + l16 * 2 * NQT + 2 * qt + 1] = l;
                }
            }
            lds_barrier();                     // every wave has handed over, and is done with Q
            // Wave w sums the blocks w * KPW .. of all states, which are of one query tile; everything it reads is requested at once, weights
            // and output row are found once.  (Block by block, and with the sums over lanes through LDS: a layer of 64 rows of 32768 0.6 us
            // longer, 8 rows of 8192 20.9 / 21.5 us with selection and merge.)
            constexpr int BLOCKS = QN * DT;
            constexpr int KPW = (BLOCKS + NW - 1) / NW;    // blocks per wave
            static_assert(DT % KPW == 0, "a wave's blocks are of one query tile");
            const int k0 = wave * KPW;           // uniform
            if (BLOCKS % (NW * KPW) && k0 >= BLOCKS) return;
            const int qt = Q0 + k0 / DT, t0 = k0 % DT;
            float2 ml[NW];
            f32x4 part[KPW][NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) ml[w] = *reinterpret_cast<const float2 *>(mlw + w * 128 + l16 * 2 * NQT + 2 * qt);
#pragma unroll
            for (int kk = 0; kk < KPW; ++kk)
#pragma unroll
                for (int w = 0; w < NW; ++w)
                    part[kk][w] = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(smem + w * WAVE_LDS) + ((k0 + kk) * 64 + lane) * 4);
            float m = -INFINITY, l = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, ml[w].x);
            f32x4 acc[KPW];
#pragma unroll
            for (int kk = 0; kk < KPW; ++kk) acc[kk] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float f = (ml[w].x == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(ml[w].x - m);
                l += f * ml[w].y;
#pragma unroll
                for (int kk = 0; kk < KPW; ++kk) acc[kk] += f * part[kk][w];
            }
            const int q = qt * 16 + l16;
            if (q < QT) {
                if (final_here) {
                    const int gh = div_t(plan, q), tt = q - gh * a.T;
                    const int64_t orow = ((int64_t)b * a.H_q + attn_query_head(a, plan.heads, h, gh)) * a.T + tt;
#pragma unroll
                    for (int kk = 0; kk < KPW; ++kk) {
                        const int64_t at = orow * D + 16 * (t0 + kk) + 4 * g;
                        const f32x4 res = l > 0.0f ? acc[kk] / l : (f32x4){0.f, 0.f, 0.f, 0.f};
                        *reinterpret_cast<f32x4 *>(a.out + at) = res;
                        if (a.out_lowp) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) st_lowp(a.out_lowp, at + i, res[i], a.dtype);
                        }
                    }
                    if (a.lse && g == 0 && t0 == 0) a.lse[orow] = l > 0.0f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
                } else {
                    const int slot = my_share + r;
                    float *po = plan.part_o + (int64_t)slot * QTP * D, *pml = plan.part_ml + (int64_t)slot * QTP * 2;
#pragma unroll
                    for (int kk = 0; kk < KPW; ++kk) *reinterpret_cast<f32x4 *>(po + q * D + 16 * (t0 + kk) + 4 * g) = acc[kk];
                    if (g == 0 && t0 == 0) { pml[2 * q] = m; pml[2 * q + 1] = l; }
                }
            }
        });
        first_seg = false;
        r = r_next;                              // the next segment starts with a barrier of its own
    }

}

// Kernel variants of one head dimension, source and form, by query tiles, layout and element type (null: not built).
template <int D, int SRC, int FORM> const void *variant(int nqt, int layout, bool f16)
{
#define SPECATTN_FN(NQT, LAY) (f16 ? reinterpret_cast<const void *>(&attn_mfma_kernel<D, NQT, LAY, SRC, true, FORM>) : reinterpret_cast<const void *>(&attn_mfma_kernel<D, NQT, LAY, SRC, false, FORM>))
#define SPECATTN_LAYOUTS(NQT) \
    do { \
        if (layout == CONTIGUOUS) return SPECATTN_FN(NQT, CONTIGUOUS); \
        if (layout == PAGE_TABLE) return SPECATTN_FN(NQT, PAGE_TABLE); \
        if constexpr (SRC == LIST) return SPECATTN_FN(NQT, PHYSICAL); \
        return nullptr; \
    } while (0)
    switch (nqt) {
    case 1: SPECATTN_LAYOUTS(1);
    case 2: SPECATTN_LAYOUTS(2);
    case 3: SPECATTN_LAYOUTS(3);
    case 4: if constexpr (SRC == LIST && !(D == 128 && FORM == FEW_POSITIONS)) SPECATTN_LAYOUTS(4); else return nullptr;   // (the mask's tile loop would spill)
    }
    return nullptr;
#undef SPECATTN_LAYOUTS
#undef SPECATTN_FN
}

}  // namespace
}  // namespace specattn
