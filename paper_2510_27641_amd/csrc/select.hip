// Sorting-free exact top-p selection (Section 3.4, Algorithm 2; objective Appendix A, Eq. 8).
//
// Algorithm 2 bisects the threshold in value space and evaluates the kept mass once per step.
// The kernels here reach the exact threshold tau* = max{t : mass{a >= t} >= p * sum a} with radix passes over the
// fp32 bit pattern instead (non-negative floats order like their bits).
// All entries of one bin share their exponent, so a bin's mass is kept as an exact integer sum
// of significands next to the count in one 64-bit LDS counter; bin masses are therefore
// independent of summation order and the result is deterministic.  fp64 appears only in the
// suffix sums over bins.  The kept positions are then written in ascending order (no dense mask, no CSR conversion as in
// Section 3.5).
//
// Rows of up to 65536 entries: one workgroup per row, which holds it in registers for all passes (one HBM read;
// select_resident.h).  Few long rows: split over many workgroups.  Many long rows: one workgroup streams the row in every pass.
// The latter two take pass 1: 2048 bins on bits[30:20], pass 2: 1024 bins on bits[19:10] inside the boundary bin,
// pass 3: 1024 bins on bits[9:0].
#include "common.h"

namespace specattn {
namespace {

constexpr int NB1 = 2048;                     // bins of pass 1
constexpr int NB2 = 1024;                     // bins of passes 2 and 3
constexpr int CNT_SHIFT = 44;                 // counter = count << 44 | sum of significands
constexpr unsigned long long CNT_ONE = 1ull << CNT_SHIFT;
constexpr unsigned long long SIG_MASK = CNT_ONE - 1;

typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load from any float's address

// Histograms in LDS leave a counter free after every NB / 64 bins: the rows of bins that the lanes of the locating wave
// add up then start two banks apart, and neighbouring bins, which are the busy ones, still lie in neighbouring banks.
template <int NB> __device__ __forceinline__ uint32_t hist_slot(uint32_t bin) { return bin + bin / (NB / 64); }
constexpr int HIST1 = NB1 + 64, HIST2 = NB2 + 64;

struct Located {                 // outcome of one locate step
    double target, m_above;
    unsigned long long packed;
    unsigned c_above;
    int bin;
};

// What an entry adds to its bin's counter: one to the count, and its 23 significand bits with bit 23 set.  For
// normal numbers that is the significand; subnormal ones (exponent field 0) have no hidden bit, which mass_of
// takes back out for the bins they fall into - cheaper than a compare and a select for every entry.
__device__ __forceinline__ unsigned long long packed_entry(uint32_t u)
{
    return CNT_ONE | ((u & 0x7fffffu) | 0x800000u);
}

// value of a bin whose entries all carry biased exponent field e: (significand sum) * 2^(max(e,1)-150),
// exact (the sum is below 2^44 and the scale is a power of two well inside the fp64 range)
__device__ __forceinline__ double mass_of(unsigned long long packed, int e_field)
{
    long long sig = (long long)(packed & SIG_MASK);
    if (e_field == 0) sig -= (long long)(packed >> CNT_SHIFT) << 23;       // subnormal entries: no hidden bit
    const double s = (double)sig;
    const int e = (e_field > 0 ? e_field : 1) - 150;
    return s * __hiloint2double((1023 + e) << 20, 0);
}

// Cross-lane moves on the vector ALU (no LDS traffic): lanes without a source lane receive 0.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ int dpp_int(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK> __device__ __forceinline__ double dpp_double(double v)
{
    return __hiloint2double(dpp_int<CTRL, ROW_MASK>(__double2hiint(v)), dpp_int<CTRL, ROW_MASK>(__double2loint(v)));
}
// Inclusive prefix sums over the 64 lanes of a wave: shifts by 1, 2, 4, 8 inside each row of 16 lanes, then
// lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ void wave_prefix(double &m, unsigned &c)
{
#define SPECATTN_SCAN_STEP(CTRL, RM) \
    do { m += dpp_double<CTRL, RM>(m); c += (unsigned)dpp_int<CTRL, RM>((int)c); } while (0)
    SPECATTN_SCAN_STEP(0x111, 0xf);    // row_shr:1
    SPECATTN_SCAN_STEP(0x112, 0xf);    // row_shr:2
    SPECATTN_SCAN_STEP(0x114, 0xf);    // row_shr:4
    SPECATTN_SCAN_STEP(0x118, 0xf);    // row_shr:8
    SPECATTN_SCAN_STEP(0x142, 0xa);    // row_bcast:15 into rows 1 and 3
    SPECATTN_SCAN_STEP(0x143, 0xc);    // row_bcast:31 into rows 2 and 3
#undef SPECATTN_SCAN_STEP
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Kept-position mask: every lane holds the keep flags of four consecutive positions (bit c = position 4 * lane + c
// of a run of 256); the eight lanes that share a 32-position word combine their nibbles on the vector ALU
// (neighbour, pair and half-row exchanges), after which each of them holds the whole word.
__device__ __forceinline__ uint32_t mask_word(uint32_t nibble, int lane)
{
    int v = (int)(nibble << (4 * (lane & 7)));
    v |= __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);     // quad_perm [1,0,3,2]
    v |= __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);     // quad_perm [2,3,0,1]
    v |= __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);    // row_half_mirror: lane i <-> 7 - i of its eight
    return (uint32_t)v;
}

// One radix pass decision.  `hist` holds the packed counters of this pass (bin b at hist_slot<NB>(b)).
// On return (uniform over the block): bin = highest non-empty bin b with
// m_above + mass(bins >= b) >= target (lowest non-empty bin if rounding leaves none; -1 without any mass),
// and m_above / c_above advanced to cover the bins above it.
// With top_p = 1 the boundary is the lowest non-empty bin, whatever the rounding of the sums above it.  Bins count as empty
// there from the octave down from which on the entries all together add less than one unit in the last place of the row's
// total: fp64 sums taken in another order differ by as much.
// Used by the streaming kernel and the split selection; rows in registers have bins and decisions of their own.
// The first wave does it alone and the others wait at the one barrier: its lanes own NB / 64 bins each from the top down (lane
// 0 the highest), add them up as integers (bins of one exponent add exactly), and a prefix over the lanes tells every lane the
// mass above its bins; the bins of the lane that holds the boundary are then searched one per lane.  (All waves together, with
// the totals of the waves through LDS and two barriers, took 2.1 us per step of 2048 bins.)
// Beside few registers (the streaming kernel) the bins are read an exponent's at a time, else (TOGETHER) all at once.
template <int NB, bool FIRST, bool TOGETHER = false>
__device__ __forceinline__ int locate_bin(const unsigned long long *hist, Located &found, int e_field_fixed, float top_p, double &target,
                                          double &m_above, unsigned &c_above, unsigned long long &bin_packed)
{
    constexpr int BPL = NB / 64;
    constexpr int RUN = FIRST ? 8 : BPL;                       // bins of one exponent
    constexpr int RUNS = BPL / RUN;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const unsigned long long *mine = hist + (63 - lane) * (BPL + 1);       // this lane's lowest bin
        unsigned long long sum[RUNS];
#pragma unroll
        for (int g = 0; g < RUNS; ++g) {
            sum[g] = 0ull;
            if constexpr (TOGETHER) continue;
#pragma unroll
            for (int j = 0; j < RUN; ++j) sum[g] += mine[g * RUN + j];
            __builtin_amdgcn_sched_barrier(0);                 // (not all loads at once: 1100 streamed rows of 66000 271.3 / 269.4 us)
        }
        if constexpr (TOGETHER) {
            unsigned long long v[BPL];
#pragma unroll
            for (int j = 0; j < BPL; ++j) v[j] = mine[j];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < BPL; ++j) sum[j / RUN] += v[j];
        }
        auto exponent = [&](int g) { return FIRST ? (63 - lane) * RUNS + g : e_field_fixed; };
        int cut = -1;                                          // exponent fields up to this one count as empty
        double lm, incl_m;
        unsigned lc, incl_c;
        auto add_up = [&]() {
            lm = 0.0;
            lc = 0;
#pragma unroll
            for (int g = 0; g < RUNS; ++g)
                if (exponent(g) > cut) { lm += mass_of(sum[g], exponent(g)); lc += (unsigned)(sum[g] >> CNT_SHIFT); }
            incl_m = lm;
            incl_c = lc;
            wave_prefix(incl_m, incl_c);
        };
        add_up();
        const double total = read_lane(incl_m, 63);
        if (FIRST && !(top_p < 1.0f) && total > 0.0) {
            // sums from the bottom up: the lanes in reverse order, then each lane's octaves
            double tail = __shfl(lm, 63 - lane, 64);
            unsigned none = 0;
            wave_prefix(tail, none);
            tail = __shfl(dpp_double<0x138, 0xf>(tail), 63 - lane, 64);
            const double ulp = __hiloint2double((((__double2hiint(total) >> 20) & 0x7ff) - 52) << 20, 0);
            int fields = 0;
#pragma unroll
            for (int g = 0; g < RUNS; ++g) {
                tail += mass_of(sum[g], exponent(g));
                fields += __popcll(__ballot(tail < ulp));
            }
            cut = fields - 1;
            add_up();
        }
        // mass and count of the lanes before this one (wave_shr:1)
        const double before = dpp_double<0x138, 0xf>(incl_m);
        const unsigned before_c = (unsigned)dpp_int<0x138, 0xf>((int)incl_c);
        Located out = {FIRST ? (double)top_p * total : target, m_above, 0ull, c_above, -1};    // Algorithm 2: M_target = p * sum a
        const double goal = top_p < 1.0f ? out.target : INFINITY;
        if (!FIRST || total > 0.0) {
            // Masses are non-negative, so the running sum never decreases: the first lane whose sum reaches the target holds
            // the boundary.  (If rounding leaves none, the row total itself fell short by an ulp: the lowest entries do.)
            const unsigned long long some = __ballot(lc > 0), holds = __ballot(lc > 0 && m_above + (before + lm) >= goal);
            const int at = holds ? (int)__ffsll((long long)holds) - 1 : 63 - __clzll((long long)some);
            const double above = read_lane(before, at);
            const unsigned above_c = (unsigned)__builtin_amdgcn_readlane((int)before_c, at);
            const int low = (63 - at) * BPL;                   // the boundary lane's lowest bin
            const int bin = low + BPL - 1 - lane;              // lane 0 looks at its highest
            const int e_bin = FIRST ? bin >> 3 : e_field_fixed;
            const unsigned long long hj = lane < BPL && (!FIRST || e_bin > cut) ? hist[hist_slot<NB>(low) + BPL - 1 - lane] : 0ull;
            const unsigned cj = (unsigned)(hj >> CNT_SHIFT);
            double run = cj ? mass_of(hj, e_bin) : 0.0;
            unsigned runc = cj;
            wave_prefix(run, runc);
            const unsigned long long filled = __ballot(cj > 0), ok = __ballot(cj > 0 && m_above + (above + run) >= goal);
            const int pick = ok ? (int)__ffsll((long long)ok) - 1 : 63 - __clzll((long long)filled);
            const double inside = pick ? read_lane(run, pick - 1) : 0.0;
            const unsigned inside_c = pick ? (unsigned)__builtin_amdgcn_readlane((int)runc, pick - 1) : 0u;
            out.m_above = m_above + (above + inside);
            out.c_above = c_above + above_c + inside_c;
            out.packed = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(hj >> 32), pick) << 32 |
                         (unsigned)__builtin_amdgcn_readlane((int)(uint32_t)hj, pick);
            out.bin = low + BPL - 1 - pick;
        }
        if (lane == 0) found = out;
    }
    __syncthreads();
    target = found.target;
    m_above = found.m_above;
    c_above = found.c_above;
    bin_packed = found.packed;
    return found.bin;
}

template <int THREADS, int N>
__device__ __forceinline__ void clear_hist(unsigned long long *hist)
{
#pragma unroll
    for (int b = 0; b < N; b += THREADS)
        if (b + (int)threadIdx.x < N) hist[b + threadIdx.x] = 0ull;
}

// The mass of chunk c of a row of `len` positions (Section 4: chunk-granular selection; the score of a chunk is its mass):
// its entries added up in fp64 in ascending position order, rounded once to fp32; NaN if one of them is invalid.
// Bound by the reads' latency: a thread has its chunk to itself, and its four requests bring half a cache line.  (A test of every entry by
// itself, with the requests in whatever order / the largest entry, requests in order, us: 32 x 2044 / 16 5.8 / 5.6, 300 x 30000 / 256 23.5 /
// 17.3, 300 x 60000 / 512 41.7 / 29.3, 1100 x 32768 / 16 31.0 / 29.5.  Sixteen entries ahead: 300 x 60000 / 512 33.2, and 1100 rows 69 instead of 58 -
// their lines leave the caches before they are used up.)
__device__ __forceinline__ float chunk_mass(const float *row, int len, int c, int chunk_shift)
{
    const int chunk = 1 << chunk_shift;
    const int p0 = c << chunk_shift;
    int p1 = p0 + chunk;
    p1 = p1 > len ? len : p1;
    double sum = 0.0;
    bool bad = false;
    if (p1 == p0 + chunk && chunk >= 4) {
        // As an unsigned number a sign bit or an exponent of all ones makes an entry too large: then the chunk is looked at again (-0.0 is
        // zero).
        uint32_t top = 0u;
        auto add = [&](u32x4a v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                top = v[e] > top ? v[e] : top;
                sum += (double)__uint_as_float(v[e]);
            }
        };
        if (chunk >= 16) {
            for (int p = p0; p < p1; p += 16) {                // four requests, in order, then their entries
                u32x4a v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[k] = *reinterpret_cast<const u32x4a *>(row + p + 4 * k);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) add(v[k]);
            }
        } else {
            for (int p = p0; p < p1; p += 4) add(*reinterpret_cast<const u32x4a *>(row + p));
        }
        bad = top >= 0x7f800000u;
    }
    if (bad || p1 != p0 + chunk || chunk < 4) {
        sum = 0.0;
        bad = false;
        for (int p = p0; p < p1; ++p) {
            const uint32_t u = __float_as_uint(row[p]);
            bad = bad || (u >= 0x7f800000u && u != 0x80000000u);                   // negative, infinite or NaN
            sum += (double)row[p];
        }
    }
    return bad ? __uint_as_float(0x7fc00000u) : (float)sum;
}

#include "select_resident.h"

// Rows too long for the registers: one workgroup per row, which streams it in every pass.
constexpr int STREAM_THREADS = 1024, STREAM_WAVES = STREAM_THREADS / 64, STREAM_ITEM = STREAM_THREADS * 4;
__global__ __launch_bounds__(STREAM_THREADS, 4) void topp_select_stream_kernel(SelectLaunch a)
{
    __shared__ Located found;
    __shared__ unsigned wave_tot[2][STREAM_WAVES];
    __shared__ unsigned running;
    __shared__ unsigned long long hist1[HIST1 + HIST2];
    unsigned long long *hist2 = hist1 + HIST1;
    const int r = blockIdx.x;
    const int b = r / a.H_kv, h = r - b * a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int len = a.seq_lens ? a.seq_lens[b] : a.n_tokens;
    len = len < 0 ? 0 : (len > a.n_tokens ? a.n_tokens : len);
    len = (len + (1 << a.chunk_shift) - 1) >> a.chunk_shift;     // rows of chunk masses: length in chunks
    len = len > a.n_max ? a.n_max : len;
    const float *row = a.probs + (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    const int n_items = (len + STREAM_ITEM - 1) / STREAM_ITEM;

    // -0.0 is zero; negative, infinite and NaN entries make the row invalid.  Branch-free: the largest bit pattern
    // seen is tested once per thread, and an invalid entry is clamped to the largest finite value so that its bin
    // stays inside the histogram (the row's result is discarded anyway).
    uint32_t worst = 0u;
    auto clean = [&](uint32_t x) -> uint32_t {
        x = (x == 0x80000000u) ? 0u : x;
        worst = worst > x ? worst : x;
        return x < 0x7f7fffffu ? x : 0x7f7fffffu;
    };
    auto clean4 = [&](uint4 u) -> uint4 { return make_uint4(clean(u.x), clean(u.y), clean(u.z), clean(u.w)); };
    // Slow form of an item's load (rows of fewer than four entries).
    auto load_item = [&](int i) -> uint4 {
        const int p = (i * STREAM_THREADS + tid) * 4;
        uint4 u = make_uint4(0, 0, 0, 0);
        if (p < len) u.x = __float_as_uint(row[p]);
        if (p + 1 < len) u.y = __float_as_uint(row[p + 1]);
        if (p + 2 < len) u.z = __float_as_uint(row[p + 2]);
        if (p + 3 < len) u.w = __float_as_uint(row[p + 3]);
        return clean4(u);
    };
    // Fast form: plain 16-byte loads from any float's address.  An item that reaches past the row's end loads the row's last
    // whole vector instead (in bounds) and is masked afterwards; the at most three entries behind it are fetched once.
    const bool vec_ok = len >= 4;                              // uniform
    const int last4 = (len - 4) & ~3;                          // start of the row's last whole vector
    const int tail_p = (len & 3) ? (len & ~3) : -1;            // start of the partial vector, if any
    uint4 tailv = make_uint4(0, 0, 0, 0);
    if (vec_ok && tail_p >= 0 && tid == (tail_p % STREAM_ITEM) / 4) {
        tailv.x = __float_as_uint(row[tail_p]);
        if (tail_p + 1 < len) tailv.y = __float_as_uint(row[tail_p + 1]);
        if (tail_p + 2 < len) tailv.z = __float_as_uint(row[tail_p + 2]);
    }
    auto raw_load = [&](int i) -> uint4 {
        const int p = (i * STREAM_THREADS + tid) * 4;
        const u32x4a v = __builtin_nontemporal_load(reinterpret_cast<const u32x4a *>(row + (p < last4 ? p : last4)));
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    auto finish_item = [&](int i, uint4 u) -> uint4 {
        const int p = (i * STREAM_THREADS + tid) * 4;
        if (p + 3 >= len) u = (p == tail_p) ? tailv : make_uint4(0, 0, 0, 0);
        return clean4(u);
    };
    clear_hist<STREAM_THREADS, HIST1 + HIST2>(hist1);
    __syncthreads();
    auto for_items = [&](auto &&fn) {
        for (int i0 = 0; i0 < n_items; i0 += 4) {              // four loads in flight per thread
            uint4 u[4];
            if (vec_ok) {
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = raw_load(i0 + k);
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = finish_item(i0 + k, u[k]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) u[k] = (i0 + k < n_items) ? load_item(i0 + k) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i0 + k < n_items) fn(i0 + k, u[k]);
        }
    };

    // ---- pass 1: bits[30:20] -----------------------------------------------------------------
    for_items([&](int, uint4 u) {
        if (u.x) atomicAdd(&hist1[hist_slot<NB1>(u.x >> 20)], packed_entry(u.x));
        if (u.y) atomicAdd(&hist1[hist_slot<NB1>(u.y >> 20)], packed_entry(u.y));
        if (u.z) atomicAdd(&hist1[hist_slot<NB1>(u.z >> 20)], packed_entry(u.z));
        if (u.w) atomicAdd(&hist1[hist_slot<NB1>(u.w >> 20)], packed_entry(u.w));
    });
    const bool any_bad = __syncthreads_or(worst >= 0x7f800000u ? 1 : 0) != 0;     // also orders the atomics

    double target = 0.0, m_above = 0.0;
    unsigned c_above = 0;
    unsigned long long bin_packed = 0;
    const int b1 = locate_bin<NB1, true>(hist1, found, 0, a.top_p, target, m_above, c_above, bin_packed);
    const double row_sum = (double)target / (double)a.top_p;     // only used for the boundary flag
    if (any_bad || b1 < 0 || len == 0) {
        if (tid == 0) {
            a.counts[r] = 0;
            if (a.thresholds) a.thresholds[r] = 0.0f;
            if (a.row_flags) a.row_flags[r] = SPECATTN_ROW_INVALID;
        }
        if (a.block_counts)
            for (int k = tid; k < a.blocks_per_row; k += STREAM_THREADS) a.block_counts[(int64_t)r * a.blocks_per_row + k] = 0;
        if (a.kept_mask)
            for (int k = tid; k < a.blocks_per_row * (SEL_BLOCK / 32); k += STREAM_THREADS)
                a.kept_mask[(int64_t)r * a.blocks_per_row * (SEL_BLOCK / 32) + k] = 0u;
        return;
    }
    const int e_field = b1 >> 3;

    // A boundary bin that holds a single entry pins tau*: the bin's significand sum is that entry's
    // significand, and the exponent is the bin's.  Otherwise refine inside the bin.
    auto single_entry_bits = [&](unsigned long long packed) -> uint32_t {
        return ((uint32_t)e_field << 23) | ((uint32_t)packed & 0x7fffffu);
    };
    uint32_t tau_bits;
    if ((bin_packed >> CNT_SHIFT) == 1) {
        tau_bits = single_entry_bits(bin_packed);
    } else {
        // ---- pass 2: bits[19:10] inside bin b1 -----------------------------------------------
        // (as a range of bit patterns that leaves zeros out; the first pass's counters are cleared for the third on the way)
        auto refine = [&](uint32_t first, uint32_t width, auto &&count) {
            const uint32_t lo = first ? first : 1u, n = first ? width : width - 1u;
            for_items([&](int, uint4 u) {
                if (u.x - lo < n) count(u.x);
                if (u.y - lo < n) count(u.y);
                if (u.z - lo < n) count(u.z);
                if (u.w - lo < n) count(u.w);
            });
            __syncthreads();
        };
        clear_hist<STREAM_THREADS, HIST2>(hist1);
        refine((uint32_t)b1 << 20, 1u << 20, [&](uint32_t x) { atomicAdd(&hist2[hist_slot<NB2>((x >> 10) & 1023u)], packed_entry(x)); });
        const int b2 = locate_bin<NB2, false>(hist2, found, e_field, a.top_p, target, m_above, c_above, bin_packed);
        const uint32_t prefix = ((uint32_t)b1 << 10) | (uint32_t)b2;
        if ((bin_packed >> CNT_SHIFT) == 1) {
            tau_bits = single_entry_bits(bin_packed);
        } else {
            // ---- pass 3: bits[9:0] inside (b1, b2) -------------------------------------------
            refine(prefix << 10, 1u << 10, [&](uint32_t x) { atomicAdd(&hist1[hist_slot<NB2>(x & 1023u)], packed_entry(x)); });
            const int b3 = locate_bin<NB2, false>(hist1, found, e_field, a.top_p, target, m_above, c_above, bin_packed);
            tau_bits = (prefix << 10) | (uint32_t)b3;             // >= 1: zeros never enter a bin
        }
    }
    const unsigned kept = c_above + (unsigned)(bin_packed >> CNT_SHIFT);

    if (tid == 0) {
        a.counts[r] = (int32_t)kept;
        if (a.thresholds) a.thresholds[r] = __uint_as_float(tau_bits);
        if (a.row_flags) {
            const double m_excl = m_above, m_incl = m_above + mass_of(bin_packed, e_field);
            const double band = 1e-6 * row_sum;
            uint32_t f = 0;
            if (fabs(m_incl - target) <= band || fabs(m_excl - target) <= band) f |= SPECATTN_ROW_NEAR_BOUNDARY;
            if (a.indices && kept > (unsigned)a.idx_capacity) f |= SPECATTN_ROW_OVERFLOW;
            a.row_flags[r] = f;
        }
        running = 0;
    }
    if (!a.indices && !a.block_counts && !a.kept_mask) return;
    uint32_t *mask_out = a.kept_mask ? a.kept_mask + (int64_t)r * a.blocks_per_row * (SEL_BLOCK / 32) : nullptr;
    const int mask_words = a.blocks_per_row * (SEL_BLOCK / 32);
    // word (i * STREAM_THREADS + tid) / 8 of the mask covers this thread's four positions of item i; the lane that
    // holds the word's first nibble stores it
    auto emit_mask = [&](int i, uint32_t nibble) {
        const uint32_t word = mask_word(nibble, lane);
        const int w = (i * STREAM_THREADS + tid) >> 3;
        if ((lane & 7) == 0 && w < mask_words) mask_out[w] = word;
    };

    // ---- ordered compaction: {j : a_j >= tau*}, ascending (Algorithm 2, last step) -------------
    int32_t *out = a.indices ? a.indices + (int64_t)r * a.idx_stride : nullptr;
    const int32_t *ptab = (a.emit_physical && a.page_table) ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    __syncthreads();
    int it = 0;
    auto compact_item = [&](int i, uint4 u) {
        const bool f0 = u.x >= tau_bits, f1 = u.y >= tau_bits, f2 = u.z >= tau_bits, f3 = u.w >= tau_bits;
        const unsigned long long m0 = __ballot(f0), m1 = __ballot(f1), m2 = __ballot(f2), m3 = __ballot(f3);
        const unsigned before = __popcll(m0 & lt_mask) + __popcll(m1 & lt_mask) + __popcll(m2 & lt_mask) +
                                __popcll(m3 & lt_mask);
        const unsigned wtot = __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
        if (mask_out) emit_mask(i, (f0 ? 1u : 0u) | (f1 ? 2u : 0u) | (f2 ? 4u : 0u) | (f3 ? 8u : 0u));
        const int buf = it & 1;
        if (lane == 0) wave_tot[buf][wave] = wtot;
        __syncthreads();
        unsigned base = running, all = 0;
#pragma unroll
        for (int w = 0; w < STREAM_WAVES; ++w) {
            const unsigned t = wave_tot[buf][w];
            if (w < wave) base += t;
            all += t;
        }
        if (a.block_counts) {
            constexpr int BPI = STREAM_ITEM / SEL_BLOCK;              // selection blocks per item
            constexpr int WPB = STREAM_WAVES / BPI;                      // waves per block
            if (tid < BPI) {
                unsigned c = 0;
                for (int w = 0; w < WPB; ++w) c += wave_tot[buf][tid * WPB + w];
                const int blk = i * BPI + tid;
                if (blk < a.blocks_per_row) a.block_counts[(int64_t)r * a.blocks_per_row + blk] = (int32_t)c;
            }
        }
        if (out) {
            unsigned o = base + before;
            const int p = (i * STREAM_THREADS + tid) * 4;
            auto emit = [&](bool f, int pos) {
                if (f) {
                    if (o < (unsigned)a.idx_capacity) {
                        int32_t val = pos;
                        if (ptab) val = (ptab[pos >> a.page_shift] << a.page_shift) | (pos & ((1 << a.page_shift) - 1));
                        out[o] = val;
                    }
                    ++o;
                }
            };
            emit(f0, p); emit(f1, p + 1); emit(f2, p + 2); emit(f3, p + 3);
        }
        __syncthreads();                                       // everyone has read `running`
        if (tid == 0) running = base + all;                 // wave 0: base == running
        ++it;
    };
    for_items(compact_item);
    if (a.block_counts) {                                      // blocks past the row's end
        constexpr int BPI = STREAM_ITEM / SEL_BLOCK;
        for (int k = n_items * BPI + tid; k < a.blocks_per_row; k += STREAM_THREADS)
            a.block_counts[(int64_t)r * a.blocks_per_row + k] = 0;
    }
    if (mask_out)                                              // words past the last item
        for (int k = n_items * (STREAM_ITEM / 32) + tid; k < mask_words; k += STREAM_THREADS) mask_out[k] = 0u;
}

template <int THREADS, int NV4, bool CHUNKED = false> specattn_status launch_one(const SelectLaunch &asked, hipStream_t stream)
{
    SelectLaunch a = asked;
    a.per_h = FastDivisor(a.H_kv);
    // Rows of different lengths that come in turns: the longest first, so that no long one starts when the others are done.  Not where all
    // workgroups are on the chip at once (16 waves to a CU) nor for more than three turns, over which lengths even out and long rows
    // side by side only wait for the same things, nor for short rows, to which a workgroup's search for its sequence is 0.5 to 1 us more
    // (chunk sums take a quarter of the time of as many entries); and up to 64 sequences, which the lanes of a wave compare.  In the order
    // of the batch / from the longest down, us, sequences x heads of a sixteenth to the whole length: 64 x 8 of 65536 44.9 / 38.8, 48 x 8
    // 42.0 / 32.5, 64 x 12 60.7 / 57.0; 40 x 8 of 40000 29.5 / 26.8; 64 x 13 of 32768 35.1 / 32.2, 64 x 24 49.7 / 48.0; 64 x 20 of 14000
    // 24.7 / 23.6; but 64 x 17 of 65536 (4.25 turns) 82.5 / 88.5, 64 x 32 of 40000 (8) 116.6 / 121.3, of 32768 (4) 62.6 / 62.7, 64 x 17 of 8000
    // 15.2 / 16.0, of 1000 7.4 / 8.5.  In chunks of 16: 64 x 32 of 65536 58.8 / 56.5, but 64 x 24 of 33000 28.8 / 31.3.  Rows of nearly
    // one length lose 1 to 5 %.
    const int rows = a.B * a.H_kv, turn = 1024 / THREADS * cu_count();
    if (a.seq_lens && a.B > 1 && a.B <= 64 && rows > turn && rows <= 3 * turn && (CHUNKED ? a.n_tokens / 4 : a.n_max) > 12288) {
        a.by_length = 1;
        while (a.n_tokens >> (a.by_length - 1) > 255) ++a.by_length;
    }
    hipLaunchKernelGGL((topp_select_kernel<THREADS, NV4, CHUNKED>), dim3(a.B * a.H_kv), dim3(THREADS), select_lds(THREADS, NV4), stream, a);
    return check_launch("topp_select_kernel");
}

// ---- few long rows: one row split over many workgroups ------------------------------------------------
// The same radix search with one workgroup per (row, slice), in three launches; kernel boundaries separate them.
//   1. every workgroup leaves the pass-1 histogram of its slice in memory (the bins between the lowest and the highest
//      non-empty one, and those two numbers);
//   2. every workgroup adds the slices of its row up, locates the boundary bin (identical code on identical integers), notes
//      how many of its slice's entries lie above that bin and collects those that lie in it - a few per cent;
//   3. every workgroup finishes the search on the row's collected entries alone, in LDS, knows from the counts where its
//      slice's part of the list begins, and writes it.
// Nothing has to be cleared, no atomic goes to memory, and no pass only counts.  32 rows of 131072: 28 us; three
// histogram passes that added up by atomics in memory, with a launch to clear them, one for the threshold and the mask and
// compaction passes of the union, took 50 us.  Bound by the trips to memory of each launch (ranges, then
// histograms, then entries, about a microsecond each) and the locate steps (2 us each), not by the row's bytes.
// With less workspace than that asks for (a histogram per slice), the slices of a row add theirs up in one histogram of
// the row, by atomics in memory after a launch that clears it (integers: any order gives the same sums), and as many of the
// boundary bin's entries are collected as there is room for: 32 heavy-tailed rows of 131072 in an eighth of the workspace 24.4 us
// (24.1 with all of it, 71 without any), 8 of 65536 20.8 (19.2, 26.7).
// The three kernels' arguments in dependent turns with two divisions, the bins of a locate step eight at a time, a wave's second slice behind its
// first one / arguments in one batch, all bins at once, both slices together, us: 32 rows of 131072 24.5 / 23.8, 8 of them 19.4 / 18.2, 16 of 250001
// 27.8 / 26.6, 32 of 70000 23.8 / 23.0, 8 of 65536 20.9 / 19.9.
constexpr int MW_THREADS = 512;
constexpr int MW_WAVES = MW_THREADS / 64;
constexpr int MW_ITEM = MW_THREADS * 4;           // positions a workgroup loads with one instruction
constexpr int MW_FLIGHT = 4;                      // such loads in flight per thread
constexpr int MW_MOST_SLICES = 32;                // (the lanes of a wave hold the slices' bin ranges)

constexpr int MW_COLLECT_SHIFT = 2;               // a quarter of a slice's entries can be collected (rows so flat that one bin
                                                  // of an eighth of an octave holds more are read again instead)
constexpr int MW_LDS_ENTRIES = 12288;             // ... and per row that step 3 keeps in LDS (two workgroups to a CU)

struct MwState {                     // outcome of the first locate step
    unsigned long long bin_packed;
    double target, m_above;
    unsigned c_above;
    int bin;
    int invalid;                     // a NaN, negative or infinite entry, no mass, or an empty row: nothing else holds then
};
struct MwHead { int lo, hi, bad, pad; };     // non-empty bins of a slice's histogram (lo > hi: none)
struct MwLaunch {
    SelectLaunch a;
    unsigned long long *hist;        // [rows * slices][NB1]; LEAN: [rows][NB1]
    MwHead *head;                    // [rows * slices]; LEAN: [rows], all bins
    uint32_t *entries;               // [rows * slices][collect] a slice's entries in the boundary bin, in any order
    int4 *counts;                    // [rows * slices] a slice's entries above the boundary bin and in it; smallest and largest of the latter
    MwState *state;                  // [rows]
    int slices, slice_len;           // workgroups per row; positions per workgroup (a multiple of MW_ITEM)
    int collect;                     // entries of a slice that can be collected: slice_len >> MW_COLLECT_SHIFT; LEAN: at most
};

// What the three kernels use, in one batch (left to the compiler, the row and slice alone take three dependent turns).
__device__ __forceinline__ void mw_preload(const MwLaunch &w)
{
    SPECATTN_PRELOAD(w.a.probs); SPECATTN_PRELOAD(w.a.stride_b); SPECATTN_PRELOAD(w.a.stride_h); SPECATTN_PRELOAD(w.a.H_kv); SPECATTN_PRELOAD(w.a.n_max);
    SPECATTN_PRELOAD(w.a.seq_lens); SPECATTN_PRELOAD(w.a.top_p); SPECATTN_PRELOAD(w.a.n_tokens); SPECATTN_PRELOAD(w.a.per_h.mul); SPECATTN_PRELOAD(w.a.per_h.shift);
    SPECATTN_PRELOAD(w.hist); SPECATTN_PRELOAD(w.head); SPECATTN_PRELOAD(w.entries); SPECATTN_PRELOAD(w.counts); SPECATTN_PRELOAD(w.state);
    SPECATTN_PRELOAD(w.slices); SPECATTN_PRELOAD(w.slice_len); SPECATTN_PRELOAD(w.collect);
}

__device__ __forceinline__ int mw_row_len(const SelectLaunch &a, int b)
{
    int len = a.seq_lens ? a.seq_lens[b] : a.n_tokens;
    len = len < 0 ? 0 : (len > a.n_tokens ? a.n_tokens : len);
    return len > a.n_max ? a.n_max : len;
}

// A slice's entries, MW_FLIGHT vectors per thread at a time; the first ones are requested on construction.  The loads are
// unconditional, so that nothing between them waits: a vector that reaches past the slice's end is fetched ending there and
// moved into place when it is used.
struct MwSlice {
    const float *row;
    int begin, end, p0;
    u32x4a raw[MW_FLIGHT];
    __device__ __forceinline__ MwSlice(const MwLaunch &w, int b, int h, int sl, int len)
    {
        row = w.a.probs + (int64_t)b * w.a.stride_b + (int64_t)h * w.a.stride_h;
        begin = sl * w.slice_len;
        end = begin + w.slice_len;
        end = end < len ? end : len;
        request(begin);
    }
    __device__ __forceinline__ void request(int at)
    {
        p0 = at;
        if (p0 >= end) return;                                   // (uniform)
        if (end < 4) {
            if (threadIdx.x == 0)
#pragma unroll
                for (int c = 0; c < 4; ++c) raw[0][c] = c < end ? __float_as_uint(row[c]) : 0u;
            return;
        }
#pragma unroll
        for (int i = 0; i < MW_FLIGHT; ++i) {
            const int p = p0 + i * MW_ITEM + (int)threadIdx.x * 4;
            raw[i] = *reinterpret_cast<const u32x4a *>(row + (p < end - 4 ? p : end - 4));
        }
    }
    __device__ __forceinline__ uint4 entries(int i) const
    {
        const int p = p0 + i * MW_ITEM + (int)threadIdx.x * 4;
        const u32x4a v = raw[i];
        const int over = end < 4 ? (p > 0 ? 4 : 0) : p - (end - 4);      // entries of the vector that come before p
        if (over <= 0) return make_uint4(v[0], v[1], v[2], v[3]);
        return make_uint4(over == 1 ? v[1] : over == 2 ? v[2] : over == 3 ? v[3] : 0u, over == 1 ? v[2] : over == 2 ? v[3] : 0u,
                          over == 1 ? v[3] : 0u, 0u);
    }
    template <typename F> __device__ __forceinline__ void each(F &&visit)
    {
        for (int at = begin; at < end; at += MW_FLIGHT * MW_ITEM) {
            if (at != begin) request(at);
#pragma unroll
            for (int i = 0; i < MW_FLIGHT; ++i) {
                const uint4 u = entries(i);
                visit(u.x); visit(u.y); visit(u.z); visit(u.w);
            }
        }
    }
};

// The row's histogram in `hist` from those of its slices; `mine`: lane j holds slice j's range (lanes past the slices
// slice 0's).  cnt[k]: entries that slice `sl` has in this thread's bin k * MW_THREADS + tid.  Returns whether any slice met
// an invalid entry.
__device__ __forceinline__ bool mw_gather(unsigned long long *hist, const MwHead &mine, const unsigned long long *h, int slices, int sl,
                                          int (&cnt)[NB1 / MW_THREADS])
{
    const int tid = threadIdx.x;
    int lo = mine.lo, hi = mine.hi;
    const bool bad = __any(mine.bad != 0);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int l = __shfl_xor(lo, off, 64), g = __shfl_xor(hi, off, 64);
        lo = l < lo ? l : lo;
        hi = g > hi ? g : hi;
    }
#pragma unroll
    for (int k = 0; k < NB1 / MW_THREADS; ++k) {
        const int bin = k * MW_THREADS + tid;
        unsigned long long sum = 0ull;
        cnt[k] = 0;
        if (k * MW_THREADS <= hi && (k + 1) * MW_THREADS > lo) {       // (uniform)
            for (int j0 = 0; j0 < slices; j0 += 16) {
                unsigned long long v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int j = j0 + i < slices ? j0 + i : slices - 1;
                    const int jl = __builtin_amdgcn_readlane(mine.lo, j), jh = __builtin_amdgcn_readlane(mine.hi, j);
                    v[i] = (j0 + i < slices && bin >= jl && bin <= jh) ? h[(size_t)j * NB1 + bin] : 0ull;
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    sum += v[i];
                    if (j0 + i == sl) cnt[k] += (int)(v[i] >> CNT_SHIFT);
                }
            }
        }
        hist[hist_slot<NB1>(bin)] = sum;
    }
    __syncthreads();
    return bad;
}

// Sum of v over the workgroup (every thread returns it).  `slot` is used by this call alone.
__device__ __forceinline__ int mw_sum(int v, int *slot)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_inclusive_sum(v);
    if (lane == 63) slot[wave] = v;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int w = 0; w < MW_WAVES; ++w) s += slot[w];
    return s;
}

// Step 1.
template <bool LEAN> __device__ __forceinline__ void mw_hist(const MwLaunch &w)
{
    __shared__ unsigned long long hist[NB1];
    __shared__ int range[2][MW_WAVES];
    const SelectLaunch &a = w.a;
    mw_preload(w);
    const int r = blockIdx.x, sl = blockIdx.y;
    const int b = a.per_h.divide(r), h = r - b * a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    MwSlice slice(w, b, h, sl, mw_row_len(a, b));
#pragma unroll
    for (int k = 0; k < NB1 / MW_THREADS; ++k) hist[k * MW_THREADS + tid] = 0ull;
    __syncthreads();
    bool bad = false;
    slice.each([&](uint32_t x) {
        if (x == 0x80000000u) x = 0u;                                   // -0.0 is zero
        if (x >= 0x7f800000u) { bad = true; return; }                   // negative, infinite, NaN
        if (x) atomicAdd(&hist[x >> 20], packed_entry(x));
    });
    const bool any_bad = __syncthreads_or(bad ? 1 : 0) != 0;             // also orders the LDS atomics
    if constexpr (LEAN) {
#pragma unroll
        for (int k = 0; k < NB1 / MW_THREADS; ++k) {
            const int bin = k * MW_THREADS + tid;
            const unsigned long long v = hist[bin];
            if (v) atomicAdd(&w.hist[(size_t)r * NB1 + bin], v);
        }
        if (any_bad && tid == 0) w.head[r].bad = 1;
        return;
    }
    // lowest and highest non-empty bin: every wave looks at its 64 bins of each group
    unsigned long long bins[NB1 / MW_THREADS];
    int lo = NB1, hi = -1;
#pragma unroll
    for (int k = 0; k < NB1 / MW_THREADS; ++k) {
        bins[k] = hist[k * MW_THREADS + tid];
        const unsigned long long some = __ballot(bins[k] != 0ull);
        if (some) {
            const int first = k * MW_THREADS + wave * 64;
            if (lo == NB1) lo = first + (int)__ffsll((long long)some) - 1;
            hi = first + 63 - __clzll((long long)some);
        }
    }
    if (lane == 0) { range[0][wave] = lo; range[1][wave] = hi; }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < MW_WAVES; ++k) {
        lo = range[0][k] < lo ? range[0][k] : lo;
        hi = range[1][k] > hi ? range[1][k] : hi;
    }
    const size_t at = (size_t)r * w.slices + sl;
#pragma unroll
    for (int k = 0; k < NB1 / MW_THREADS; ++k) {
        const int bin = k * MW_THREADS + tid;
        if (bin >= lo && bin <= hi) w.hist[at * NB1 + bin] = bins[k];
    }
    if (tid == 0) w.head[at] = MwHead{lo, hi, any_bad ? 1 : 0, 0};
}

__global__ __launch_bounds__(MW_THREADS) void mw_hist_kernel(MwLaunch w) { mw_hist<false>(w); }

// Step 2.
template <bool LEAN> __device__ __forceinline__ void mw_collect(const MwLaunch &w)
{
    __shared__ unsigned long long hist[HIST1];
    __shared__ Located located;
    __shared__ int sums[MW_WAVES];
    __shared__ int ends[2][MW_WAVES];
    __shared__ int found;
    const SelectLaunch &a = w.a;
    mw_preload(w);
    const int r = blockIdx.x, sl = blockIdx.y;
    const int b = a.per_h.divide(r), h = r - b * a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int len = mw_row_len(a, b);
    const size_t row_at = (size_t)r * w.slices, at = row_at + sl;
    // (requested ahead of the slice: the histograms are fetched as soon as the ranges are here)
    const MwHead head = w.head[LEAN ? (size_t)r : row_at + (lane < w.slices ? lane : 0)];
    MwSlice slice(w, b, h, sl, len);
    if (tid == 0) found = 0;
    int cnt[NB1 / MW_THREADS];
    const bool bad = mw_gather(hist, head, w.hist + (LEAN ? (size_t)r : row_at) * NB1, LEAN ? 1 : w.slices, LEAN ? 0 : sl, cnt);
    double target = 0.0, m_above = 0.0;
    unsigned c_above = 0;
    unsigned long long bin_packed = 0;
    const int bin = locate_bin<NB1, true, true>(hist, located, 0, a.top_p, target, m_above, c_above, bin_packed);
    const bool invalid = bad || bin < 0 || len == 0;                     // uniform
    if (sl == 0 && tid == 0) w.state[r] = MwState{bin_packed, target, m_above, c_above, bin, invalid ? 1 : 0};
    if (invalid) return;
    const uint32_t want = (uint32_t)bin;
    uint32_t *mine = w.entries + at * w.collect;
    int lo = 0x7fffffff, hi = 0, counted = 0;
    slice.each([&](uint32_t x) {
        if constexpr (LEAN) counted += ((int)x >> 20) > bin ? 1 : 0;     // (-0.0 is below every bin)
        if ((x >> 20) == want && x) {
            const int k = atomicAdd(&found, 1);
            if (k < w.collect) mine[k] = x;
            lo = (int)x < lo ? (int)x : lo;
            hi = (int)x > hi ? (int)x : hi;
        }
    });
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int l = __shfl_xor(lo, off, 64), g = __shfl_xor(hi, off, 64);
        lo = l < lo ? l : lo;
        hi = g > hi ? g : hi;
    }
    if (lane == 0) { ends[0][tid >> 6] = lo; ends[1][tid >> 6] = hi; }
    int above = counted;
    if constexpr (!LEAN) {
#pragma unroll
        for (int k = 0; k < NB1 / MW_THREADS; ++k)
            if (k * MW_THREADS + tid > bin) above += cnt[k];
    }
    above = mw_sum(above, sums);                                         // (a barrier: `found` and `ends` are complete)
#pragma unroll
    for (int k = 0; k < MW_WAVES; ++k) {
        lo = ends[0][k] < lo ? ends[0][k] : lo;
        hi = ends[1][k] > hi ? ends[1][k] : hi;
    }
    if (tid == 0) w.counts[at] = make_int4(above, found, lo, hi);
}

__global__ __launch_bounds__(MW_THREADS) void mw_collect_kernel(MwLaunch w) { mw_collect<false>(w); }

// Step 3: tau*, count and flags of the row (slice 0), and the list entries of the slice.
__global__ __launch_bounds__(MW_THREADS) void mw_emit_kernel(MwLaunch w)
{
    __shared__ unsigned long long hist2[HIST2], hist3[HIST2];
    __shared__ Located located;
    __shared__ uint32_t kept_lds[MW_LDS_ENTRIES];
    __shared__ int sums[MW_WAVES];
    __shared__ unsigned tot[2][MW_FLIGHT * MW_WAVES];
    const SelectLaunch &a = w.a;
    mw_preload(w);
    const int r = blockIdx.x, sl = blockIdx.y;
    const int b = a.per_h.divide(r), h = r - b * a.H_kv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int len = mw_row_len(a, b);
    const size_t row_at = (size_t)r * w.slices;
    const MwState st = w.state[r];
    int4 count = w.counts[row_at + (lane < w.slices ? lane : 0)];        // lane j: slice j's (never written for an invalid row)
    clear_hist<MW_THREADS, HIST2>(hist2);                                // (while they are on their way)
    clear_hist<MW_THREADS, HIST2>(hist3);
    if (lane >= w.slices) count.x = count.y = 0;                         // (slice 0's smallest and largest again)
    if (st.invalid) {
        if (sl == 0 && tid == 0) {
            a.counts[r] = 0;
            if (a.thresholds) a.thresholds[r] = 0.0f;
            if (a.row_flags) a.row_flags[r] = SPECATTN_ROW_INVALID;
        }
        return;
    }
    const int e_field = st.bin >> 3;
    const uint32_t want = (uint32_t)st.bin;
    const int place = wave_inclusive_sum(count.y);                       // the row's collected entries up to slice `lane`
    const int all = __builtin_amdgcn_readlane(place, 63);
    const int earlier = sl ? __builtin_amdgcn_readlane(place, sl - 1) : 0;
    int base = lane < sl ? count.x : 0;
    base = __builtin_amdgcn_readlane(wave_inclusive_sum(base), 63);      // kept positions of the slices before this one: so far those above the bin
    const bool in_lds = all <= MW_LDS_ENTRIES && !__any(count.y > w.collect);
    // fn(entry, its number in slice order) for the row's entries in the boundary bin, of slices 0 .. last
    auto each_from_memory = [&](int last, auto &&fn) {
        // Two slices per wave at a time, eight loads of either in flight.
        for (int j = wave; j <= last; j += 2 * MW_WAVES) {
            const uint32_t *src[2];
            int n[2], first[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int js = j + s * MW_WAVES;
                src[s] = w.entries + (row_at + min(js, w.slices - 1)) * w.collect;
                n[s] = __builtin_amdgcn_readlane(count.y, js & 63);
                first[s] = __builtin_amdgcn_readlane(place, js & 63) - n[s];
                if (js > last || n[s] > w.collect) n[s] = 0;
            }
            for (int k0 = 0; k0 < max(n[0], n[1]); k0 += 512) {
                uint32_t x[2][8];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[s][i] = src[s][min(k0 + i * 64 + lane, max(n[s], 1) - 1)];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (k0 + i * 64 + lane < n[s]) fn(x[s][i], first[s] + k0 + i * 64 + lane);
            }
        }
        if (in_lds) return;
        for (int j = 0; j <= last; ++j) {                                // flat rows: the slice again (its entries have no numbers)
            const int n = __builtin_amdgcn_readlane(count.y, j);
            if (n <= w.collect) continue;
            MwSlice other(w, b, h, j, len);
            other.each([&](uint32_t x) { if ((x >> 20) == want && x) fn(x, 0); });
        }
    };
    auto each_entry = [&](auto &&fn) {
        if (in_lds) {
            for (int k = tid; k < all; k += MW_THREADS) fn(kept_lds[k], k);
        } else {
            each_from_memory(w.slices - 1, fn);
        }
    };
    // An entry into its bin of a histogram.  Lanes that hold the same value as the first one are added by that lane (a
    // row of ties would otherwise queue up at one counter; both fields of a counter scale with the number of entries).
    auto add = [&](unsigned long long *hist, uint32_t x, uint32_t bin) {
        const uint32_t at = hist_slot<NB2>(bin);
        const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
        const unsigned long long same = __ballot(x == lead);
        if (x != lead) atomicAdd(&hist[at], packed_entry(x));
        else if (lane == (int)__ffsll((long long)same) - 1) atomicAdd(&hist[at], packed_entry(x) * (unsigned long long)__popcll(same));
    };
    int lo = count.z, hi = count.w;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int l = __shfl_xor(lo, off, 64), g = __shfl_xor(hi, off, 64);
        lo = l < lo ? l : lo;
        hi = g > hi ? g : hi;
    }
    const bool tied = lo == hi;                                          // one entry, or entries of one value: that is tau*
    double target = st.target, m_above = st.m_above;
    unsigned c_above = st.c_above;
    unsigned long long bin_packed = st.bin_packed;
    uint32_t tau_bits = (uint32_t)lo;
    if (in_lds && !tied) each_from_memory(w.slices - 1, [&](uint32_t x, int k) { kept_lds[k] = x; });
    MwSlice slice(w, b, h, sl, len);
    if (tied) {
        base += earlier;
    } else {
        __syncthreads();                                                 // the histograms are clear, the entries in LDS
        each_entry([&](uint32_t x, int) { add(hist2, x, (x >> 10) & 1023u); });
        __syncthreads();
        const int b2 = locate_bin<NB2, false, true>(hist2, located, e_field, a.top_p, target, m_above, c_above, bin_packed);
        const uint32_t prefix = (want << 10) | (uint32_t)b2;
        if ((bin_packed >> CNT_SHIFT) == 1) {
            tau_bits = ((uint32_t)e_field << 23) | ((uint32_t)bin_packed & 0x7fffffu);
        } else {
            each_entry([&](uint32_t x, int) { if ((x >> 10) == prefix) add(hist3, x, x & 1023u); });
            __syncthreads();
            const int b3 = locate_bin<NB2, false, true>(hist3, located, e_field, a.top_p, target, m_above, c_above, bin_packed);
            tau_bits = (prefix << 10) | (uint32_t)b3;
        }
        int mine = 0;
        if (in_lds) {
            for (int k = tid; k < earlier; k += MW_THREADS) mine += kept_lds[k] >= tau_bits ? 1 : 0;
        } else {
            each_from_memory(sl - 1, [&](uint32_t x, int) { mine += x >= tau_bits ? 1 : 0; });
        }
        base += mw_sum(mine, sums);
    }
    if (sl == 0 && tid == 0) {
        const unsigned kept = c_above + (unsigned)(bin_packed >> CNT_SHIFT);
        a.counts[r] = (int32_t)kept;
        if (a.thresholds) a.thresholds[r] = __uint_as_float(tau_bits);
        if (a.row_flags) {
            const double row_sum = target / (double)a.top_p;
            const double m_incl = m_above + mass_of(bin_packed, e_field), band = 1e-6 * row_sum;
            uint32_t f = (fabs(m_incl - target) <= band || fabs(m_above - target) <= band) ? SPECATTN_ROW_NEAR_BOUNDARY : 0u;
            if (kept > (unsigned)a.idx_capacity) f |= SPECATTN_ROW_OVERFLOW;
            a.row_flags[r] = f;
        }
    }
    int32_t *out = a.indices + (int64_t)r * a.idx_stride;
    const int32_t *ptab = (a.emit_physical && a.page_table) ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    int turn = 0;
    for (int p0 = slice.begin; p0 < slice.end; p0 += MW_FLIGHT * MW_ITEM, turn ^= 1) {
        if (p0 != slice.begin) slice.request(p0);
        // (compared as signed integers: -0.0, the only signed value of a valid row, is below any threshold)
        unsigned before[MW_FLIGHT], keep[MW_FLIGHT];
#pragma unroll
        for (int i = 0; i < MW_FLIGHT; ++i) {
            const int t = (int)tau_bits;
            const uint4 u = slice.entries(i);
            const bool f0 = (int)u.x >= t, f1 = (int)u.y >= t, f2 = (int)u.z >= t, f3 = (int)u.w >= t;
            const unsigned long long m0 = __ballot(f0), m1 = __ballot(f1), m2 = __ballot(f2), m3 = __ballot(f3);
            const unsigned long long below = (1ull << lane) - 1ull;
            before[i] = __popcll(m0 & below) + __popcll(m1 & below) + __popcll(m2 & below) + __popcll(m3 & below);
            keep[i] = (f0 ? 1u : 0u) | (f1 ? 2u : 0u) | (f2 ? 4u : 0u) | (f3 ? 8u : 0u);
            if (lane == 0) tot[turn][i * MW_WAVES + wave] = __popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3);
        }
        __syncthreads();
        const int part = lane < MW_FLIGHT * MW_WAVES ? (int)tot[turn][lane] : 0;
        const int inc = wave_inclusive_sum(part);
#pragma unroll
        for (int i = 0; i < MW_FLIGHT; ++i) {
            int o = base + __shfl(inc - part, i * MW_WAVES + wave, 64) + (int)before[i];
            const int p = p0 + i * MW_ITEM + tid * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((keep[i] >> c) & 1u) {
                    const int pos = p + c;
                    if (o < a.idx_capacity)
                        out[o] = ptab ? ((ptab[pos >> a.page_shift] << a.page_shift) | (pos & ((1 << a.page_shift) - 1))) : pos;
                    ++o;
                }
        }
        base += __builtin_amdgcn_readlane(inc, 63);
    }
}
static_assert(MW_FLIGHT * MW_WAVES <= 64, "a wave scans the totals of a round");

// The lean form.  (These kernels stand behind the three above: between them they cost those half a microsecond of 50,
// by where the code then lies.)  Clears a row per workgroup.
__global__ __launch_bounds__(MW_THREADS) void mw_clear_kernel(MwLaunch w)
{
#pragma unroll
    for (int k = 0; k < NB1 / MW_THREADS; ++k) w.hist[(size_t)blockIdx.x * NB1 + k * MW_THREADS + threadIdx.x] = 0ull;
    if (threadIdx.x == 0) w.head[blockIdx.x] = MwHead{0, NB1 - 1, 0, 0};
}
__global__ __launch_bounds__(MW_THREADS) void mw_hist_lean_kernel(MwLaunch w) { mw_hist<true>(w); }
__global__ __launch_bounds__(MW_THREADS) void mw_collect_lean_kernel(MwLaunch w) { mw_collect<true>(w); }

inline size_t mw_align(size_t x) { return (x + 255) & ~(size_t)255; }

struct MwPlan { int slices, slice_len; };
MwPlan mw_plan(int rows, int n)
{
    MwPlan p;
    // One workgroup per CU while it gets its slice with one round of loads (8192 positions), else two; at most 16 slices of
    // up to 8192 positions each (added up with 16 loads in flight), 32 for longer rows.  Measured with one / two per CU: 32 rows of
    // 65536 21.8 / 26.2 us, 64 of 32768 20.9 / 25.2, 32 of 131072 29.0 / 28.6, 64 of 131072 40.9 / 36.1; 8 rows of 65536 with
    // 16 / 32 slices 20.4 / 22.8, 8 of 200001 30.0 / 26.5.
    constexpr int ONE_ROUND = MW_FLIGHT * MW_ITEM;
    const int per_cu = (int64_t)rows * n <= (int64_t)ONE_ROUND * cu_count() ? 1 : 2;
    const int most = n <= MW_MOST_SLICES / 2 * ONE_ROUND ? MW_MOST_SLICES / 2 : MW_MOST_SLICES;
    int want = (per_cu * cu_count() + rows - 1) / rows;
    want = want > most ? most : want;
    p.slice_len = ((n + want - 1) / want + MW_ITEM - 1) / MW_ITEM * MW_ITEM;
    p.slices = (n + p.slice_len - 1) / p.slice_len;
    return p;
}

// One thread per (row, chunk), where the selection does not add the chunks up itself (select_takes_chunks).
__global__ __launch_bounds__(256) void chunk_mass_kernel(const float *__restrict__ probs, int64_t stride_b,
                                                         int64_t stride_h, int H, int n_tokens,
                                                         const int32_t *__restrict__ seq_lens, int chunk_shift,
                                                         int n_chunks, int64_t total, float *__restrict__ mass)
{
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= total) return;
    const int64_t r = gid / n_chunks;
    const int c = (int)(gid - r * n_chunks);
    const int b = (int)(r / H), h = (int)(r - (int64_t)b * H);
    int len = seq_lens ? seq_lens[b] : n_tokens;
    len = len < 0 ? 0 : (len > n_tokens ? n_tokens : len);
    mass[gid] = chunk_mass(probs + (int64_t)b * stride_b + (int64_t)h * stride_h, len, c, chunk_shift);
}

}  // namespace

specattn_status launch_chunk_masses(const float *probs, int64_t stride_b, int64_t stride_h, int B, int H, int n_tokens,
                                    const int32_t *seq_lens, int chunk_shift, int n_chunks, float *mass,
                                    hipStream_t stream)
{
    const int64_t total = (int64_t)B * H * n_chunks;
    const unsigned grid = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(chunk_mass_kernel, dim3(grid), dim3(256), 0, stream, probs, stride_b, stride_h, H, n_tokens,
                       seq_lens, chunk_shift, n_chunks, total, mass);
    return check_launch("chunk_mass_kernel");
}

bool select_multi_wg_preferred(int rows, int n, float top_p)
{
    // One workgroup per row leaves most of the chip idle when there are few rows, takes a CU to itself beyond 32768 entries
    // and streams the row in every pass beyond 65536; the split costs two more launches.  Lists of more than 24576 positions take the one
    // workgroup a second round, so calls that ask for nearly all of the mass are split earlier.  Measured, one workgroup per row / split, us:
    // top_p = 0.9       8 x 34816 17.3 / 19.3, x 36800 18.7 / 19.5, x 40000 19.4 / 19.1, x 65536 21.2 / 20.2; 32 x 34816 17.7 / 19.6, x 36800 19.0 / 19.5,
    //                   x 40000 19.5 / 19.2, x 65536 23.9 / 20.2; 64 x 34816 18.0 / 23.9, x 40000 18.2 / 23.7, x 65536 24.3 / 25.6;
    //                   96 x 60000 23.5 / 44.1; 128 x 65536 25.6 / 34.0; 512 x 65536 59.5 / 92.4; 256 x 131072 104 / 86
    // top_p = 0.99      8 x 34816 17.8 / 19.4, x 36800 18.4 / 19.4; 32 x 34816 19.1 / 19.9, x 36800 20.4 / 19.8; 64 x 34816 20.0 / 24.8
    // top_p = 0.999     8 x 34816 22.4 / 18.8, x 36800 23.9 / 19.0; 32 x 34816 23.2 / 19.3, x 36800 25.5 / 19.3; 64 x 34816 23.3 / 24.2
    // top_p = 1         8 x 34816 10.8 / 15.7, with zeros in the rows 21.3 / 15.7; 32 x 34816 11.2 / 18.5, 22.8 / 18.5; 64 x 34816 12.0 / 23.6, 21.9 / 23.4
    const int cus = cu_count();
    if (n > SELECT_RESIDENT) return rows <= 4 * cus;
    return n > (top_p > 0.99f && rows <= cus / 8 ? 32768 : 36863) && rows <= cus / 4;
}

size_t select_multi_wg_bytes(int rows, int n)
{
    const MwPlan plan = mw_plan(rows, n);
    const size_t S = (size_t)rows * plan.slices;
    return mw_align(S * NB1 * 8) + mw_align(S * (plan.slice_len >> MW_COLLECT_SHIFT) * 4) + mw_align(S * sizeof(MwHead)) + mw_align(S * sizeof(int4)) +
           mw_align((size_t)rows * sizeof(MwState));
}

// `scratch` holds select_multi_wg_bytes, or at least 20 KiB per row
specattn_status launch_select_multi_wg(const SelectLaunch &a, void *scratch, size_t scratch_bytes, hipStream_t stream)
{
    const int rows = a.B * a.H_kv;
    const MwPlan plan = mw_plan(rows, a.n_max);
    const size_t S = (size_t)rows * plan.slices;
    const bool lean = scratch_bytes < select_multi_wg_bytes(rows, a.n_max);
    const size_t hists = lean ? (size_t)rows : S;
    MwLaunch w;
    w.a = a;
    w.a.per_h = FastDivisor(a.H_kv);
    w.slices = plan.slices;
    w.slice_len = plan.slice_len;
    w.collect = plan.slice_len >> MW_COLLECT_SHIFT;
    if (lean) {
        const size_t fixed = mw_align(hists * NB1 * 8) + mw_align(hists * sizeof(MwHead)) + mw_align(S * sizeof(int4)) + mw_align((size_t)rows * sizeof(MwState));
        if (scratch_bytes < fixed) { set_error("workspace has %zu bytes, too few for the split selection", scratch_bytes); return SPECATTN_EWORKSPACE; }
        const size_t room = ((scratch_bytes - fixed) & ~(size_t)255) / 4 / S;
        if (room < (size_t)w.collect) w.collect = (int)room;
    }
    char *p = static_cast<char *>(scratch);
    w.hist = reinterpret_cast<unsigned long long *>(p); p += mw_align(hists * NB1 * 8);
    w.entries = reinterpret_cast<uint32_t *>(p); p += mw_align(S * w.collect * 4);
    w.head = reinterpret_cast<MwHead *>(p); p += mw_align(hists * sizeof(MwHead));
    w.counts = reinterpret_cast<int4 *>(p); p += mw_align(S * sizeof(int4));
    w.state = reinterpret_cast<MwState *>(p);
    // The slices of a row on one XCD (rows a multiple of eight): what they hand each other stays in its L2.  Next to each other, so dealt to all
    // XCDs / so, us: 32 rows of 131072 23.8 / 22.4, 8 of them 17.8 / 17.0, 32 of 70000 22.8 / 21.9, 8 of 65536 19.7 / 18.7, 24 of 131072 23.1 / 22.1.
    const dim3 grid((unsigned)rows, (unsigned)plan.slices);
    if (lean) {
        hipLaunchKernelGGL(mw_clear_kernel, dim3(rows), dim3(MW_THREADS), 0, stream, w);
        hipLaunchKernelGGL(mw_hist_lean_kernel, grid, dim3(MW_THREADS), 0, stream, w);
        hipLaunchKernelGGL(mw_collect_lean_kernel, grid, dim3(MW_THREADS), 0, stream, w);
    } else {
        hipLaunchKernelGGL(mw_hist_kernel, grid, dim3(MW_THREADS), 0, stream, w);
        hipLaunchKernelGGL(mw_collect_kernel, grid, dim3(MW_THREADS), 0, stream, w);
    }
    hipLaunchKernelGGL(mw_emit_kernel, grid, dim3(MW_THREADS), 0, stream, w);
    return check_launch("mw_emit_kernel");
}

bool select_takes_chunks(int rows, int n_tokens, int n_chunks)
{
    // A launch and the masses' way through memory less, and with many rows a row's reads overlap other rows' passes; few
    // long rows are read faster by more workgroups than they have.  Measured, us, masses by a kernel of their own / added
    // up in the selection (rows x positions / chunk): 32 x 2044 / 16 8.9 / 5.6, 64 x 16384 / 8 9.0 / 8.5, 384 x 32768 / 16 16.9 / 12.8,
    // 2048 x 32768 / 8 68.8 / 54.1, 512 x 65536 / 32 29.9 / 27.5, 32 x 30000 / 512 47.6 / 36.5; 8 x 65536 / 32 9.6 / 13.3, 32 x 65536 / 32 8.9 / 12.8,
    // 8 x 131072 / 64 9.5 / 19.7; nearly even between: 8 x 40000 / 32 9.1 / 10.1, 32 x 59000 / 16 10.5 / 11.2, 128 x 65536 / 32 12.8 / 13.8,
    // x 131072 / 64 20.9 / 21.8.
    return n_chunks <= 4096 && (n_tokens < 60000 || rows > cu_count() / 4);
}

// a.probs: rows of positions, a.n_max: chunks of a row.  Workgroups as launch_select takes them, but 512 threads for the
// shortest rows too: adding the chunks up is most of their work.
specattn_status launch_select_chunks(const SelectLaunch &a, hipStream_t stream)
{
    const bool few = a.B * a.H_kv <= 2 * cu_count();
    if (a.n_max > 2048) return few ? launch_one<512, 2, true>(a, stream) : launch_one<256, 4, true>(a, stream);
    if (few) return launch_one<512, 1, true>(a, stream);
    return a.n_max <= 1024 ? launch_one<256, 1, true>(a, stream) : launch_one<256, 2, true>(a, stream);
}

specattn_status launch_select(const SelectLaunch &a, hipStream_t stream)
{
    const int n = a.n_max, rows = a.B * a.H_kv, cus = cu_count();
    // Few rows: as many threads as shorten a row's passes (512 up to 8192 entries, 1024 beyond while every row has a CU of its
    // own).  Many rows: the shape that fits most rows on the chip at once, so that one row's load overlaps another row's
    // passes (workgroups of 256 / 512 / 1024 threads: four to six / two or three / one to a CU).
    // Block counts are per 1024 positions, so every variant has THREADS*4 a multiple of 1024.
    // Measured, us (256 CUs; shape: time):
    //   2044 x 64 rows      512x1 6.3, 256x2 6.8;        2044 x 1024   256x2 8.4, 512x1 9.4
    //   4096 x 512          512x2 7.9, 256x4 8.1;        4096 x 1024   256x4 10.3, 512x2 11.0
    //   8192 x 128          512x4 8.0, 1024x2 8.4;       8192 x 512    512x4 10.7, 256x8 11.3
    //   8192 x 768          256x8 12.7, 512x4 12.9;      8192 x 1024   256x8 14.3, 512x4 17.3
    //   13001 x 64          1024x4 9.4, 512x8 9.7;       16384 x 256   1024x4 10.7, 512x8 11.5
    //   16384 x 512         512x8 14.8, 256x16 16.6;     13001 x 1024  256x16 21.2, 512x8 24.6
    //   16384 x 2048        256x16 37.7, 512x8 49.8
    //   32768 x 256         1024x8 15.8, 512x16 18.2;    32768 x 384   512x16 22.9, 1024x8 29.8
    if (n <= 1024) return launch_one<256, 1>(a, stream);
    if (n <= 2048) return rows <= 2 * cus ? launch_one<512, 1>(a, stream) : launch_one<256, 2>(a, stream);
    if (n <= 4096) return rows <= 2 * cus ? launch_one<512, 2>(a, stream) : launch_one<256, 4>(a, stream);
    if (n <= 8192) return rows <= 2 * cus ? launch_one<512, 4>(a, stream) : launch_one<256, 8>(a, stream);
    if (n <= 16384) {
        if (rows <= cus) return launch_one<1024, 4>(a, stream);
        return rows <= 2 * cus ? launch_one<512, 8>(a, stream) : launch_one<256, 16>(a, stream);
    }
    if (n <= 32768) return rows > cus ? launch_one<512, 16>(a, stream) : launch_one<1024, 8>(a, stream);
    if (n <= SELECT_RESIDENT) return launch_one<1024, 16>(a, stream);
    hipLaunchKernelGGL(topp_select_stream_kernel, dim3(rows), dim3(STREAM_THREADS), 0, stream, a);
    return check_launch("topp_select_stream_kernel");
}

}  // namespace specattn
