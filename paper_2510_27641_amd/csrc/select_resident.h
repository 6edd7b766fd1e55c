// Selection of rows that one workgroup holds in its registers (up to THREADS * 4 * NV4 entries; read once from memory).  Part of
// select.hip, which has the method.
//
// The passes over the registers are bound by instruction issue and by the LDS unit's 64-bit atomics, and short rows by the chain of
// barriers and locate steps, so the digits are chosen for few and cheap passes: the first one covers the 32 octaves below the row's
// largest entry with 64 bins each, so that the boundary bin holds three entries of a thousand instead of thirty.  What lies below these
// octaves is added up in fp64 for the row's sum and gets bins, one per octave, in a pass of its own if the boundary turns out to lie there.
// The second pass, over ten more bits, then finds few entries and nearly always leaves a bin with a single one, which is tau*.  With eight
// bins per octave over all exponents, as the split selection has them, every wave met entries of the boundary bin in nearly every vector of
// the second pass, and every other row took a third one.
// Compaction works on words of 32 kept bits, which costs two instructions per entry, instead of on ranks of single entries.
// Rows x entries with eight bins per octave and ranks / now, us: 1024 x 32768 60.4 / 44.2 (the LDS unit is busy 45 % of the time, the vector
// ALU 50 %), 2048 x 32768 108 / 80, 512 x 65536 87 / 61, 2048 x 16384 60.0 / 38.2, 64 x 13001 10.6 / 9.4, 128 x 4096 7.2 / 6.0, 8 x 8192 8.2 / 8.1,
// 8 x 1024 5.6 / 5.3.  Rows of equal entries save no pass and pay for the row's largest entry: 200 x 200 6.5 / 6.8.
#pragma once

// Bins of the first pass: FINE of them from the lowest exponent of the window up.  A bin's entries share their exponent, so its mass is an
// exact integer sum.  Entries below the window, should they be needed: one bin per exponent field.
constexpr int FINE_OCTAVES = 32, FINE_SHIFT = 17, FINE = FINE_OCTAVES << (23 - FINE_SHIFT), OCTAVES = 256;
constexpr int DIGIT = 10, DIGIT_BINS = 1 << DIGIT;               // later passes
constexpr int RES_HIST = FINE + DIGIT_BINS;
static_assert(OCTAVES <= DIGIT_BINS, "the octaves below the window use the second histogram");

// Counters here hold the count and the sum of the 23 fraction bits; the hidden bits are put back where a mass is read.
__device__ __forceinline__ unsigned long long fraction_entry(uint32_t u) { return CNT_ONE | (u & 0x7fffffu); }
__device__ __forceinline__ double fraction_mass(unsigned long long packed, int e_field)
{
    const unsigned long long hidden = e_field > 0 ? (packed >> CNT_SHIFT) << 23 : 0ull;
    const double s = (double)(long long)((packed & SIG_MASK) + hidden);
    return s * __hiloint2double((1023 + (e_field > 0 ? e_field : 1) - 150) << 20, 0);
}

struct Place {                   // outcome of a locate step
    double target, m_above;      // p * (row sum); mass above the boundary bin
    unsigned long long packed;   // the boundary bin's counter
    unsigned c_above;            // entries above it
    uint32_t lo;                 // its lowest bit pattern, and how many bits it leaves open; bits < 0: no mass at all
    int bits;
};

// The entries of a boundary bin of at most FINE_SHIFT open bits, as distances from its lowest pattern, and for each of them the number
// of those not below it (upper byte) and the sum of their distances (128 distances below 2^17 stay below 2^24).
constexpr int LISTED = 128;
struct BinList {
    alignas(16) int entry[LISTED];                             // -1: none
    uint32_t not_below[LISTED];
    int n;
};

struct ResidentShared {
    BinList list;
    Place place;
    uint32_t top[16];            // largest entry of every wave; all ones: an invalid one
    double low[16];              // sum of every wave's entries below the window
    double window_mass;          // of the entries in the window, and how many they are
    unsigned window_count;
    int below;                   // the boundary may lie below the window
    unsigned wave_sum[16];
};

// Sum of BPL counters of a lane's row of bins.  Rows start 128 or 256 bytes apart: every lane takes them in an order of its own, so
// that the lanes of a read fall on different banks.  Bound by the reads' latency: PAIRED ones bring two counters each and are all on their way
// together, half as many as before in rounds of eight (us: 8 rows of 1024 5.2 / 4.8, of 8192 7.2 / 7.1, 256 of 16384 11.0 / 10.8).  Beside a row of 64 entries
// per thread there are no registers for that (1024 rows of 32768 46.4 / 51.8): there single ones, eight at a time.
template <int BPL, bool PAIRED> __device__ __forceinline__ unsigned long long row_of_bins(const unsigned long long *row, int lane)
{
    unsigned long long sum = 0ull;
    if constexpr (PAIRED) {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
        constexpr int PAIRS = BPL / 2;
        const int swizzle = BPL == 32 ? lane & 15 : (lane >> 1) & 7;
        const u64x2 *pairs = reinterpret_cast<const u64x2 *>(row);
        u64x2 v[PAIRS];
#pragma unroll
        for (int j = 0; j < PAIRS; ++j) v[j] = pairs[j ^ swizzle];
        __builtin_amdgcn_sched_barrier(0);
        unsigned long long other = 0ull;                   // (two chains)
#pragma unroll
        for (int j = 0; j < PAIRS; ++j) { sum += v[j][0]; other += v[j][1]; }
        return sum + other;
    }
    const int swizzle = BPL == 32 ? lane & 31 : (lane >> 1) & (BPL - 1);
#pragma unroll
    for (int j0 = 0; j0 < BPL; j0 += 8) {
        unsigned long long v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row[(j0 + j) ^ swizzle];
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += v[j];
        __builtin_amdgcn_sched_barrier(0);                 // (not all loads at once)
    }
    return sum;
}

// The bin among 64 or fewer, one per lane from the highest down, whose mass takes the sum above it to the goal (the last non-empty
// one if rounding leaves none).  `counter` is zero for lanes that hold none.
__device__ __forceinline__ int pick_bin(unsigned long long counter, int e_field, double goal, double &m_above, unsigned &c_above, unsigned long long &packed)
{
    const unsigned c = (unsigned)(counter >> CNT_SHIFT);
    double run = c ? fraction_mass(counter, e_field) : 0.0;
    unsigned runc = c;
    wave_prefix(run, runc);
    const unsigned long long filled = __ballot(c > 0), ok = __ballot(c > 0 && m_above + run >= goal);
    const int pick = ok ? (int)__ffsll((long long)ok) - 1 : 63 - __clzll((long long)filled);
    if (pick) { m_above += read_lane(run, pick - 1); c_above += (unsigned)__builtin_amdgcn_readlane((int)runc, pick - 1); }
    packed = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(counter >> 32), pick) << 32 |
             (unsigned)__builtin_amdgcn_readlane((int)(uint32_t)counter, pick);
    return pick;
}

// Decision of the first pass, by the first wave alone.  Its lanes own half an octave of the window each, lane 0 the highest.  (sh.below:
// the window's entries do not reach the target, or top_p is 1, and there are entries below it.)
template <int NW, bool PAIRED> __device__ __forceinline__ void locate_first(const unsigned long long *fine, int e_low, float top_p, ResidentShared &sh)
{
    const int lane = threadIdx.x;
    double low = lane < NW ? sh.low[lane] : 0.0;
    const unsigned long long sum = row_of_bins<FINE / 64, PAIRED>(fine + (63 - lane) * (FINE / 64), lane);
    const double lm = fraction_mass(sum, e_low + ((63 - lane) >> 1));
    const unsigned lc = (unsigned)(sum >> CNT_SHIFT);
    double incl = lm;
    unsigned inclc = lc;
    wave_prefix(incl, inclc);
    double total = read_lane(incl, 63);
    const bool any_low = __any(low != 0.0);
    if (any_low) {                                             // (uniform)
        unsigned none = 0;
        wave_prefix(low, none);
        if (lane == 0) { sh.window_mass = total; sh.window_count = (unsigned)__builtin_amdgcn_readlane((int)inclc, 63); }
        total += read_lane(low, 63);
    }
    Place out;
    out.target = (double)top_p * total;                        // Algorithm 2: M_target = p * sum a
    const double goal = top_p < 1.0f ? out.target : INFINITY;
    // mass and count of the lanes before this one (wave_shr:1)
    const double before = dpp_double<0x138, 0xf>(incl);
    const unsigned beforec = (unsigned)dpp_int<0x138, 0xf>((int)inclc);
    // Masses are non-negative, so the running sum never decreases: the first lane whose sum reaches the target holds the boundary.
    const unsigned long long some = __ballot(lc > 0), holds = __ballot(lc > 0 && before + lm >= goal);
    const int at = holds ? (int)__ffsll((long long)holds) - 1 : some ? 63 - __clzll((long long)some) : 0;
    out.m_above = read_lane(before, at);
    out.c_above = (unsigned)__builtin_amdgcn_readlane((int)beforec, at);
    const int high = (63 - at) * (FINE / 64) + FINE / 64 - 1;  // the boundary lane's highest bin
    const int pick = pick_bin(lane < FINE / 64 ? fine[high - lane] : 0ull, e_low + (high >> (23 - FINE_SHIFT)), goal, out.m_above, out.c_above, out.packed);
    out.lo = ((uint32_t)e_low << 23) + ((uint32_t)(high - pick) << FINE_SHIFT);
    out.bits = FINE_SHIFT;
    if (lane == 0) {
        sh.place = out;
        sh.below = any_low && !holds;
    }
}

// Decision among the octaves below the window, by the first wave: lane 0 owns the four highest exponent fields.  top_p = 1 takes the
// lowest non-empty bin, whatever the rounding of the sums above it; octaves count as empty there from the one down from which on the
// entries all together add less than one unit in the last place of the row's total (a non-empty half octave of the window always adds
// more: it lies within 2^-32 of the largest of at most 65536 entries).
__device__ __forceinline__ void locate_below(const unsigned long long *octave, float top_p, ResidentShared &sh)
{
    const int lane = threadIdx.x;
    unsigned long long four[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) four[g] = octave[(63 - lane) * 4 + g];
    int cut = -1;                                              // exponent fields up to this one count as empty
    double lm, incl;
    unsigned lc, inclc;
    auto add_up = [&]() {
        lm = 0.0;
        lc = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int e = (63 - lane) * 4 + g;
            if (e > cut) { lm += fraction_mass(four[g], e); lc += (unsigned)(four[g] >> CNT_SHIFT); }
        }
        incl = lm;
        inclc = lc;
        wave_prefix(incl, inclc);
    };
    add_up();
    if (!(top_p < 1.0f)) {
        // sums from the bottom up: the lanes in reverse order, then each lane's octaves
        const double total = sh.window_mass + read_lane(incl, 63);
        double tail = __shfl(lm, 63 - lane, 64);
        unsigned none = 0;
        wave_prefix(tail, none);
        tail = __shfl(dpp_double<0x138, 0xf>(tail), 63 - lane, 64);
        const double ulp = __hiloint2double((((__double2hiint(total) >> 20) & 0x7ff) - 52) << 20, 0);
        int fields = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            tail += fraction_mass(four[g], (63 - lane) * 4 + g);
            fields += __popcll(__ballot(tail < ulp));
        }
        cut = fields - 1;
        add_up();
    }
    const unsigned long long some = __ballot(lc > 0);
    if (!some) return;                                         // (the window's lowest bin it is)
    Place out;
    out.target = sh.place.target;
    const double goal = top_p < 1.0f ? out.target : INFINITY;
    const double before = sh.window_mass + dpp_double<0x138, 0xf>(incl);
    const unsigned beforec = sh.window_count + (unsigned)dpp_int<0x138, 0xf>((int)inclc);
    const unsigned long long holds = __ballot(lc > 0 && before + lm >= goal);
    const int at = holds ? (int)__ffsll((long long)holds) - 1 : 63 - __clzll((long long)some);
    out.m_above = read_lane(before, at);
    out.c_above = (unsigned)__builtin_amdgcn_readlane((int)beforec, at);
    const int e = (63 - at) * 4 + 3 - lane;                    // lane 0 looks at the lane's highest octave
    out.lo = (uint32_t)((63 - at) * 4 + 3 - pick_bin(lane < 4 && e > cut ? octave[e] : 0ull, e, goal, out.m_above, out.c_above, out.packed)) << 23;
    out.bits = 23;
    if (lane == 0) sh.place = out;
}

// Decision of a later pass: DIGIT_BINS bins of 2^shift bit patterns each from `place.lo` up.
template <bool PAIRED> __device__ __forceinline__ void locate_next(const unsigned long long *hist, int shift, float top_p, Place &place)
{
    constexpr int BPL = DIGIT_BINS / 64;
    const int lane = threadIdx.x, e_field = (int)(place.lo >> 23);
    const double goal = top_p < 1.0f ? place.target : INFINITY;
    const unsigned long long sum = row_of_bins<BPL, PAIRED>(hist + (63 - lane) * BPL, lane);
    const double lm = fraction_mass(sum, e_field);
    const unsigned lc = (unsigned)(sum >> CNT_SHIFT);
    double incl = lm;
    unsigned inclc = lc;
    wave_prefix(incl, inclc);
    const double before = dpp_double<0x138, 0xf>(incl);
    const unsigned beforec = (unsigned)dpp_int<0x138, 0xf>((int)inclc);
    const unsigned long long some = __ballot(lc > 0), holds = __ballot(lc > 0 && place.m_above + (before + lm) >= goal);
    const int at = holds ? (int)__ffsll((long long)holds) - 1 : 63 - __clzll((long long)some);
    place.m_above += read_lane(before, at);
    place.c_above += (unsigned)__builtin_amdgcn_readlane((int)beforec, at);
    const int high = (63 - at) * BPL + BPL - 1;
    const int pick = pick_bin(lane < BPL ? hist[high - lane] : 0ull, e_field, goal, place.m_above, place.c_above, place.packed);
    place.lo += (uint32_t)(high - pick) << shift;
    place.bits = shift;
}

// Largest v of the wave, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    auto step = [&](uint32_t w) { v = v > w ? v : w; };
    step((uint32_t)dpp_int<0x111, 0xf>((int)v));    // row_shr:1
    step((uint32_t)dpp_int<0x112, 0xf>((int)v));    // row_shr:2
    step((uint32_t)dpp_int<0x114, 0xf>((int)v));    // row_shr:4
    step((uint32_t)dpp_int<0x118, 0xf>((int)v));    // row_shr:8
    step((uint32_t)dpp_int<0x142, 0xa>((int)v));    // row_bcast:15 into rows 1 and 3
    step((uint32_t)dpp_int<0x143, 0xc>((int)v));    // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Decision inside a boundary bin whose entries are listed: every wave compares them with a part of the list, and then takes the
// decision by itself.  Uniform over the workgroup, one barrier.
template <int NW> __device__ __forceinline__ void locate_listed(BinList &list, float top_p, Place &place)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = (int)(place.packed >> CNT_SHIFT);
    const bool two = n > 64;                                   // (uniform)
    const int v0 = list.entry[lane], v1 = two ? list.entry[lane + 64] : -1;
    uint32_t s0 = 0u, s1 = 0u;
    for (int j = wave * 4; j < n; j += NW * 4) {               // (all lanes read the same four)
        const int4 w = *reinterpret_cast<const int4 *>(&list.entry[j]);
        auto compare = [&](int x) {                            // (-1 is below every entry)
            const uint32_t one = (1u << 24) + (uint32_t)x;
            s0 += x >= v0 ? one : 0u;
            if (two) s1 += x >= v1 ? one : 0u;
        };
        compare(w.x); compare(w.y); compare(w.z); compare(w.w);
    }
    if (lane < n) atomicAdd(&list.not_below[lane], s0);
    if (lane + 64 < n) atomicAdd(&list.not_below[lane + 64], s1);
    __syncthreads();
    s0 = list.not_below[lane];
    s1 = two ? list.not_below[lane + 64] : 0u;
    const int e_field = (int)(place.lo >> 23);
    const double goal = top_p < 1.0f ? place.target : INFINITY;
    // packed counter of `c` entries whose distances add up to `sum` (at most 128 fractions: below 2^31)
    const uint32_t fraction = place.lo & 0x7fffffu;
    auto counter = [&](unsigned c, uint32_t sum) { return (unsigned long long)c << CNT_SHIFT | (c * fraction + sum); };
    auto reaches = [&](int v, uint32_t s) { return v >= 0 && place.m_above + fraction_mass(counter(s >> 24, s & 0xffffffu), e_field) >= goal; };
    const int reached = (int)wave_max(max(reaches(v0, s0) ? v0 + 1 : 0, reaches(v1, s1) ? v1 + 1 : 0));
    const int tau = reached ? reached - 1 : (int)~wave_max(~min((uint32_t)v0, (uint32_t)v1));
    const unsigned long long at0 = __ballot(v0 == tau), at1 = __ballot(v1 == tau);
    const uint32_t s = (uint32_t)(at0 ? __builtin_amdgcn_readlane((int)s0, (int)__ffsll((long long)at0) - 1)
                                      : __builtin_amdgcn_readlane((int)s1, (int)__ffsll((long long)at1) - 1));
    const unsigned ties = (unsigned)(__popcll(at0) + __popcll(at1)), above = (s >> 24) - ties;
    if (above) place.m_above += fraction_mass(counter(above, (s & 0xffffffu) - ties * (uint32_t)tau), e_field);
    place.c_above += above;
    place.packed = counter(ties, ties * (uint32_t)tau);
    place.lo += (uint32_t)tau;
    place.bits = 0;
}

__device__ __forceinline__ uint32_t median(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t m;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}

// Rows of at most BRIEF chunks: every wave adds up, for each entry, those of a part of the row that are not below it, and then takes the
// whole decision by itself (`v0`, `v1`: the row's entries, two to a lane, zeros behind its end).  A sum takes its terms in the same order for
// every entry, so sums never decrease towards smaller entries.  Uniform over the workgroup, one barrier.
constexpr int BRIEF = 128;
template <int NW> __device__ __forceinline__ Place locate_brief(const uint32_t *entries, uint32_t v0, uint32_t v1, int len, double *sums, float top_p)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool two = len > 64;                                 // (uniform)
    double m0 = 0.0, m1 = 0.0;
    for (int j = wave * (BRIEF / NW); j < (wave + 1) * (BRIEF / NW) && j < len; j += 4) {
        const uint4 w = *reinterpret_cast<const uint4 *>(entries + j);           // (all lanes read the same four)
        auto add = [&](uint32_t x) {
            m0 += (double)__uint_as_float(x >= v0 ? x : 0u);
            if (two) m1 += (double)__uint_as_float(x >= v1 ? x : 0u);
        };
        add(w.x); add(w.y); add(w.z); add(w.w);
    }
    sums[wave * BRIEF + lane] = m0;
    sums[wave * BRIEF + 64 + lane] = m1;
    __syncthreads();
    m0 = m1 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        m0 += sums[w * BRIEF + lane];
        m1 += sums[w * BRIEF + 64 + lane];
    }
    const uint32_t least = ~wave_max(max(v0 ? ~v0 : 0u, v1 ? ~v1 : 0u));
    auto sum_at = [&](uint32_t v) {                            // of the entries from v up, v one of them
        const unsigned long long at0 = __ballot(v0 == v), at1 = __ballot(v1 == v);
        return at0 ? read_lane(m0, (int)__ffsll((long long)at0) - 1) : read_lane(m1, (int)__ffsll((long long)at1) - 1);
    };
    Place out;
    out.target = (double)top_p * sum_at(least);
    const uint32_t tau = wave_max(max(v0 && m0 >= out.target ? v0 : 0u, v1 && m1 >= out.target ? v1 : 0u));
    const unsigned ties = (unsigned)(__popcll(__ballot(v0 == tau)) + __popcll(__ballot(v1 == tau)));
    out.c_above = (unsigned)(__popcll(__ballot(v0 > tau)) + __popcll(__ballot(v1 > tau)));
    out.m_above = sum_at(tau) - (double)ties * (double)__uint_as_float(tau);
    out.packed = (unsigned long long)ties << CNT_SHIFT | (ties * (tau & 0x7fffffu));
    out.lo = tau;
    out.bits = 0;
    return out;
}

// Eight lanes with eight nibbles each: lane l receives nibble l of every lane, of lane m in nibble m.  (Three exchanges on the vector ALU.)
__device__ __forceinline__ uint32_t transpose_nibbles(uint32_t x, int lane)
{
    const bool b4 = lane & 4, b2 = lane & 2, b1 = lane & 1;
    auto merge = [](uint32_t keep, uint32_t a, uint32_t b) { return (a & keep) | (b & ~keep); };
    int y = __builtin_amdgcn_update_dpp(0, (int)x, 0x104, 0xf, 0x5, false);      // row_shl:4 into the lanes with bit 2 clear ...
    y = __builtin_amdgcn_update_dpp(y, (int)x, 0x114, 0xf, 0xa, false);          // ... and row_shr:4 into the others: lane ^ 4
    x = merge(b4 ? 0xffff0000u : 0x0000ffffu, x, __builtin_amdgcn_alignbit((uint32_t)y, (uint32_t)y, 16));
    y = __builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false);           // quad_perm [2,3,0,1]: lane ^ 2
    x = merge(b2 ? 0xff00ff00u : 0x00ff00ffu, x, __builtin_amdgcn_alignbit((uint32_t)y, (uint32_t)y, b2 ? 8 : 24));
    y = __builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);           // quad_perm [1,0,3,2]: lane ^ 1
    return merge(b1 ? 0xf0f0f0f0u : 0x0f0f0f0fu, x, __builtin_amdgcn_alignbit((uint32_t)y, (uint32_t)y, b1 ? 4 : 28));
}

// Dynamic LDS: the histograms, and afterwards in their place the buffer in which a row's list is put together in list order for
// contiguous stores, 16 bits to a position.  Longer lists take several rounds, and every round walks all of the row's kept bits: so it
// holds 24576 positions of rows beyond 16384, 16384 below that and, at 256 threads, several of which share a CU, 13312.  Lists with top_p =
// 0.99, 8192 positions of 32 bits (4096 at 256 threads) / now, us: 24 x 33054 24.2 / 18.4, 64 x 32768 20.7 / 15.9, 1024 x 32768 68.2 / 55.0,
// 512 x 65536 94.0 / 78.6, 2048 x 16384 61.3 / 48.5, 1024 x 8192 20.4 / 17.4; top_p = 0.97, 1024 x 32768 59.6 / 52.1.
constexpr unsigned select_lds(int threads, int nv4)
{
    return threads * nv4 * 4 > 16384 ? 49152 : threads > 256 ? 32768 : 26624;
}

// The sequence that comes k-th (k < n <= 64) when n of them are taken from the longest down, sequences of one level in their order: from the
// top bit of the levels down, those with the bit set come first.  `len`: sequence i's in lane i.  (A level is a length of eight bits.)
__device__ __forceinline__ int kth_longest(int len, int shift, int n, int k)
{
    const uint32_t level = (uint32_t)len >> shift;
    unsigned long long left = n < 64 ? (1ull << n) - 1ull : ~0ull;
    auto halve = [&](unsigned long long first) {
        const unsigned long long with = left & first;
        const int c = __popcll(with);
        left = k < c ? with : left & ~first;
        k -= k < c ? 0 : c;
    };
#pragma unroll
    for (int bit = 7; bit >= 0; --bit) halve(__ballot((level >> bit) & 1u));
    halve(0x00000000ffffffffull);
    halve(0x0000ffff0000ffffull);
    halve(0x00ff00ff00ff00ffull);
    halve(0x0f0f0f0f0f0f0f0full);
    halve(0x3333333333333333ull);
    halve(0x5555555555555555ull);
    return (int)__ffsll((long long)left) - 1;
}

// CHUNKED: a.probs are rows of positions; the workgroup adds the chunks up itself, into the LDS that the histograms take over.
template <int THREADS, int NV4, bool CHUNKED = false>
__global__ __launch_bounds__(THREADS, 4) void topp_select_kernel(SelectLaunch a)
{
    constexpr int NW = THREADS / 64;
    constexpr int ITEM = THREADS * 4;                 // positions per item (one uint4 per thread)
    // A boundary bin of a long row holds tens of entries: three to ten rows in a hundred then met two of them in the boundary bin of the
    // next pass and took one more (1.9 us), and a call waits for its slowest row.  Up to 128 entries go into a list instead and are
    // compared with each other.  Rows x entries, bins / list, us: 64 x 13001 10.4 / 9.4, 4 x 16384 10.2 / 9.3, 256 x 16384 11.5 / 10.5,
    // 256 x 32768 16.9 / 16.3.  Up to 8192 entries the bins are the faster way: few entries, seldom another pass (8 x 8192 7.2 / 7.4,
    // 8 x 2048 5.2 / 5.5), and where rows come in turns (NV4 = 16) another row fills the wait (1024 x 32768 48.1 / 48.2).
    constexpr bool LISTS = ITEM * NV4 > 8192 && NV4 <= 8;
    // (row_of_bins; not where its registers would cost a fifth workgroup per CU: 1088 rows of 8000 12.9 / 15.1 us)
    constexpr bool PAIRED = NV4 <= 8 && !(THREADS == 256 && NV4 == 8);
    constexpr bool FLAT = ITEM * NV4 >= 4096;         // flat rows are added up before they reach a counter
    constexpr bool WORDS = NV4 >= 8;                  // compaction by words of 32 positions instead of item by item
    constexpr int TABLE = WORDS ? ITEM / 32 * NV4 : (NV4 * NW + 63) / 64 * 64;
    __shared__ ResidentShared sh;
    __shared__ __align__(16) unsigned table[TABLE + 4];   // kept entries per word, or per (item, wave), then their exclusive prefix
    extern __shared__ __align__(16) unsigned long long select_dyn[];
    static_assert(RES_HIST * 8 <= (int)select_lds(THREADS, NV4), "the histograms share the list's buffer");
    unsigned long long *hist1 = select_dyn, *hist2 = select_dyn + FINE;
    SPECATTN_PRELOAD(a.probs); SPECATTN_PRELOAD(a.stride_b); SPECATTN_PRELOAD(a.stride_h); SPECATTN_PRELOAD(a.B); SPECATTN_PRELOAD(a.H_kv); SPECATTN_PRELOAD(a.n_max);
    SPECATTN_PRELOAD(a.seq_lens); SPECATTN_PRELOAD(a.top_p); SPECATTN_PRELOAD(a.indices); SPECATTN_PRELOAD(a.idx_stride); SPECATTN_PRELOAD(a.idx_capacity);
    SPECATTN_PRELOAD(a.counts); SPECATTN_PRELOAD(a.thresholds); SPECATTN_PRELOAD(a.row_flags); SPECATTN_PRELOAD(a.page_table); SPECATTN_PRELOAD(a.emit_physical);
    SPECATTN_PRELOAD(a.block_counts); SPECATTN_PRELOAD(a.blocks_per_row); SPECATTN_PRELOAD(a.n_tokens); SPECATTN_PRELOAD(a.chunk_shift); SPECATTN_PRELOAD(a.kept_mask);
    SPECATTN_PRELOAD(a.per_h.mul); SPECATTN_PRELOAD(a.per_h.shift); SPECATTN_PRELOAD(a.by_length);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = a.per_h.divide(blockIdx.x), len;
    const int h = blockIdx.x - b * a.H_kv;
    auto clamped = [&](int n) { return n < 0 ? 0 : (n > a.n_tokens ? a.n_tokens : n); };
    if (a.by_length) {                                         // (uniform)
        const int lens = lane < a.B ? clamped(a.seq_lens[lane]) : 0;
        b = __builtin_amdgcn_readfirstlane(kth_longest(lens, a.by_length - 1, a.B, b));
        len = __builtin_amdgcn_readlane(lens, b);
    } else {
        len = clamped(a.seq_lens ? a.seq_lens[b] : a.n_tokens);
    }
    const int r = b * a.H_kv + h;
    const int positions = len;
    len = (len + (1 << a.chunk_shift) - 1) >> a.chunk_shift;     // rows of chunk masses: length in chunks
    len = len > a.n_max ? a.n_max : len;
    const float *row = a.probs + (int64_t)b * a.stride_b + (int64_t)h * a.stride_h;
    // Items of which this wave holds entries.  (For all waves alike, nearly every wave of a row of odd length held an empty item and took
    // it for zeros: 1100 x 16000 31.2 us, now 29.4; 2048 x 12000 37.6 / 36.1; 520 x 8000 12.8 / 12.4.)
    const int n_items = (len - wave * 256 + ITEM - 1) / ITEM;

    // Every thread issues plain 16-byte loads with nothing between them that waits for data, so all of a thread's loads are in
    // flight together.  They need no more than the 4-byte alignment of a float: the rows of an odd length start anywhere (entry
    // by entry, 64 rows of 13001 took 2 us longer).  An item that reaches past the row's end loads the row's last whole vector
    // instead (in bounds) and is masked afterwards; the at most three entries behind the last whole vector are fetched once, by
    // the thread that owns them.
    uint4 data[NV4];
    uint4 tailv = make_uint4(0, 0, 0, 0);
    const int tail_p = (len & 3) ? (len & ~3) : -1;            // start of the partial vector, if any
    // Short lists of chunks.  The work grows with the square of the chunks, and the line lies where two entries per lane end: with four of
    // them the comparisons break even at 144 chunks for few rows and lose to the bins from 64 on for many.  Bins / comparisons, two to a
    // lane / four, us: 8 rows of 64 chunks 5.7 / 4.2 / 5.4, of 128 5.7 / 4.4 / 5.5, of 144 5.8 / - / 5.8, of 192 5.9 / - / 6.6; 256 of 128 6.0 / 4.6 /
    // 5.9, of 192 6.1 / - / 7.1; 1024 of 64 7.6 / 6.1 / 8.2, of 128 7.7 / 7.0 / 10.2, of 192 8.0 / - / 12.5.  (top_p = 1 has a rule of its own
    // for entries that add nothing.)
    const bool brief = CHUNKED && len <= BRIEF && a.top_p < 1.0f;              // (uniform)
    uint32_t *const entries = reinterpret_cast<uint32_t *>(select_dyn);
    constexpr int BRIEF_SUMS = ITEM * NV4 * 4;                // byte at which the sums start
    if constexpr (CHUNKED) {
        static_assert(BRIEF <= ITEM && BRIEF_SUMS >= ITEM * NV4 * 4 && BRIEF_SUMS % 8 == 0 && BRIEF_SUMS + NW * BRIEF * 8 <= (int)select_lds(THREADS, NV4),
                      "a row's masses wait in dynamic LDS, and behind all of them the sums of locate_brief: waves that still read masses meet no sums");
        float *mass = reinterpret_cast<float *>(select_dyn);
        for (int c = tid; c < ITEM * NV4; c += THREADS) mass[c] = c < len ? chunk_mass(row, positions, c, a.chunk_shift) : 0.0f;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NV4; ++i) data[i] = reinterpret_cast<const uint4 *>(mass)[i * THREADS + tid];
        if (!brief) __syncthreads();
    } else {
        if (tail_p >= 0 && tid == (tail_p % ITEM) / 4) {
            tailv.x = __float_as_uint(row[tail_p]);
            if (tail_p + 1 < len) tailv.y = __float_as_uint(row[tail_p + 1]);
            if (tail_p + 2 < len) tailv.z = __float_as_uint(row[tail_p + 2]);
        }
        const int last4 = (len - 4) & ~3;                      // start of the row's last whole vector
        if (len >= 4) {
#pragma unroll
            for (int i = 0; i < NV4; ++i) {
                const int p = (i * THREADS + tid) * 4;
                // streaming load: a row is read once and should not displace anything in the caches
                const u32x4a v = __builtin_nontemporal_load(reinterpret_cast<const u32x4a *>(row + (p < last4 ? p : last4)));
                data[i] = make_uint4(v.x, v.y, v.z, v.w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NV4; ++i) data[i] = make_uint4(0, 0, 0, 0);
        }
    }
    // the histograms are cleared while the loads are in flight
    if (!brief) clear_hist<THREADS, RES_HIST>(hist1);
    if (LISTS && tid < LISTED) { sh.list.entry[tid] = -1; sh.list.not_below[tid] = 0u; }
    if (LISTS && tid == 0) sh.list.n = 0;

    // Largest and smallest entry.  As an unsigned number a sign bit or an exponent of all ones makes an entry too large: then the thread
    // looks closer (-0.0 is zero; negative, infinite and NaN entries make the row invalid).
    uint32_t row_top = 0u, wave_top = 0u, wave_least = 0u, v0 = 0u, v1 = 0u;
    if (brief) {                                               // (masses are never -0.0)
        v0 = entries[lane];
        v1 = entries[64 + lane];
        row_top = wave_max(max(v0, v1));
    } else {
        uint32_t top = 0u, least = 0xffffffffu;
        auto range = [&](const uint4 &u) {
            const uint32_t x = u.x > u.y ? u.x : u.y, y = u.z > u.w ? u.z : u.w, v = u.x < u.y ? u.x : u.y, w = u.z < u.w ? u.z : u.w;
            top = x > top ? x : top;
            top = y > top ? y : top;
            least = v < least ? v : least;
            least = w < least ? w : least;
        };
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            if (!CHUNKED && (i + 1) * ITEM > len) {                // (uniform) an item that the row does not fill
                const int p = (i * THREADS + tid) * 4;
                if (p + 3 >= len) data[i] = p == tail_p ? tailv : make_uint4(0, 0, 0, 0);
            }
            if (i < n_items) range(data[i]);
        }
        if (top >= 0x7f800000u) {
            bool bad = false;
            auto clean = [&](uint32_t x) -> uint32_t {
                x = x == 0x80000000u ? 0u : x;
                bad = bad || x >= 0x7f800000u;
                return x;
            };
            top = 0u;
            least = 0xffffffffu;
#pragma unroll
            for (int i = 0; i < NV4; ++i) {
                data[i] = make_uint4(clean(data[i].x), clean(data[i].y), clean(data[i].z), clean(data[i].w));
                if (i < n_items) range(data[i]);
            }
            if (bad) top = 0xffffffffu;
        }
        wave_top = wave_max(top);
        wave_least = ~wave_max(~least);
        if (lane == 0) sh.top[wave] = wave_top;
        __syncthreads();                                           // (also: the histograms are clear)
#pragma unroll
        for (int w = 0; w < NW; ++w) row_top = sh.top[w] > row_top ? sh.top[w] : row_top;
        row_top = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_top);
    }
    uint32_t *mask_out = a.kept_mask ? a.kept_mask + (int64_t)r * a.blocks_per_row * (SEL_BLOCK / 32) : nullptr;
    const int mask_words = a.blocks_per_row * (SEL_BLOCK / 32);
    if (row_top == 0u || row_top >= 0x7f800000u) {             // an invalid entry, or no mass at all
        if (tid == 0) {
            a.counts[r] = 0;
            if (a.thresholds) a.thresholds[r] = 0.0f;
            if (a.row_flags) a.row_flags[r] = SPECATTN_ROW_INVALID;
        }
        if (a.block_counts)
            for (int k = tid; k < a.blocks_per_row; k += THREADS) a.block_counts[(int64_t)r * a.blocks_per_row + k] = 0;
        if (mask_out)
            for (int k = tid; k < mask_words; k += THREADS) mask_out[k] = 0u;
        return;
    }
    auto for_entries = [&](auto &&fn) {
        int items = n_items;
        asm volatile("" : "+s"(items));                        // (compared anew in every pass: the outcomes are not held through the kernel)
#pragma unroll
        for (int i = 0; i < NV4; ++i)
            if (i < items) { fn(data[i].x); fn(data[i].y); fn(data[i].z); fn(data[i].w); }
    };
    // Flat rows: entries that meet in one counter are added to it one after the other, 7.6 cycles each.  Where all that a wave has to add
    // goes into one bin (from `from`, `width` bit patterns), it adds them up by itself.  Added one by one / by the wave, us: equal entries,
    // 520 x 65536 600 / 143, 8 x 34000 108 / 30, 520 x 8000 75 / 21, 8 x 4000 16.5 / 8.4; one bin of three values, 520 x 65536 528 / 225.
    // (Shorter rows have few entries to a counter, and the test for it costs them up to 0.2 us.)
    auto add_together = [&](unsigned long long *counter, uint32_t from, uint32_t width) {
        unsigned c = 0;
        uint32_t sum = 0u;                                     // of distances below 2^23, 64 at most
        for_entries([&](uint32_t x) {
            const uint32_t y = x - from;
            c += y < width ? 1u : 0u;
            sum += y < width ? y : 0u;
        });
        double all = (double)sum;
        wave_prefix(all, c);
        if (lane == 63) atomicAdd(counter, (unsigned long long)c << CNT_SHIFT | ((unsigned long long)all + (unsigned long long)c * (from & 0x7fffffu)));
    };

    Place at;
    if (brief) {
        at = locate_brief<NW>(entries, v0, v1, len, reinterpret_cast<double *>(entries + BRIEF_SUMS / 4), a.top_p);
    } else {
        // ---- first pass: 64 bins per octave from exponent field e_low up ----------------------------------------------
        const int e_top = (int)(row_top >> 23), e_low = (e_top > FINE_OCTAVES ? e_top : FINE_OCTAVES) - (FINE_OCTAVES - 1);      // (>= 1)
        {
            unsigned long long *base = hist1 - (e_low << (23 - FINE_SHIFT));
            const uint32_t least_in = (uint32_t)e_low << 23;
            // What is below the window counts in the row's sum, zeros not at all.  (With a bin per octave for it in this pass, which every
            // other lane of a wide row then hit at the same time, and a test for zeros per entry, us: logits of ten times the usual
            // spread, 200 x 16000 10.9 / 9.7, 8 x 12000 9.3 / 8.6, 200 x 8000 7.9 / 7.5, and the same when nothing is below.)
            double low = 0.0;
            const uint32_t top_bin = wave_top >> FINE_SHIFT;
            bool flat = FLAT && wave_least >> FINE_SHIFT == top_bin;               // (uniform over the wave, like what follows)
            if (FLAT && !flat && wave_top >= least_in && __all(data[0].x < least_in || data[0].x >> FINE_SHIFT == top_bin)) {
                bool one = true;
                for_entries([&](uint32_t x) { one = one && (x < least_in || x >> FINE_SHIFT == top_bin); });
                flat = __all(one);
            }
            if (flat) {
                if (wave_top >= least_in) add_together(base + top_bin, top_bin << FINE_SHIFT, 1u << FINE_SHIFT);
                if (wave_least < least_in) for_entries([&](uint32_t x) { low += (double)__uint_as_float(x < least_in ? x : 0u); });
            } else if (wave_least >= least_in) {                   // no zeros, nothing below the window
                for_entries([&](uint32_t x) { atomicAdd(base + (x >> FINE_SHIFT), fraction_entry(x)); });
            } else {
                for_entries([&](uint32_t x) {
                    low += (double)__uint_as_float(x < least_in ? x : 0u);
                    if (x >= least_in) atomicAdd(base + (x >> FINE_SHIFT), fraction_entry(x));
                });
            }
            if (__any(low > 0.0)) { unsigned none = 0; wave_prefix(low, none); }
            if (lane == 63) sh.low[wave] = low;
        }
        __syncthreads();
        if (wave == 0) locate_first<NW, PAIRED>(hist1, e_low, a.top_p, sh);
        __syncthreads();
        if (sh.below) {                                            // (uniform) rare
            for_entries([&](uint32_t x) { if (x && (int)(x >> 23) < e_low) atomicAdd(hist2 + (x >> 23), fraction_entry(x)); });
            __syncthreads();
            if (wave == 0) locate_below(hist2, a.top_p, sh);
            __syncthreads();
            clear_hist<THREADS, OCTAVES>(hist2);
            __syncthreads();
        }
        // ---- later passes, ten bits each, inside the boundary bin (zeros left out), until it holds a single entry or value ---
        at = sh.place;
        {
            unsigned long long *cur = hist2, *used = hist1;
            while (at.bits > 0 && (at.packed >> CNT_SHIFT) != 1) { // (uniform)
                const int shift = at.bits > DIGIT ? at.bits - DIGIT : 0;
                const uint32_t first = at.lo ? at.lo : 1u, width = (1u << at.bits) - (first - at.lo);
                const bool listed = LISTS && at.bits <= FINE_SHIFT && (at.packed >> CNT_SHIFT) <= LISTED;              // (uniform)
                if (!listed) clear_hist<THREADS, DIGIT_BINS>(used);                  // (read out; the next pass takes it)
                uint32_t fraction = 0x7fffffu;
                asm volatile("" : "+s"(fraction));                 // (keeps 64 masked entries from being computed ahead of the loop)
                auto add = [&](uint32_t y) {                       // y: distance from `first`
                    const uint32_t z = y + (first - at.lo);
                    if (listed) sh.list.entry[atomicAdd(&sh.list.n, 1)] = (int)z;
                    else atomicAdd(&cur[z >> shift], CNT_ONE | ((at.lo + z) & fraction));
                };
                // A bin of few entries: no thread is likely to hold more than two of them, and those are its smallest distances, three
                // instructions per entry and no branch (compared one by one, 64 entries took 3.1 us of 1024 rows' 24 per pair, now 1.9).
                uint32_t y1 = 0xffffffffu, y2 = 0xffffffffu, y3 = 0xffffffffu;       // the three smallest, in order
                bool one_by_one = (at.packed >> CNT_SHIFT) > THREADS / 2;            // (uniform)
                if (!one_by_one) {
                    for_entries([&](uint32_t x) {
                        const uint32_t y = x - first;
                        y3 = median(y2, y3, y);
                        y2 = median(y1, y2, y);
                        y1 = y < y1 ? y : y1;
                    });
                    one_by_one = __any(y3 < width);                // (uniform over the wave)
                    if (!one_by_one) {
                        if (y1 < width) add(y1);
                        if (y2 < width) add(y2);
                    }
                }
                if (FLAT && one_by_one && (at.packed >> CNT_SHIFT) >= 2 * THREADS) {              // (uniform) flat rows, as above
                    uint32_t least = 0xffffffffu, most = 0u;
                    for_entries([&](uint32_t x) {
                        const uint32_t y = x - first;
                        least = y < least ? y : least;
                        most = y < width && y > most ? y : most;
                    });
                    least = ~wave_max(~least);
                    most = wave_max(most);
                    const uint32_t z = least + (first - at.lo), bin = z >> shift;
                    if (least >= width) one_by_one = false;    // (none here)
                    else if (bin == (most + (first - at.lo)) >> shift) {
                        const uint32_t from = at.lo + (bin << shift), skip = from ? 0u : 1u;
                        add_together(&cur[bin], from + skip, (1u << shift) - skip);
                        one_by_one = false;
                    }
                }
                if (one_by_one)
                    for_entries([&](uint32_t x) { if (x - first < width) add(x - first); });
                __syncthreads();
                if (listed) {
                    locate_listed<NW>(sh.list, a.top_p, at);
                    break;
                }
                if (wave == 0) {
                    locate_next<PAIRED>(cur, shift, a.top_p, at);
                    if (lane == 0) sh.place = at;
                }
                __syncthreads();
                at = sh.place;
                unsigned long long *const swap = cur;
                cur = used;
                used = swap;
            }
        }
    }
    // A boundary bin that holds a single entry pins tau*: the bin's fraction sum is that entry's fraction.
    const uint32_t tau_bits = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(at.bits > 0 ? (at.lo & 0x7f800000u) | ((uint32_t)at.packed & 0x7fffffu) : at.lo));           // >= 1: zeros never enter a bin
    const unsigned kept = at.c_above + (unsigned)(at.packed >> CNT_SHIFT);

    if (tid == 0) {
        a.counts[r] = (int32_t)kept;
        if (a.thresholds) a.thresholds[r] = __uint_as_float(tau_bits);
        if (a.row_flags) {
            const double m_incl = at.m_above + fraction_mass(at.packed, (int)(at.lo >> 23));
            const double band = 1e-6 * (at.target / (double)a.top_p);
            uint32_t f = 0;
            if (fabs(m_incl - at.target) <= band || fabs(at.m_above - at.target) <= band) f |= SPECATTN_ROW_NEAR_BOUNDARY;
            if (a.indices && kept > (unsigned)a.idx_capacity) f |= SPECATTN_ROW_OVERFLOW;
            a.row_flags[r] = f;
        }
    }
    if (!a.indices && !a.block_counts && !a.kept_mask) return;

    // ---- ordered compaction: {j : a_j >= tau*}, ascending (Algorithm 2, last step) -------------
    int32_t *out = a.indices ? a.indices + (int64_t)r * a.idx_stride : nullptr;
    const int32_t *ptab = (a.emit_physical && a.page_table) ? a.page_table + (int64_t)b * a.max_pages : nullptr;
    // The list is put together in LDS, in list order, and goes out with contiguous stores over the whole workgroup: whole cache
    // lines, whatever the kept counts of the single waves are.  Lists longer than the buffer take several rounds.
    constexpr unsigned CH = select_lds(THREADS, NV4) / 2;
    static_assert(ITEM * NV4 <= 65536 && CH % 4 == 0, "positions of 16 bits, copied out by fours");
    uint16_t *stage = reinterpret_cast<uint16_t *>(select_dyn);
    const unsigned cap = kept < (unsigned)a.idx_capacity ? kept : (unsigned)a.idx_capacity;
    const bool one_round = kept <= CH;                         // (uniform) every rank of the row fits the buffer, also those beyond a smaller capacity
    typedef int32_t i32x4a __attribute__((ext_vector_type(4), aligned(4)));        // (a list starts anywhere)
    auto place = [&](int32_t val) { return ptab ? (ptab[val >> a.page_shift] << a.page_shift) | (val & ((1 << a.page_shift) - 1)) : val; };
    auto copy_out = [&](unsigned c0) {
        __syncthreads();
        const unsigned nround = (cap - c0) < CH ? (cap - c0) : CH;
        // Streaming stores: a list is read by later launches on any XCD, and what waits in an L2 as changed lines is written back at the
        // launch's end (without / with, us: verify step of 16 layers 811.5 / 796.2, 512 ragged rows of up to 65536 609 / 598, 2048 x
        // 16384 42.2 / 39.7, 64 rows of 13001 with attention 46.1 / 45.8; mask words that way: a union of 1024 members 180.9 / 181.6).
        if constexpr (WORDS) {
            for (unsigned k = tid * 4; k < nround; k += ITEM) {
                const ushort4 v = *reinterpret_cast<const ushort4 *>(stage + k);   // (reaches past the list, not past the buffer)
                if (k + 4 <= nround) {
                    __builtin_nontemporal_store((i32x4a){place(v.x), place(v.y), place(v.z), place(v.w)}, reinterpret_cast<i32x4a *>(out + c0 + k));
                } else {
                    out[c0 + k] = place(v.x);
                    if (k + 1 < nround) out[c0 + k + 1] = place(v.y);
                    if (k + 2 < nround) out[c0 + k + 2] = place(v.z);
                }
            }
        } else {                                               // (short lists: by fours 8 rows of 1024 take 0.1 us longer)
            for (unsigned k = tid; k < nround; k += THREADS) __builtin_nontemporal_store(place(stage[k]), out + c0 + k);
        }
    };
    // Every position (flat rows, top_p = 1), where lists may take several rounds.  By rounds / like this, us: equal entries, 8 x 34816 30 / 16.8;
    // top_p = 1, 64 x 32768 21.1 / 13.9, 1000 x 32768 69 / 45.
    if (ITEM * NV4 > (int)CH && kept == (unsigned)len && out && !a.block_counts && !mask_out) {              // (uniform)
        for (unsigned k = tid * 4; k < cap; k += ITEM) {
            if (k + 4 <= cap) {
                __builtin_nontemporal_store((i32x4a){place(k), place(k + 1), place(k + 2), place(k + 3)}, reinterpret_cast<i32x4a *>(out + k));
            } else {
                for (unsigned j = k; j < cap; ++j) out[j] = place(j);
            }
        }
        return;
    }
    if constexpr (WORDS) {
        // Long rows: one bit per entry, two instructions each, then the eight lanes that hold 32 consecutive positions of eight items
        // exchange their nibbles, so that every lane holds whole words of the row's kept bits; what follows (counts, prefix,
        // emission bit by bit) is work per word or per kept entry instead of per entry.
        constexpr int GROUPS = NV4 / 8;
        constexpr int WORDS_PER_ITEM = ITEM / 32;
        uint32_t word[GROUPS];
        int at_word[GROUPS];
#pragma unroll
        for (int gr = 0; gr < GROUPS; ++gr) {
            uint32_t x = 0u;
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                const uint4 u = data[gr * 8 + i];
                x = x + x + (u.w >= tau_bits ? 1u : 0u);
                x = x + x + (u.z >= tau_bits ? 1u : 0u);
                x = x + x + (u.y >= tau_bits ? 1u : 0u);
                x = x + x + (u.x >= tau_bits ? 1u : 0u);
            }
            word[gr] = transpose_nibbles(x, lane);             // of item gr * 8 + lane % 8
            at_word[gr] = (gr * 8 + (lane & 7)) * WORDS_PER_ITEM + wave * 8 + (lane >> 3);
            table[at_word[gr]] = __popc(word[gr]);
            if (mask_out && at_word[gr] < mask_words) mask_out[at_word[gr]] = word[gr];
        }
        if (mask_out)                                          // words past the last item
            for (int k = NV4 * WORDS_PER_ITEM + tid; k < mask_words; k += THREADS) mask_out[k] = 0u;
        if (!out && !a.block_counts) return;
        __syncthreads();
        unsigned c[GROUPS], sum = 0;
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) { c[k] = table[tid * GROUPS + k]; sum += c[k]; }
        const unsigned inc = (unsigned)wave_inclusive_sum((int)sum);
        if (lane == 63) sh.wave_sum[wave] = inc;
        __syncthreads();
        unsigned base = inc - sum;
#pragma unroll
        for (int w = 0; w < NW; ++w) base += w < wave ? sh.wave_sum[w] : 0u;
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) { table[tid * GROUPS + k] = base; base += c[k]; }
        if (tid == THREADS - 1) table[TABLE] = base;
        __syncthreads();
        if (a.block_counts)
            for (int k = tid; k < a.blocks_per_row; k += THREADS) {
                constexpr int WPB = SEL_BLOCK / 32;
                a.block_counts[(int64_t)r * a.blocks_per_row + k] = k * WPB < TABLE ? (int32_t)(table[(k + 1) * WPB] - table[k * WPB]) : 0;
            }
        if (!out) return;
        for (unsigned c0 = 0; c0 < cap; c0 += CH) {
            if (c0) __syncthreads();                           // the round before has been read out
#pragma unroll
            for (int gr = 0; gr < GROUPS; ++gr) {
                uint32_t left = word[gr];
                unsigned rank = table[at_word[gr]] - c0;       // (wraps around below c0)
                const int p = at_word[gr] * 32;
                if (one_round) {
                    for (; left; left &= left - 1, ++rank) stage[rank] = (uint16_t)(p + __ffs((int)left) - 1);
                } else if (rank < CH || rank + 32u < CH + 32u) {
                    for (; left; left &= left - 1, ++rank)
                        if (rank < CH) stage[rank] = (uint16_t)(p + __ffs((int)left) - 1);
                }
            }
            copy_out(c0);
        }
    } else {
        // Short rows: item by item.  First only counts: every wave's kept entries per item (the compares are cheaper to repeat than to
        // store), then every wave adds the (item, wave) counts up by itself, which gives it its place in the list.
        static_assert(NV4 * NW <= 64, "a wave adds the counts up");
        unsigned my_tot = 0;                                   // lane i: this wave's kept entries of item i
        auto keep = [&](const uint4 &u, bool (&f)[4]) {
            f[0] = u.x >= tau_bits; f[1] = u.y >= tau_bits; f[2] = u.z >= tau_bits; f[3] = u.w >= tau_bits;
        };
#pragma unroll
        for (int i = 0; i < NV4; ++i) {
            bool f[4];
            keep(data[i], f);
            const unsigned wtot = __popcll(__ballot(f[0])) + __popcll(__ballot(f[1])) + __popcll(__ballot(f[2])) + __popcll(__ballot(f[3]));
            if (lane == i) my_tot = wtot;
            if (mask_out) {                                    // word (i * THREADS + tid) / 8 covers this thread's four positions
                const uint32_t word = mask_word((f[0] ? 1u : 0u) | (f[1] ? 2u : 0u) | (f[2] ? 4u : 0u) | (f[3] ? 8u : 0u), lane);
                const int w = (i * THREADS + tid) >> 3;
                if ((lane & 7) == 0 && w < mask_words) mask_out[w] = word;
            }
        }
        if (mask_out)                                          // words past the last item
            for (int k = NV4 * (ITEM / 32) + tid; k < mask_words; k += THREADS) mask_out[k] = 0u;
        if (lane < NV4) table[lane * NW + wave] = my_tot;
        __syncthreads();
        if (a.block_counts) {
            constexpr int BPI = ITEM / SEL_BLOCK;              // selection blocks per item
            constexpr int WPB = NW / BPI;                      // waves per block
            for (int blk = tid; blk < a.blocks_per_row; blk += THREADS) {
                unsigned c = 0;
                if (blk < NV4 * BPI)
                    for (int w = 0; w < WPB; ++w) c += table[(blk / BPI) * NW + (blk % BPI) * WPB + w];
                a.block_counts[(int64_t)r * a.blocks_per_row + blk] = (int32_t)c;
            }
        }
        if (!out) return;
        const unsigned v = lane < NV4 * NW ? table[lane] : 0u, excl = (unsigned)wave_inclusive_sum((int)v) - v;
        for (unsigned c0 = 0; c0 < cap; c0 += CH) {
            if (c0) __syncthreads();                           // the round before has been read out
#pragma unroll
            for (int i = 0; i < NV4; ++i) {
                bool f[4];
                keep(data[i], f);
                const unsigned long long m0 = __ballot(f[0]), m1 = __ballot(f[1]), m2 = __ballot(f[2]), m3 = __ballot(f[3]);
                const unsigned before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m3 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m3,
                                        __builtin_amdgcn_mbcnt_hi((uint32_t)(m2 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m2,
                                        __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m1,
                                        __builtin_amdgcn_mbcnt_hi((uint32_t)(m0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m0, 0u))))))));
                unsigned o = (unsigned)__builtin_amdgcn_readlane((int)excl, i * NW + __builtin_amdgcn_readfirstlane(wave)) - c0 + before;      // (wraps around below c0)
                const int p = (i * THREADS + tid) * 4;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (f[k] && (one_round || o < CH)) stage[o] = (uint16_t)(p + k);
                    o += f[k] ? 1u : 0u;
                }
            }
            copy_out(c0);
        }
    }
}
