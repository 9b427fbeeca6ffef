// Fused decode attention over compressed keys (Alg. 2, Eq. (score-exact)): query rotation,
// split-K main kernels, split merge.
#ifndef OCTOPUS_DECODE_HPP_
#define OCTOPUS_DECODE_HPP_

#include <cstddef>

#include "octopus_device.hpp"

namespace octopus {

constexpr float kLog2e = 1.4426950408889634f;

// 2^x as the bare v_exp_f32 (about one ulp; results below 2^-126 become zero, which is all a softmax
// weight that small is worth).  exp2f() wraps the same instruction in a range fix-up for denormal
// results that costs five more instructions per value.
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr int kDecodeWaves = 4;  // wavefronts per workgroup of the main kernels
constexpr int kStreamPolicy = 2; // cache policy of the buffer loads of streamed data: non-temporal

// ---- D1-D7: split-K main kernels --------------------------------------------------------------
// Work unit = one wavefront over a range of steps of one (sequence, KV head, row group): the wave walks
// its 64-token tiles with one key per lane (two tiles per step up to d = 128) and keeps its own running
// (m, l, acc); the waves of a workgroup share the LDS tables and merge their results at the end of a segment.
// How the work is cut into segments is described below.
//
// Per tile: the lane loads its record (16 bytes at a time, coalesced thanks to the tile-interleaved
// layout, one tile ahead of use), unpacks the code fields with compile-time shifts, looks up the
// direction (and the norm centroids, a group of codes at a time) in LDS tables and accumulates the RG
// scores against the wave-uniform rotated queries, which arrive through scalar loads.  The tables
// are replicated so that neighbouring lanes always read different LDS banks whatever their codes.
// Two kernels differ in P.V only: decode_kernel_mfma (bf16 values) feeds the probabilities to the
// matrix cores; decode_kernel_valu (fp32 values) multiplies on the vector ALUs.

// Replication of a table of `bytes` bytes: up to 8 copies within a 64 KB budget (one workgroup runs
// per compute unit and may use most of its 160 KB of LDS).
constexpr int table_rep(int bytes) {
    return bytes * 8 <= 65536 ? 8 : (bytes * 4 <= 65536 ? 4 : (bytes * 2 <= 65536 ? 2 : 1));
}

template <int BD>
struct DirTable {
    static constexpr int ENTRIES = 1 << (2 * BD);
    static constexpr int REP = table_rep(ENTRIES * 16);
    static constexpr int FLOAT4S = ENTRIES * REP;
};

// Entry e of copy r sits at float4 index e * REP + r: lanes l and l' with l % REP != l' % REP never
// share a bank, whatever e.
template <int BD>
__device__ __forceinline__ void build_dir_table(float4 *table, const float *c_xi, int tid, int nthreads) {
    using T = DirTable<BD>;
    constexpr int K = 1 << BD;
    for (int e = tid; e < T::FLOAT4S; e += nthreads) {
        const int code = e / T::REP;
        table[e] = oct_decode(c_xi[code & (K - 1)], c_xi[code >> BD]);
    }
}

// Norm codes are looked up a group at a time: NTG consecutive BN-bit indices form one table index and
// the entry holds their NTG centroids (4 one-bit codes, or 2 two- or three-bit codes, per lookup).
template <int BN>
struct RhoTable {
    static constexpr int NTG = BN == 1 ? 4 : (BN <= 3 ? 2 : 1);   // (4 bits and more: one code per lookup)
    static constexpr int BITS = BN * NTG;
    static constexpr int ENTRIES = 1 << BITS;
    static constexpr int REP = 32 / NTG;   // 8 x 16 bytes, 16 x 8 bytes or 32 x 4 bytes = all 32 banks
    static constexpr int FLOATS = ENTRIES * REP * NTG;
};

template <int BN>
__device__ __forceinline__ void build_rho_table(float *table, const float *c_rho, int tid, int nthreads) {
    using T = RhoTable<BN>;
    for (int e = tid; e < T::FLOATS; e += nthreads) {
        const int t = e % T::NTG, entry = e / (T::NTG * T::REP);
        table[e] = c_rho[(entry >> (BN * t)) & ((1 << BN) - 1)];
    }
}

// Where the direction and norm codes of a triplet together have at most 10 bits (every plan up to 3 bits
// per coordinate), one table indexed by (norm code, xi code, eta code) holds the products
// rho^ * n^ themselves: one lookup per triplet, no multiply.  Otherwise (5 + 5 + 3 bits) directions and
// norm centroids come from the two tables above.
constexpr bool joint_codes(int bd, int bn) { return 2 * bd + bn <= 10; }

// Layout [direction code][norm code][copy]: the byte offset of the entry lane l reads is
//   (direction code << CS) | (norm code << NS) | ((l % REP) << 4),
// the copies making neighbouring lanes hit different banks.  For 4 + 4 + 2 bits with 4 copies CS is 8
// and the direction code is a whole byte of the record: one byte permute puts it in place together with
// the lane part, a bit-field extract and a shift-or add the norm code -- three instructions per triplet.
template <int BD, int BN>
struct JointTable {
    static constexpr int BITS = 2 * BD + BN;
    static constexpr int ENTRIES = 1 << BITS;
    static constexpr int REP = table_rep(ENTRIES * 16);
    static constexpr int LOG_REP = REP == 8 ? 3 : (REP == 4 ? 2 : (REP == 2 ? 1 : 0));
    static constexpr int NS = 4 + LOG_REP;
    static constexpr int CS = NS + BN;
    static constexpr int FLOAT4S = ENTRIES * REP;
    static constexpr bool BYTE_CODES = (2 * BD == 8) && (CS == 8);
};

template <int BD, int BN>
__device__ __forceinline__ void build_joint_table(float4 *table, const float *c_xi, const float *c_rho, int tid,
                                                  int nthreads) {
    using T = JointTable<BD, BN>;
    constexpr int K = 1 << BD;
    for (int e = tid; e < T::ENTRIES; e += nthreads) {
        const int dir = e >> BN, nrm = e & ((1 << BN) - 1);
        const float4 n = oct_decode(c_xi[dir & (K - 1)], c_xi[dir >> BD]);
        const float rho = c_rho[nrm];
        const float4 val = make_float4(rho * n.x, rho * n.y, rho * n.z, 0.0f);
#pragma unroll
        for (int r = 0; r < T::REP; ++r) table[e * T::REP + r] = val;
    }
}

// ---- operands of the matrix-core score pass --------------------------------------------------------
// fp32 -> two bf16 numbers whose sum represents it to about 2^-17 (round to nearest even both times; the
// difference x - hi is exact in fp32).
__device__ __forceinline__ uint32_t bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
// (x, y, z) -> 16 bytes: bf16 hi of (x, y, z, 0), then bf16 lo of (x, y, z, 0): the k = 4 operand of
// v_mfma_f32_4x4x4_16b_bf16, once for the leading parts and once for the remainders.
__device__ __forceinline__ uint4 split_triplet(float x, float y, float z) {
    const uint32_t hx = bf16_rne(x), hy = bf16_rne(y), hz = bf16_rne(z);
    const uint32_t lx = bf16_rne(x - __uint_as_float(hx << 16)), ly = bf16_rne(y - __uint_as_float(hy << 16)),
                   lz = bf16_rne(z - __uint_as_float(hz << 16));
    return make_uint4(hx | (hy << 16), hz, lx | (ly << 16), lz);
}

// The joint table of a class with its entries in that form (same size and addressing as the fp32 table).  A thread takes
// a direction with all its norm codes (or, with fewer directions than threads, a share of them).  Neighbouring threads
// start with different norm codes and copies, so that the 16-byte writes of a wavefront spread over all banks (the entries
// of neighbouring directions lie 256 bytes apart).
template <int BD, int BN>
__device__ __forceinline__ void build_joint_table_mx(float4 *table, const float *c_xi, const float *c_rho, int tid,
                                                     int nthreads) {
    using T = JointTable<BD, BN>;
    constexpr int K = 1 << BD, M = 1 << BN;
    uint4 *out = reinterpret_cast<uint4 *>(table);
    const int per = nthreads / (K * K) > 1 ? (nthreads / (K * K) < M ? nthreads / (K * K) : M) : 1;   // threads per direction
    const int part = tid % per;
#pragma unroll 1
    for (int dir = tid / per; dir < K * K; dir += nthreads / per) {
        const float4 n = oct_decode(c_xi[dir & (K - 1)], c_xi[dir >> BD]);
#pragma unroll 1
        for (int q = part; q < M; q += per) {
            const int nrm = (q + dir / T::REP) & (M - 1);
            const float rho = c_rho[nrm];
            const uint4 val = split_triplet(rho * n.x, rho * n.y, rho * n.z);
#pragma unroll
            for (int r = 0; r < T::REP; ++r) out[(dir * M + nrm) * T::REP + ((r + dir) & (T::REP - 1))] = val;
        }
    }
}

template <int BD, int BN>
constexpr int dir_table_float4s() {
    return joint_codes(BD, BN) ? JointTable<BD, BN>::FLOAT4S : DirTable<BD>::FLOAT4S;
}

template <class P>
struct DecodeTables {
    static constexpr bool J0 = joint_codes(P::BD0, P::BN0);
    static constexpr bool J1 = P::NCLASS == 2 && joint_codes(P::BD1, P::BN1);
    float4 dir0[dir_table_float4s<P::BD0, P::BN0>()];
    float4 dir1[P::NCLASS == 2 ? dir_table_float4s<(P::BD1 > 0 ? P::BD1 : 1), (P::BN1 > 0 ? P::BN1 : 1)>() : 1];
    __attribute__((aligned(16))) float rho0[J0 ? 4 : RhoTable<P::BN0>::FLOATS];
    __attribute__((aligned(16))) float rho1[P::NCLASS == 2 && !J1 ? RhoTable<(P::BN1 > 0 ? P::BN1 : 1)>::FLOATS : 4];
    float c_xi[2][1 << (P::BD0 > P::BD1 ? P::BD0 : P::BD1)];
    float c_rho[2][P::BN0 > 1 || P::BN1 > 1 ? 1 << (P::BN0 > P::BN1 ? P::BN0 : P::BN1) : 2];
};

// Plans whose every class has a joint table (all up to 3 bits per coordinate) can score on the matrix cores.
template <class P>
constexpr bool mx_scores() { return DecodeTables<P>::J0 && (P::NCLASS == 1 || DecodeTables<P>::J1); }

// Centroids of the levels that plan P has, from the kernel's first argument (a DeviceBooks) to LDS: one level per lane,
// requested at the kernel's start and stored when the tables are built.  (Reading them one by one with compile-time indices
// took sixty instructions; straight-line code that runs once costs the fetch of its instructions, which in a kernel this
// size is more than their execution.)
template <class P>
struct BookLevels {
    static constexpr int NX = sizeof(DecodeTables<P>::c_xi[0]) / 4, NR = sizeof(DecodeTables<P>::c_rho[0]) / 4;
    static_assert(NX <= kWave && NR <= kWave, "a level per lane");
    float xi[P::NCLASS], rho[P::NCLASS];
    __device__ __forceinline__ void load(int lane) {
        typedef const float __attribute__((address_space(4))) *arg_t;
        arg_t arg = (arg_t)__builtin_amdgcn_kernarg_segment_ptr();
#pragma unroll
        for (int c = 0; c < P::NCLASS; ++c) {   // (kMaxLevels levels each: every lane reads one)
            xi[c] = arg[offsetof(DeviceBooks, c_xi) / 4 + c * kMaxLevels + lane];
            rho[c] = arg[offsetof(DeviceBooks, c_rho) / 4 + c * kMaxLevels + lane];
        }
    }
    __device__ __forceinline__ void store(DecodeTables<P> &tb, int tid) const {
#pragma unroll
        for (int c = 0; c < P::NCLASS; ++c) {
            if (tid < NX) tb.c_xi[c][tid] = xi[c];
            if (tid < NR) tb.c_rho[c][tid] = rho[c];
        }
    }
};

// MX: joint tables hold bf16 hi / lo operands (the matrix-core score pass) instead of fp32 vectors.
template <class P, bool MX = false>
__device__ __forceinline__ void build_tables(DecodeTables<P> &tb, int tid, int nthreads) {
    __syncthreads();   // (the levels are in place)
    if constexpr (MX) {
        static_assert(mx_scores<P>(), "matrix-core scores need joint tables");
        build_joint_table_mx<P::BD0, P::BN0>(tb.dir0, tb.c_xi[0], tb.c_rho[0], tid, nthreads);
        if constexpr (P::NCLASS == 2) build_joint_table_mx<P::BD1, P::BN1>(tb.dir1, tb.c_xi[1], tb.c_rho[1], tid, nthreads);
        __syncthreads();
        return;
    }
    if constexpr (DecodeTables<P>::J0) {
        build_joint_table<P::BD0, P::BN0>(tb.dir0, tb.c_xi[0], tb.c_rho[0], tid, nthreads);
    } else {
        build_dir_table<P::BD0>(tb.dir0, tb.c_xi[0], tid, nthreads);
        build_rho_table<P::BN0>(tb.rho0, tb.c_rho[0], tid, nthreads);
    }
    if constexpr (P::NCLASS == 2) {
        if constexpr (DecodeTables<P>::J1) {
            build_joint_table<P::BD1, P::BN1>(tb.dir1, tb.c_xi[1], tb.c_rho[1], tid, nthreads);
        } else {
            build_dir_table<P::BD1>(tb.dir1, tb.c_xi[1], tid, nthreads);
            build_rho_table<P::BN1>(tb.rho1, tb.c_rho[1], tid, nthreads);
        }
    }
    __syncthreads();
}

// Work distribution of the split-K kernels.  The steps of the call (a step = tiles_per_step 64-token tiles) lie in a row:
// sequences in order, the (KV head, row group) pairs of a sequence in order, the steps of a pair in order.  The row is
// divided evenly over the workgroups (one per compute unit), and a workgroup walks its share as one SEGMENT per pair that it
// touches: all its wavefronts together, interleaved (step_begin, step_begin + item_waves, ...), so that the workgroup streams
// through memory front to back.  At the end of a segment the wavefronts' partial results are merged in LDS and one partial per
// query row goes to memory, at slot (workgroup + pair), which no two segments share.  Every workgroup computes its
// share from the sequence lengths by itself (one load and a scan of 64 lanes): nothing is planned by an earlier kernel and
// nothing is handed out at run time.
// This took the place of up to 2048 items cut by an earlier kernel and taken from a counter, four partials each: on a ragged
// batch an item was three steps, its start-up several times their work.  Calls with and without (rotation in the kernel and
// merge in LDS included): 24 sequences of 125 - 8000 tokens, 8 KV heads of 8 query rows, d = 128, paged, with a window:
// 194 -> 146 us; 32 sequences of 1 k - 64 k, d = 256: 877 -> 830 us; one head, 4096 tokens, fp32: 28.6 -> 21.3 us;
// equal lengths (16 x 32768): 213.4 -> 211.7 us.
// A segment has a fixed cost (queries rotated, operands built, first loads, merge, four barriers) of the order of a round of
// steps, which an even division does not see.  It serves calls of fewer pairs than workgroups, of much the same length and with
// steps enough for all;
//   * where there are no more BLOCKS of item_waves steps (the last one of a pair may have fewer) than workgroups, a block is
//     a workgroup's: one step per wavefront and one segment per workgroup, whatever the lengths;
//   * where there are as many pairs as workgroups or more, or some are short beside the others (short_pairs), every pair counts
//     kSegmentTiles more than its whole blocks, and only whole blocks are handed out.  Divided evenly, the pairs of a few short
//     sequences are one workgroup's segments: of 24 ragged sequences to 8000 tokens the worst has ten, of which each costs as much
//     as a round of steps.
// Fewer pairs than workgroups, ragged (1 / 64 of the longest and up), d = 128, b = 3, evenly / weighed: 24 sequences to 8000, 8 KV
// heads of eight rows 104 / 56.5 us (over quantised values, four rows 95 / 50; fp32 values 174 / 116), 100 to 5000, 2 KV heads
// 62 / 41, 16 to 30000, 4 KV heads 67 / 59.5, one of 60000 and eight of 300 58 / 39; 16 of half to full 12000 equal.  Pairs of equal
// length stay evenly divided: weighed, 24 x 1024 28 / 24 but 28 x 1100 28.3 / 29.5, 16 x 1500 20.7 / 22, 24 x 4096 52 / 53; so do
// pairs longer than a share, and calls of shares under three rounds, which whole blocks round up too much (evenly / weighed, 8 sequences
// to 1326, 24 KV heads, d = 64 18.8 / 20.5).  24 x 512 with blocks counted exactly: 26.4 / 19.3.
// decode_kernel_valu, whose steps are one tile, goes by blocks of two rounds (each one segment) where its even shares are between
// one round and two, or else a share that straddles two pairs costs a second segment.  Evenly / by blocks, 8 KV heads over fp32 values at
// d = 128: 2 sequences to 8179, eight rows 50.3 / 41.5 us, four 35.7 / 31.4, one 25.5 / 25.7; five to 4000, four rows 39.0 / 30.8; 20
// to 5000, 2 KV heads 36.4 / 30.4; eight rows over quantised values, 2 to 8179 48.6 / 40.3.  Equal pairs, a power of two of them, whose
// even shares end where the pairs do, stay even (2 x 6000, eight rows 38.8 / 40.6, one row 23.3 / 24.5).
// Calls with every length divided evenly / as here, d = 128, b = 3, ragged (lengths of 1 / 64 of the longest and up): 32
// sequences to 372 tokens, one KV head of eight rows 43.2 / 17.7 us, 64 to 500, 8 KV heads of four rows 50.5 / 25.8, 256 to 500
// 156 / 84, 256 to 4000 358 / 239, the same over quantised values 371 / 225, 40 to 16000 162 / 135 (kSegmentTiles half or twice
// as many: 239 - 247, 135 - 145; with eight wavefronts 222 - 258).  Where the division stays even, choosing costs 0.1 - 0.2 us, in calls of few steps 0.1 - 0.4.
constexpr int kDecodeWorkgroups = 256;   // one per compute unit
constexpr int kSegmentTiles = 8;         // what a segment's fixed cost is counted for (twice with eight wavefronts)

// (tiles_per_step: 1 or 2)
__device__ __forceinline__ int steps_of(int len, int max_len, int tiles_per_step) {
    const uint32_t l = static_cast<uint32_t>(min(max(len, 0), max_len));
    const uint32_t tiles = (l + kWave - 1) / kWave;
    return static_cast<int>(tiles_per_step == 2 ? (tiles + 1) / 2 : tiles);
}

// Inclusive sum over the wavefront's lanes.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    auto take = [](uint32_t x, auto ctrl, auto rows) __attribute__((always_inline)) {
        return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), decltype(ctrl)::value,
                                                                 decltype(rows)::value, 0xf, false));
    };
    using std::integral_constant;
    v += take(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr:1, 2, 4, 8
    v += take(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    v += take(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1 and 3
    v += take(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2 and 3
    return v;
}

// floor(a / b) of whole numbers below 2^53 with a / b < 2^31: the quotient in double precision is never rounded up to a
// whole number it does not reach (it would have to be within 2^-53 of it, relatively, and is 1 / b away at least).
// (A 64-bit division by integer instructions is over a hundred of them.)
__device__ __forceinline__ uint32_t divide(uint64_t a, uint64_t b) {
    return static_cast<uint32_t>(static_cast<double>(a) / static_cast<double>(b));
}

// How a call's steps are divided: in units, of which a pair has fixed() and then those of its quanta in order; a workgroup
// takes the quanta whose first unit lies in its share.  (Quanta are never further apart than a share is long -- one unit, or
// item_waves units of a total of item_waves kDecodeWorkgroups at least -- so the workgroups that have quanta of a pair are
// consecutive.)  waves_log2, tps: log2 of the wavefronts per workgroup, tiles per step.
struct Division {
    int kind;
    int waves_log2, tps;
    int rounds_log2 = 0;   // kBlockEach: rounds of steps to a block

    // Sequences whose pairs are under three quarters of the mean pair and shorter than an even share, where a share is at least
    // three rounds of steps (st: the steps of this lane's sequence, sum and total: of all sequences and pairs, present: sequences
    // with tokens).
    static __device__ __forceinline__ uint64_t short_pairs(uint32_t st, uint64_t sum, uint64_t total, uint32_t present, int waves_log2) {
        if (total < static_cast<uint64_t>(3 * kDecodeWorkgroups) << waves_log2) return 0u;
        const float share = static_cast<float>(total) * (1.0f / kDecodeWorkgroups), mean = 0.75f * static_cast<float>(sum);
        const float x = static_cast<float>(st);
        return __ballot(st > 0u && x < share && x * static_cast<float>(present) < mean);
    }
    static __device__ __forceinline__ uint32_t with_tokens(uint32_t st) { return __popcll(__ballot(st > 0u)); }
    static __device__ __forceinline__ uint64_t blocks_of(uint32_t st, int log2) {
        return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wave_scan((st + (1u << log2) - 1u) >> log2)), kWave - 1));
    }
    // Most calls are known to be divided evenly by their steps alone (and code that runs costs its fetch here).
    // TWO: shp.two_round_blocks may be set; calls of one to two rounds are then even where the pairs are equal and a power of two.
    template <bool TWO>
    static __device__ __forceinline__ bool surely_even(const DecodeShape &shp, uint32_t st, uint64_t sum, uint64_t total, int waves_log2) {
        if (shp.pairs_fill != 0 || shp.n_seq > kWave || total <= static_cast<uint64_t>(kDecodeWorkgroups) << waves_log2) return false;
        if (TWO && __builtin_expect(shp.two_round_blocks != 0 && total <= static_cast<uint64_t>(2 * kDecodeWorkgroups) << waves_log2, 0)) {
            const uint32_t present = with_tokens(st), pairs = present * static_cast<uint32_t>(shp.n_kv_heads * shp.n_row_groups);
            return (pairs & (pairs - 1u)) == 0u && __ballot(st > 0u && st * present != static_cast<uint32_t>(sum)) == 0u;
        }
        return short_pairs(st, sum, total, with_tokens(st), waves_log2) == 0u;
    }
    // The kind, from the steps of all sequences and pairs; steps_at(s0): the steps of sequence s0 + lane (0: none).
    template <bool TWO, class Steps>
    __device__ __forceinline__ void set(const DecodeShape &shp, uint64_t sum, const Steps &steps_at) {
        const uint64_t G = static_cast<uint64_t>(shp.n_kv_heads) * shp.n_row_groups, total = sum * G;
        constexpr uint64_t kWgs = kDecodeWorkgroups;
        const int two_log2 = waves_log2 + 1;
        if (shp.n_seq == 1) {   // (as below, where a lone sequence is never short; without the scans)
            const uint32_t n = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(steps_at(0))));
            const uint64_t blocks = static_cast<uint64_t>((n + (1u << waves_log2) - 1u) >> waves_log2) * G;
            kind = blocks <= kWgs ? kBlockEach : (G >= kWgs ? kPairsWeighed : kDivideEvenly);
            if (TWO && __builtin_expect(shp.two_round_blocks != 0 && blocks > kWgs, 0) && ((n + (1u << two_log2) - 1u) >> two_log2) * G <= kWgs &&
                (G & (G - 1)) != 0) {
                kind = kBlockEach;
                rounds_log2 = 1;
            }
            return;
        }
        uint32_t present = 0;
        for (int s0 = 0; s0 < shp.n_seq; s0 += kWave) present += with_tokens(steps_at(s0));
        const uint64_t pairs = present * G;
        kind = kBlockEach;
        if (total + (pairs << waves_log2) - pairs <= kWgs << waves_log2) return;   // (blocks have at most a rest per pair more)
        if (total <= kWgs << waves_log2) {   // (else the blocks are more than the workgroups)
            uint64_t blocks = 0;
            for (int s0 = 0; s0 < shp.n_seq; s0 += kWave) blocks += blocks_of(steps_at(s0), waves_log2);
            if (blocks * G <= kWgs) return;
        }
        if (TWO && __builtin_expect(shp.two_round_blocks != 0 && total <= kWgs << two_log2, 0)) {
            uint64_t blocks = 0, unequal = pairs & (pairs - 1);
            for (int s0 = 0; s0 < shp.n_seq; s0 += kWave) {
                const uint32_t st = steps_at(s0);
                blocks += blocks_of(st, two_log2);
                unequal |= __ballot(st > 0u && st * present != static_cast<uint32_t>(sum));   // (sum <= 2048 << 3 here)
            }
            if (blocks * G <= kWgs && unequal != 0u) {
                rounds_log2 = 1;
                return;
            }
        }
        kind = pairs >= kWgs ? kPairsWeighed : kDivideEvenly;
        if (pairs < kWgs)
            for (int s0 = 0; s0 < shp.n_seq; s0 += kWave)
                if (short_pairs(steps_at(s0), sum, total, present, waves_log2) != 0u) kind = kPairsWeighed;
    }
    __device__ __forceinline__ uint32_t fixed() const {
        return kind == kPairsWeighed ? static_cast<uint32_t>((waves_log2 == 3 ? 2 * kSegmentTiles : kSegmentTiles) / tps) : 0u;
    }
    __device__ __forceinline__ int steps_log2() const { return kind == kDivideEvenly ? 0 : (kind == kPairEach ? 30 : waves_log2 + rounds_log2); }   // steps per quantum
    __device__ __forceinline__ int units_log2() const { return kind == kPairsWeighed ? waves_log2 : 0; }   // units per quantum
    __device__ __forceinline__ uint32_t quanta(uint32_t steps) const { return (steps + (1u << steps_log2()) - 1u) >> steps_log2(); }
    __device__ __forceinline__ uint32_t units(uint32_t steps) const {
        return steps > 0u ? fixed() + (quanta(steps) << units_log2()) : 0u;
    }
    // quanta of a pair that begin before its unit x
    __device__ __forceinline__ uint32_t quanta_before(uint32_t x) const {
        return x > fixed() ? (x - fixed() + (1u << units_log2()) - 1u) >> units_log2() : 0u;
    }
    // the share of workgroup b, and the workgroup that has unit x
    __device__ __forceinline__ void share(uint64_t total, int b, uint64_t *pos, uint64_t *end) const {
        if (__builtin_expect(kind == kBlockEach || kind == kPairEach, 0)) {   // (at most as many units as workgroups)
            *pos = min(static_cast<uint32_t>(b), static_cast<uint32_t>(total));
            *end = min(static_cast<uint32_t>(b) + 1u, static_cast<uint32_t>(total));
        } else {
            const uint64_t t = total * static_cast<uint32_t>(b);
            *pos = t / kDecodeWorkgroups;
            *end = (t + total) / kDecodeWorkgroups;
        }
    }
    __device__ __forceinline__ int owner(uint64_t total, uint64_t x) const {
        return kind == kBlockEach ? static_cast<int>(x) : static_cast<int>(divide((x + 1) * kDecodeWorkgroups - 1, total));
    }
};

__device__ __forceinline__ uint32_t last_lane(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), kWave - 1));
}

struct WaveWork {
    int seq, kvh, grp;
    int64_t pair, group_id, slot;
    int step_begin, step_end, step_stride, step_last, len, n_tiles;
};

// The share of one workgroup and where it stands in it.  Sequences are looked at 64 at a time, one per lane.
// TPS, NW: tiles per step and wavefronts per workgroup of the kernel (the shape's tiles_per_step and item_waves).
template <int TPS, int NW, bool FRESH = true>
struct WorkSpan {
    int chunk;               // first sequence of the 64
    int lane_len;            // length of sequence chunk + lane
    uint32_t lane_sum;       // units per pair of sequences chunk .. chunk + lane
    uint64_t before;         // units per pair of the sequences before chunk
    uint64_t pos, end;       // the workgroup's units that are left
    Division div{kDivideEvenly, NW == 8 ? 3 : 2, TPS};

    static_assert(NW == 4 || NW == 8, "waves_log2");
    __device__ __forceinline__ uint32_t read(const DecodeShape &shp, const int32_t *seq_lens, int lane) {
        const int s = chunk + lane;
        const int len = seq_lens[min(s, shp.n_seq - 1)];
        lane_len = s < shp.n_seq ? min(max(len, 0), shp.max_len) : 0;
        return static_cast<uint32_t>(steps_of(lane_len, shp.max_len, TPS));
    }
    __device__ __forceinline__ void look(const DecodeShape &shp, const int32_t *seq_lens, int lane) {
        lane_sum = wave_scan(div.units(read(shp, seq_lens, lane)));
    }
    __device__ __forceinline__ uint32_t chunk_sum() const { return last_lane(lane_sum); }
    __device__ __forceinline__ void open(const DecodeShape &shp, const int32_t *seq_lens, int lane) {
        const uint64_t G = static_cast<uint64_t>(shp.n_kv_heads) * shp.n_row_groups;
        chunk = 0;
        before = 0;
        uint32_t st = read(shp, seq_lens, lane);
        lane_sum = wave_scan(st);
        uint64_t total = chunk_sum();
        if (__builtin_expect(shp.n_seq > kWave, 0)) {
            for (chunk = kWave; chunk < shp.n_seq; chunk += kWave) total += last_lane(wave_scan(read(shp, seq_lens, lane)));
            chunk = 0;
            st = read(shp, seq_lens, lane);
        }
        const uint64_t sum = total;
        total *= G;
        if (__builtin_expect(shp.kind_known != 0 || !Division::surely_even<!FRESH>(shp, st, sum, total, div.waves_log2), 0)) {
            if (shp.kind_known != 0) div.kind = shp.kind_known;
            else div.template set<!FRESH>(shp, sum, [&](int s0) __attribute__((always_inline)) {
                if (s0 == 0) return st;
                chunk = s0;
                return read(shp, seq_lens, lane);
            });
            if (div.kind != kDivideEvenly) {
                lane_sum = wave_scan(div.units(st));
                total = chunk_sum();
                for (chunk = kWave; chunk < shp.n_seq; chunk += kWave) total += last_lane(wave_scan(div.units(read(shp, seq_lens, lane))));
                total *= G;
            }
            chunk = 0;
            if (shp.n_seq > kWave) read(shp, seq_lens, lane);   // (lane_len)
        }
        div.share(total, static_cast<int>(blockIdx.x), &pos, &end);
    }
    // The next segment (wave-uniform) and this wavefront's part of it; false when the share is done.
    __device__ __forceinline__ bool next(const DecodeShape &shp, const int32_t *seq_lens, int wave, int lane, WaveWork *ww) {
        const uint64_t G = static_cast<uint64_t>(shp.n_kv_heads) * shp.n_row_groups;
        int l, len, n_steps, g;
        uint32_t lo, hi;
        // (the compiler computes what depends on the kind once and keeps it in registers across the segment's steps, which spills;
        // FRESH false: a kernel with registers to spare, where that is 0.15 us less of a call)
        Division div = this->div;
        if constexpr (FRESH) asm volatile("" : "+s"(div.kind));
        do {
            if (pos >= end) return false;
            while ((before + chunk_sum()) * G <= pos) {   // (more than 64 sequences; a later one holds unit pos, so it ends)
                before += chunk_sum();
                chunk += kWave;
                look(shp, seq_lens, lane);
            }
            l = __ffsll(static_cast<unsigned long long>(__ballot((before + lane_sum) * G > pos))) - 1;
            len = __builtin_amdgcn_readlane(lane_len, l);
            const uint32_t sum = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lane_sum), l));
            n_steps = steps_of(len, shp.max_len, TPS);   // > 0: the sequence holds unit pos
            const uint32_t n_units = div.units(static_cast<uint32_t>(n_steps));
            const uint64_t first = (before + sum - n_units) * G;
            const uint64_t local = pos - first;
            g = __builtin_amdgcn_readfirstlane(static_cast<int>(divide(local, n_units)));
            const uint64_t group_first = static_cast<uint64_t>(static_cast<uint32_t>(g)) * n_units;
            const uint64_t stop = first + group_first + n_units;
            const uint64_t seg_end = stop < end ? stop : end;
            lo = div.quanta_before(static_cast<uint32_t>(local - group_first));
            hi = div.quanta_before(static_cast<uint32_t>(seg_end - first - group_first));
            pos = seg_end;
        } while (lo >= hi);   // (none of the pair's quanta begins in this share)
        const int begin = static_cast<int>(lo << div.steps_log2());
        ww->seq = chunk + l;
        ww->grp = 0;
        ww->kvh = g;
        if (shp.n_row_groups > 1) {
            ww->kvh = g / shp.n_row_groups;
            ww->grp = g - ww->kvh * shp.n_row_groups;
        }
        ww->group_id = static_cast<int64_t>(ww->seq) * static_cast<int64_t>(G) + g;
        ww->slot = static_cast<int64_t>(blockIdx.x) + ww->group_id;
        ww->pair = static_cast<int64_t>(ww->seq) * shp.n_kv_heads + ww->kvh;
        ww->len = len;
        ww->n_tiles = static_cast<int>((static_cast<uint32_t>(len) + kWave - 1) / kWave);
        ww->step_end = min(static_cast<int>(hi << div.steps_log2()), n_steps);
        ww->step_begin = begin + wave;
        ww->step_stride = NW;
        const int more = max(ww->step_end - 1 - ww->step_begin, 0);
        ww->step_last = ww->step_begin + more / NW * NW;
        return true;
    }
};

// A segment's partial results of NW wavefronts, in LDS: acc[wave][row][channel] and ml[wave][row] = (m, l), complete after
// a barrier, merged into one partial per query row (the flash-decoding identity) at the segment's slot.
template <int D, int RG, int NW>
__device__ __forceinline__ void merge_waves(const DecodeShape &shp, const WaveWork &ww, const float *acc, int acc_stride,
                                            const float *ml, int ml_stride, float *part_ml, float *part_acc, int tid) {
#pragma unroll 1
    for (int e = tid; e < RG * D / 4; e += NW * kWave) {
        const int r = e / (D / 4);
        if (ww.grp * RG + r >= shp.rows_per_kv) continue;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m = fmaxf(m, ml[w * ml_stride + 2 * r]);
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float l = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = ml[w * ml_stride + 2 * r];
            const float f = mw == -INFINITY ? 0.0f : exp2_raw((mw - m) * kLog2e);
            const float4 x = reinterpret_cast<const float4 *>(acc + w * acc_stride)[e];
            a.x = fmaf(f, x.x, a.x); a.y = fmaf(f, x.y, a.y); a.z = fmaf(f, x.z, a.z); a.w = fmaf(f, x.w, a.w);
            l = fmaf(f, ml[w * ml_stride + 2 * r + 1], l);
        }
        if (__builtin_expect(shp.out != nullptr, 0)) {   // all of the row: the output, and no partial, which nothing would read
            const int row = ww.grp * RG + r, qi = row / shp.heads_per_kv, head = ww.kvh * shp.heads_per_kv + row % shp.heads_per_kv;
            const int64_t orow = (static_cast<int64_t>(ww.seq) * shp.n_q + qi) * shp.n_q_heads + head;
            const bool any = l > 0.0f;
            reinterpret_cast<float4 *>(shp.out + orow * D)[e % (D / 4)] =
                make_float4(any ? a.x / l : 0.0f, any ? a.y / l : 0.0f, any ? a.z / l : 0.0f, any ? a.w / l : 0.0f);
            continue;
        }
        reinterpret_cast<float4 *>(part_acc + ww.slot * (RG * D))[e] = a;
        if (e % (D / 4) == 0) {
            part_ml[(ww.slot * RG + r) * 2] = m;
            part_ml[(ww.slot * RG + r) * 2 + 1] = l;
        }
    }
}

// Calls without a merge (shp.out): workgroup b writes the output rows of pair b, zeros, if the pair has no tokens.
template <int D, int RG>
__device__ __forceinline__ void zero_empty_pair(const DecodeShape &shp, const int32_t *seq_lens, int tid, int nthreads) {
    const uint32_t b = blockIdx.x, per = static_cast<uint32_t>(shp.n_kv_heads * shp.n_row_groups);
    const uint32_t seq = b / per;
    if (seq >= static_cast<uint32_t>(shp.n_seq) || min(seq_lens[seq], shp.max_len) > 0) return;
    const int g = static_cast<int>(b % per), kvh = g / shp.n_row_groups, grp = g % shp.n_row_groups;
#pragma unroll 1
    for (int e = tid; e < RG * D; e += nthreads) {
        const int row = grp * RG + e / D;
        if (row >= shp.rows_per_kv) continue;
        const int qi = row / shp.heads_per_kv, head = kvh * shp.heads_per_kv + row % shp.heads_per_kv;
        shp.out[((static_cast<int64_t>(seq) * shp.n_q + qi) * shp.n_q_heads + head) * D + e % D] = 0.0f;
    }
}

// Tiles per step of the split-K kernels: up to d = 128 a lane carries two keys (see the kernel).  The host's
// DecodeShape carries the same number (tiles_per_step) for the division of the work.
template <int D>
constexpr int decode_keys_per_lane() { return D <= 128 ? 2 : 1; }

// ---- D0: q_rot = scale * H (s . q), one wavefront per query row ------------------------------
// Lane l holds elements l EPL .. + EPL - 1 of the row, EPL = D / 64.
// The row as the caller stores it with the signs applied; row = index among the rows of KV head kvh of sequence seq, zeros
// past the last one.
template <int D>
__device__ __forceinline__ void load_query_row(const DecodeShape &s, int seq, int kvh, int row, int lane, float (&x)[D / kWave]) {
    constexpr int EPL = D / kWave;
#pragma unroll
    for (int j = 0; j < EPL; ++j) x[j] = 0.0f;
    if (row < s.rows_per_kv) {
        const int qi = row / s.heads_per_kv;
        const int head = kvh * s.heads_per_kv + row % s.heads_per_kv;
        const int64_t base = ((static_cast<int64_t>(seq) * s.n_q + qi) * s.n_q_heads + head) * D + lane * EPL;
        const uint32_t neg = s.signs[kvh * (D / 8) + ((lane * EPL) >> 3)];
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            const float val = s.q_is_bf16 ? __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(s.q)[base + j]) << 16)
                                          : static_cast<const float *>(s.q)[base + j];
            x[j] = (neg >> ((lane * EPL + j) & 7)) & 1 ? -val : val;
        }
    }
}

// Unnormalised Walsh-Hadamard transform of the row.
template <int D>
__device__ __forceinline__ void transform_row(int lane, float (&x)[D / kWave]) {
    constexpr int EPL = D / kWave;
    // butterflies over the in-lane bits of the element index ...
#pragma unroll
    for (int h = 1; h < EPL; h <<= 1) {
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            if ((j & h) == 0) {
                const float a = x[j], b = x[j | h];
                x[j] = a + b;
                x[j | h] = a - b;
            }
        }
    }
    // ... then over the lane bits: the element with the bit clear takes a + b, the other a - b
    static_for<0, 6>([&](auto bb) {
        constexpr int m = 1 << decltype(bb)::value;
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
            const float other = lane_xor<m>(x[j], lane);
            x[j] = other + ((lane & m) ? -x[j] : x[j]);
        }
    });
}

template <int D>
__device__ __forceinline__ void rotate_row(const DecodeShape &s, int lane, float (&x)[D / kWave]) {
    transform_row<D>(lane, x);
    const float norm = s.scale * (D == 64 ? 0.125f : (D == 128 ? 0.08838834764831845f : 0.0625f));
#pragma unroll
    for (int j = 0; j < D / kWave; ++j) x[j] *= norm;
}

// Optional 1-bit QJL residual (Sec. 3.6): q2 = sqrt(pi / (2 d)) * H diag(s') q_rot, from a row rotated already.
template <int D>
__device__ __forceinline__ void rotate_row_again(const DecodeShape &s, int kvh, int lane, float (&x)[D / kWave]) {
    constexpr int EPL = D / kWave;
    const uint32_t neg = s.signs2[kvh * (D / 8) + ((lane * EPL) >> 3)];
#pragma unroll
    for (int j = 0; j < EPL; ++j) x[j] = (neg >> ((lane * EPL + j) & 7)) & 1 ? -x[j] : x[j];
    transform_row<D>(lane, x);
    // 1 / sqrt(d) of the Hadamard matrix times sqrt(pi / (2 d)) of the estimator = sqrt(pi / 2) / d
    const float c = 1.2533141373155003f / static_cast<float>(D);
#pragma unroll
    for (int j = 0; j < EPL; ++j) x[j] *= c;
}

// The kernels with a matrix-core score pass rotate the rows of a segment themselves (the queries of a row group are a few
// hundred bytes, and a launch of their own cost 4 - 5 us of the call); this kernel serves the others, which read rotated
// queries from memory.  Output layout per (sequence, KV head, row group): [QS coordinates][RG rows], so that the RG
// values a key needs for one coordinate are adjacent.  Rows past rows_per_kv and coordinates past d are written as zeros.
template <int D, int QS>
__global__ __launch_bounds__(kWave) void rotate_queries_kernel(DecodeShape s, float *__restrict__ q_rot, float *__restrict__ q2) {
    constexpr int EPL = D / kWave;  // elements per lane (1, 2, 4)
    const int lane = threadIdx.x;
    const int rg = s.rows_per_pass;
    const int padded_rows = s.n_row_groups * rg;
    const int64_t gid = blockIdx.x;  // (seq, kvh, padded row)
    const int row = static_cast<int>(gid % padded_rows);
    const int kvh = static_cast<int>((gid / padded_rows) % s.n_kv_heads);
    const int seq = static_cast<int>(gid / (static_cast<int64_t>(padded_rows) * s.n_kv_heads));
    float *dst = q_rot + (gid / rg) * (static_cast<int64_t>(QS) * rg) + (row % rg);
    float x[EPL];
    load_query_row<D>(s, seq, kvh, row, lane, x);
    rotate_row<D>(s, lane, x);
#pragma unroll
    for (int j = 0; j < EPL; ++j) dst[static_cast<int64_t>(lane * EPL + j) * rg] = x[j];
    for (int e = D + lane; e < QS; e += kWave) dst[static_cast<int64_t>(e) * rg] = 0.0f;
    if (q2 != nullptr) {
        rotate_row_again<D>(s, kvh, lane, x);
#pragma unroll
        for (int j = 0; j < EPL; ++j) q2[gid * D + lane * EPL + j] = x[j];
    }
}

// The rows of a segment's row group, RG rows over NW wavefronts: requested early (load), rotated into LDS later (store).
template <class P, int RG, int NW>
struct SegmentQueries {
    static constexpr int EPL = P::D / kWave, PER = (RG + NW - 1) / NW;
    float x[PER][EPL];
    __device__ __forceinline__ void load(const DecodeShape &s, const WaveWork &ww, int wave, int lane) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (wave + i * NW < RG) load_query_row<P::D>(s, ww.seq, ww.kvh, ww.grp * RG + wave + i * NW, lane, x[i]);
    }
    // rows[r][coordinate], zero past d; rows2[r][coordinate] (or NULL) the second rotation
    __device__ __forceinline__ void store(const DecodeShape &s, const WaveWork &ww, int wave, int lane, float (*rows)[P::QS],
                                          float (*rows2)[P::D]) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = wave + i * NW;
            if (r < RG) {
                rotate_row<P::D>(s, lane, x[i]);
#pragma unroll
                for (int j = 0; j < EPL; ++j) rows[r][lane * EPL + j] = x[i][j];
                if (P::D + lane < P::QS) rows[r][P::D + lane] = 0.0f;
                if (rows2 != nullptr) {
                    rotate_row_again<P::D>(s, ww.kvh, lane, x[i]);
#pragma unroll
                    for (int j = 0; j < EPL; ++j) rows2[r][lane * EPL + j] = x[i][j];
                }
            }
        }
    }
};

template <int REP>
__device__ __forceinline__ uint32_t lane_part(int lane) { return (static_cast<uint32_t>(lane) & (REP - 1)) << 4; }

// Triplets per chunk of the score pass, and chunks: 8 / RG, but four of one row and two keys (eight of them spill: one query
// row, 4 bits, d = 64, 8 x 16384 tokens, 8 KV heads 45 us, with the residual 56; four: 42 and 49).
template <int RG, int KPL>
constexpr int score_triplets() { return RG == 1 && KPL == 2 ? 4 : 8 / RG; }
template <class P, int RG, int KPL>
constexpr int score_chunks() { return (P::NTRI + score_triplets<RG, KPL>() - 1) / score_triplets<RG, KPL>(); }

struct NoChunkHook {
    template <class C>
    __device__ __forceinline__ void operator()(C) const {}
};

// `hook(integral_constant<chunk>)` is called once per chunk, after the requests of the next chunk and before
// the arithmetic of this one: the caller's slot for work that is to be spread evenly over the pass (the
// matrix-core kernel runs the previous step's P.V and requests this step's values there).  LDS reads the
// hook issues are complete at the top of the next chunk.
template <class P, int RG, int KPL, class Hook = NoChunkHook>
__device__ __forceinline__ void tile_scores(const uint32_t (&w)[KPL][P::NWORDS], const float *__restrict__ qg,
                                            const DecodeTables<P> &tb, int lane, float (&s)[KPL][RG],
                                            const Hook &hook = Hook{}) {
    constexpr int CT = score_triplets<RG, KPL>();    // triplets per chunk
    constexpr int NCHUNK = score_chunks<P, RG, KPL>();
    constexpr int QC = CT * 3 * RG;                  // query floats per chunk
#pragma unroll
    for (int k = 0; k < KPL; ++k)
#pragma unroll
        for (int r = 0; r < RG; ++r) s[k][r] = 0.0f;
    float rgv[KPL][4];                               // the norm centroids of the group last looked up
#pragma unroll
    for (int k = 0; k < KPL; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) rgv[k][e] = 0.0f;
    float qv[2][QC];
    float4 nv[2][CT][KPL];
    float rv[2][CT][KPL];

    auto request = [&](auto cc) __attribute__((always_inline)) {
        constexpr int ci = decltype(cc)::value;
        constexpr int c0 = ci * CT;
        constexpr int cn = (P::NTRI - c0) < CT ? (P::NTRI - c0) : CT;
        constexpr int buf = ci & 1;
#pragma unroll
        for (int e = 0; e < cn * 3 * RG; ++e) qv[buf][e] = qg[c0 * 3 * RG + e];
        static_for<0, cn>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            constexpr int i = c0 + t;
            constexpr int c = P::cls(i);
            constexpr int ii = c ? i - P::NT0 : i;   // index within the class
            constexpr int bn = P::bnrm(i);
            constexpr int bd = P::bdir(i);
            using RT = RhoTable<bn>;
            using DT = DirTable<bd>;
            static_for<0, KPL>([&](auto kk) {
                constexpr int k = decltype(kk)::value;
                const uint32_t code = field<P::dir_bit(i), 2 * bd>(w[k]);
                if constexpr (joint_codes(bd, bn)) {
                    using JT = JointTable<bd, bn>;
                    constexpr int nb = P::nrm_bit(i), db = P::dir_bit(i);
                    uint32_t off;
                    if constexpr (JT::BYTE_CODES && (nb & 31) + bn <= 32) {
                        // written out: the compiler's own choice takes four or five instructions
                        const uint32_t dl = __builtin_amdgcn_perm(w[k][db >> 5], lane_part<JT::REP>(lane),
                                                                  0x0c0c0000u | ((4u + ((db & 31) >> 3)) << 8));
                        uint32_t nrm;
                        asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(nrm) : "v"(w[k][nb >> 5]), "n"(nb & 31), "n"(bn));
                        asm("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(off) : "v"(nrm), "n"(JT::NS), "v"(dl));
                    } else {
                        off = (code << JT::CS) | (field<nb, bn>(w[k]) << JT::NS) | lane_part<JT::REP>(lane);
                    }
                    nv[buf][t][k] = *reinterpret_cast<const float4 *>(
                        reinterpret_cast<const char *>(c ? tb.dir1 : tb.dir0) + off);
                    rv[buf][t][k] = 1.0f;
                } else {
                    if constexpr (ii % RT::NTG == 0) {
                        constexpr int gbit = (c ? P::NRM1_BIT : P::NRM0_BIT) + ii * bn;
                        // the streams are padded to whole bytes, a whole number of groups; the last group
                        // may reach past the class's triplets, never past its stream
                        const uint32_t gi = field_clamped<gbit, RT::BITS, P::NWORDS>(w[k]);
                        const float *entry =
                            (c ? tb.rho1 : tb.rho0) + (gi * RT::REP + (lane & (RT::REP - 1))) * RT::NTG;
                        if constexpr (RT::NTG == 4) {
                            const float4 e = *reinterpret_cast<const float4 *>(entry);
                            rgv[k][0] = e.x; rgv[k][1] = e.y; rgv[k][2] = e.z; rgv[k][3] = e.w;
                        } else if constexpr (RT::NTG == 1) {
                            rgv[k][0] = entry[0];
                        } else {
                            const float2 e = *reinterpret_cast<const float2 *>(entry);
                            rgv[k][0] = e.x; rgv[k][1] = e.y;
                        }
                    }
                    nv[buf][t][k] = (c ? tb.dir1 : tb.dir0)[code * DT::REP + (lane & (DT::REP - 1))];
                    rv[buf][t][k] = rgv[k][ii % RT::NTG];
                }
            });
        });
    };

    request(std::integral_constant<int, 0>{});
    static_for<0, NCHUNK>([&](auto cc) {
        constexpr int ci = decltype(cc)::value;
        constexpr int c0 = ci * CT;
        constexpr int cn = (P::NTRI - c0) < CT ? (P::NTRI - c0) : CT;
        constexpr int buf = ci & 1;
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the inputs of this chunk have arrived
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ci + 1 < NCHUNK) request(std::integral_constant<int, ci + 1>{});
        hook(cc);
        static_for<0, cn>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            static_for<0, KPL>([&](auto kk) {
                constexpr int k = decltype(kk)::value;
                const float4 n = nv[buf][t][k];
                float tx = n.x, ty = n.y, tz = n.z;
                if constexpr (!joint_codes(P::bdir(c0 + t), P::bnrm(c0 + t))) {
                    const float rho = rv[buf][t][k];
                    tx *= rho; ty *= rho; tz *= rho;
                }
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    s[k][r] = fmaf(qv[buf][(3 * t) * RG + r], tx, s[k][r]);
                    s[k][r] = fmaf(qv[buf][(3 * t + 1) * RG + r], ty, s[k][r]);
                    s[k][r] = fmaf(qv[buf][(3 * t + 2) * RG + r], tz, s[k][r]);  // rotated queries are zero past d
                }
            });
        });
        // The accumulators pass through an empty volatile asm at the end of each chunk: instruction
        // selection orders side-effect-free arithmetic freely within the block, and without this anchor it
        // may defer every multiply-add past the last chunk, keeping the whole query live (spilled).
#pragma unroll
        for (int k = 0; k < KPL; ++k)
#pragma unroll
            for (int r = 0; r < RG; ++r) asm volatile("" : "+v"(s[k][r]));
        __builtin_amdgcn_sched_barrier(0);
    });
}

// ---- D2-D4 on the matrix cores ------------------------------------------------------------------------
// Once the table entry of a triplet is in hand, its contribution to the scores is a product of (x, y, z) of the query
// rows with (x, y, z) of the entry.  v_mfma_f32_16x16x32_bf16 takes 16 keys x 16 operand rows x 32 slots: lane (n, g) =
// (l % 16, l / 16) supplies 8 slots of key n, and a table entry is 8 slots: the leading parts of (x, y, z, 0) and their
// remainders.  So the four lane groups supply four triplets of the same 16 keys: lane group g takes the triplets of
// quarter g of each class, of the keys of all four blocks of 16 keys of the tile one after the other.
//   * fp32 accuracy from bf16 pairs: entry = e_hi + e_lo, q = q_hi + q_lo.  The operand rows hold q_hi (twice: against e_hi
//     and e_lo) and q_lo (twice) of every query row, so one instruction covers all four products for up to 8 rows.
//   * records arrive one key per lane; a quarter's code bits are cut out of the record with funnel shifts and moved to the
//     lanes that look them up by exchanges of lane rows (a 4 x 4 transpose per register: block of keys <-> quarter).
//   * in the accumulators of a block the rows of a key lie in lane groups [hi, lo, hi, lo] (up to four rows) or
//     [hi 0-3, hi 4-7, lo 0-3, lo 4-7]; a few more exchanges add hi and lo and leave every lane with its own key's scores.
// Bound by the issue of vector instructions and LDS reads of one wavefront per SIMD: per tile and 43 triplets this is 44
// instructions of ~17 cycles whatever the rows, 44 lookups and 11 operand reads, where a 4 x 4 x 4 product per triplet and
// four rows took 129 (258 for eight rows) of ~15 cycles, 43 lookups and 43 (86) operand reads.  Long contexts wait for
// memory either way; eight rows per KV head gain (4 x 16384 tokens, d = 256, b = 3: 91 -> 67 us with the work split; 8 x
// 16384, d = 128, b = 1: 74 -> 59).
template <class P>
struct MxSteps {
    static constexpr int NS0 = (P::NT0 + 3) / 4, NS1 = (P::NT1 + 3) / 4;   // triplets per quarter of each class
    static constexpr int N = NS0 + NS1;
};

// Query operands of a segment, in LDS: entry (step j, lane group g, operand row m) = the 4 slots (x, y, z, 0) that row m
// has for the triplet lane group g looks up in step j (zeros past the class's last triplet and past the query rows).
template <class P, int RG>
struct QueryOperands {
    static constexpr int ROWS = RG <= 4 ? 8 : 16;
    uint2 e[MxSteps<P>::N][4][ROWS];
};

template <class P, int RG>
__device__ __forceinline__ void build_query_operands(uint2 *dst, const float (*rows)[P::QS], int tid, int nthreads) {
    using M = MxSteps<P>;
    constexpr int ROWS = QueryOperands<P, RG>::ROWS;
#pragma unroll 1
    for (int e = tid; e < M::N * 4 * ROWS; e += nthreads) {
        const int m = e % ROWS, g = (e / ROWS) % 4, j = e / (4 * ROWS);
        const int r = m % (ROWS / 2), in = j < M::NS0 ? g * M::NS0 + j : g * M::NS1 + (j - M::NS0);
        const int i = j < M::NS0 ? in : P::NT0 + in;
        float x = 0.0f, y = 0.0f, z = 0.0f;
        if (r < RG && in < (j < M::NS0 ? P::NT0 : P::NT1)) {
            x = rows[r][3 * i];
            y = rows[r][3 * i + 1];
            z = rows[r][3 * i + 2];
        }
        const uint4 s = split_triplet(x, y, z);
        dst[e] = m < ROWS / 2 ? make_uint2(s.x, s.y) : make_uint2(s.z, s.w);
    }
}

// 32 bits of a record from bit POS on (zeros past its end).
template <int POS, int NW>
__device__ __forceinline__ uint32_t record_bits(const uint32_t (&w)[NW]) {
    constexpr int wi = POS >> 5, sh = POS & 31;
    if constexpr (wi >= NW) return 0u;
    else if constexpr (sh == 0) return w[wi];
    else if constexpr (wi + 1 >= NW) return w[wi] >> sh;
    else return __builtin_amdgcn_alignbit(w[wi + 1], w[wi], sh);
}

// x[s] of lane group b -> x[b] of lane group s.
__device__ __forceinline__ void transpose_groups(uint32_t (&x)[4]) {
    auto s16 = [](uint32_t &a, uint32_t &b) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    };
    auto s32 = [](uint32_t &a, uint32_t &b) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    };
    s16(x[0], x[1]);
    s16(x[2], x[3]);
    s32(x[0], x[2]);
    s32(x[1], x[3]);
}

// The code bits of one class that a lane looks up, for the four keys 16 b + n of a tile: dir[word][block] holds the
// direction codes of its quarter, nrm[word][block] the norm codes.
template <class P, int C, bool COPIES>
struct MxCodes {
    static constexpr int BD = C ? P::BD1 : P::BD0, BN = C ? P::BN1 : P::BN0;
    static constexpr int NS = C ? MxSteps<P>::NS1 : MxSteps<P>::NS0;
    static constexpr int ND = (NS * 2 * BD + 31) / 32, NN = (NS * BN + 31) / 32;
    using JT = JointTable<(BD > 0 ? BD : 1), (BN > 0 ? BN : 1)>;
    // Direction codes of whole bytes and two-bit norm codes (4 + 4 + 2 bits): the norm bits are kept in four shifted
    // copies, so that bits 6 and 7 of a byte of one of them are the code; one byte permute brings the two codes of a
    // triplet together and one and-or cuts and adds the lane part, instead of permute, bit-field extract and shift-or.
    // (COPIES false: kernels short of registers do without them)
    static constexpr bool PAIRED = COPIES && JT::BYTE_CODES && BN == 2 && JT::NS == 6;
    static constexpr int NV = PAIRED ? 4 * NN : NN;
    uint32_t dir[ND > 0 ? ND : 1][4], nrm[NV > 0 ? NV : 1][4];

    __device__ __forceinline__ void cut(const uint32_t (&w)[P::NWORDS]) {
        constexpr int db = C ? P::DIR1_BIT : P::DIR0_BIT, nb = C ? P::NRM1_BIT : P::NRM0_BIT;
        static_for<0, ND>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            static_for<0, 4>([&](auto gg) {
                constexpr int g = decltype(gg)::value;
                dir[t][g] = record_bits<db + g * NS * 2 * BD + 32 * t, P::NWORDS>(w);
            });
            transpose_groups(dir[t]);
        });
        static_for<0, NN>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            uint32_t x[4];
            static_for<0, 4>([&](auto gg) {
                constexpr int g = decltype(gg)::value;
                x[g] = record_bits<nb + g * NS * BN + 32 * t, P::NWORDS>(w);
            });
            transpose_groups(x);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if constexpr (PAIRED) {
                    nrm[4 * t][b] = x[b] << 6;
                    nrm[4 * t + 1][b] = x[b] << 4;
                    nrm[4 * t + 2][b] = x[b] << 2;
                    nrm[4 * t + 3][b] = x[b];
                } else {
                    nrm[t][b] = x[b];
                }
            }
        });
    }
    // byte offset of the table entry of triplet J of the quarter of key block b
    template <int J>
    __device__ __forceinline__ uint32_t offset(int b, uint32_t lane_bits) const {
        if constexpr (PAIRED) {
            constexpr uint32_t sel = 0x0c0c0000u | (static_cast<uint32_t>(4 + J % 4) << 8) | static_cast<uint32_t>((J % 16) / 4);
            const uint32_t both = __builtin_amdgcn_perm(dir[J / 4][b], nrm[4 * (J / 16) + J % 4][b], sel);
            uint32_t off;
            asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(off) : "v"(both), "s"(0xffc0u), "v"(lane_bits));
            return off;
        } else {
            constexpr int dp = J * 2 * BD, np = J * BN;
            uint32_t d[ND > 0 ? ND : 1], n[NN > 0 ? NN : 1];
#pragma unroll
            for (int t = 0; t < ND; ++t) d[t] = dir[t][b];
#pragma unroll
            for (int t = 0; t < NN; ++t) n[t] = nrm[t][b];
            return (field_clamped<dp, 2 * BD>(d) << JT::CS) | (field_clamped<np, BN>(n) << JT::NS) | lane_bits;
        }
    }
};

// All operands come from LDS, so the hardware counter of outstanding LDS reads is exact and the lookups of a unit (one
// step of one tile: four lookups; LEAN: half of one) can be issued AHEAD units before its products.  `hook` is called once
// per unit, after the requests and before the products (see tile_scores).
template <class P, int KPL, bool LEAN>
constexpr int mx_units() { return MxSteps<P>::N * KPL * (LEAN ? 2 : 1); }

template <class P, int RG, int KPL, class Hook = NoChunkHook, int AHEAD = 2, bool LEAN = false, bool COPIES = !LEAN>
__device__ __forceinline__ void tile_scores_mx(const uint32_t (&w)[KPL][P::NWORDS], const QueryOperands<P, RG> &qop,
                                               const DecodeTables<P> &tb, int lane, float (&s)[KPL][RG],
                                               const Hook &hook = Hook{}) {
    using M = MxSteps<P>;
    typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
    typedef __attribute__((ext_vector_type(4))) float f32x4_t;
    constexpr int NU = mx_units<P, KPL, LEAN>();
    constexpr int BPU = LEAN ? 2 : 4;   // key blocks per unit
    constexpr int LA = NU - 1 < AHEAD ? NU - 1 : AHEAD;
    constexpr int NB = LA + 1;
    constexpr int ROWS = QueryOperands<P, RG>::ROWS;
    MxCodes<P, 0, COPIES> c0[KPL];
    MxCodes<P, 1, COPIES> c1[P::NCLASS == 2 ? KPL : 1];
#pragma unroll
    for (int k = 0; k < KPL; ++k) c0[k].cut(w[k]);
    if constexpr (P::NCLASS == 2) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) c1[k].cut(w[k]);
    }
    union Op { uint4 u; bf16x8_t b; };
    Op ev[NB][BPU];
    uint2 qv[2];
    f32x4_t acc[KPL][4];
#pragma unroll
    for (int k = 0; k < KPL; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[k][b] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const uint2 *q_lane = &qop.e[0][lane >> 4][lane & (ROWS - 1)];
    const uint32_t lane0 = lane_part<JointTable<P::BD0, P::BN0>::REP>(lane);
    const uint32_t lane1 = P::NCLASS == 2 ? lane_part<JointTable<(P::BD1 > 0 ? P::BD1 : 1), (P::BN1 > 0 ? P::BN1 : 1)>::REP>(lane) : 0u;
    // units of a step: its tiles in order, (LEAN) each in two halves
    constexpr int UPS = KPL * (4 / BPU);
    auto request = [&](auto uu) __attribute__((always_inline)) {
        constexpr int u = decltype(uu)::value, j = u / UPS, k = u % UPS / (4 / BPU), b0 = u % (4 / BPU) * BPU;
        if constexpr (u % UPS == 0) qv[j & 1] = q_lane[j * 4 * ROWS];
#pragma unroll
        for (int bb = 0; bb < BPU; ++bb) {
            const int b = b0 + bb;
            if constexpr (j < M::NS0)
                ev[u % NB][bb].u = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(tb.dir0) +
                                                                   c0[k].template offset<j>(b, lane0));
            else
                ev[u % NB][bb].u = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(tb.dir1) +
                                                                   c1[P::NCLASS == 2 ? k : 0].template offset<j - M::NS0>(b, lane1));
        }
    };
    static_for<0, LA>(request);
    Op qa;
    qa.u = make_uint4(0u, 0u, 0u, 0u);
    static_for<0, NU>([&](auto uu) {
        constexpr int u = decltype(uu)::value, j = u / UPS, k = u % UPS / (4 / BPU), b0 = u % (4 / BPU) * BPU;
        if constexpr (u % UPS == 0) qa.u = make_uint4(qv[j & 1].x, qv[j & 1].y, qv[j & 1].x, qv[j & 1].y);
        if constexpr (u + LA < NU) request(std::integral_constant<int, u + LA>{});
        hook(uu);
#pragma unroll
        for (int bb = 0; bb < BPU; ++bb)
            acc[k][b0 + bb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa.b, ev[u % NB][bb].b, acc[k][b0 + bb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int k = 0; k < KPL; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x0 = acc[k][0][i], x1 = acc[k][1][i], x2 = acc[k][2][i], x3 = acc[k][3][i];
            if constexpr (RG <= 4) {
                if (i >= RG) continue;
                swap16(x0, x1);            // x0: hi of blocks 0, 1, 0, 1; x1: lo of the same
                swap16(x2, x3);
                const float a = x0 + x1, b = x2 + x3;
                s[k][i < RG ? i : 0] = lane < 32 ? a : b;
            } else {
                swap32(x0, x2);            // x0: hi of blocks 0 (rows 0-3, 4-7) and 2, x2: lo of the same
                swap32(x1, x3);
                float a = x0 + x2, b = x1 + x3;
                swap16(a, b);              // a: rows 0-3 of blocks 0 .. 3, b: rows 4-7
                s[k][i] = a;
                s[k][RG > 4 ? 4 + i : 0] = b;
            }
        }
}

template <int RG>
__device__ __forceinline__ void store_scores(const DecodeShape &shp, const WaveWork &ww, float *scores_out, int tok,
                                             const float (&s)[RG]) {
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        const int row = ww.grp * RG + r;
        if (row < shp.rows_per_kv) {
            const int qi = row / shp.heads_per_kv, head = ww.kvh * shp.heads_per_kv + row % shp.heads_per_kv;
            scores_out[((static_cast<int64_t>(ww.seq) * shp.n_q + qi) * shp.n_q_heads + head) * shp.t_capacity + tok] =
                s[r];
        }
    }
}

// ---- bf16 values: P.V on the matrix cores -------------------------------------------------------
// v_mfma_f32_16x16x32_bf16 computes D[16x16] += A[16x32] B[32x16]; lane l holds row l%16 of A and
// column l%16 of B, each for the 8 k-slots of lane group l/16, and rows 4*(l/16)..+3 of column l%16
// of D.  Here M = probability rows, K = keys, N = channels:
//   * a 64-key tile is two k-steps; k-slot (g, j) of step ks is key 32*ks + 4*j + g, so that one
//     wave-wide value load (fixed j) reads 4 consecutive value rows (measured faster than 4 rows that
//     lie 8 apart);
//   * lane (n, g) loads CPL = d/16 channels of its 8 keys per k-step, 16 bytes (8 bytes at d = 64) of every
//     256-byte piece of the row, so that one load instruction of the wavefront reads whole cache lines;
//     N-block c of the MFMA is the channel set {lane n's c-th channel}, so B operands are byte permutes of
//     the loaded registers and values are never converted;
//   * values come through buffer loads whose descriptor ends at the sequence's last token: rows past
//     it read as zeros without any address clamping;
//   * a probability is split into two bf16 numbers, hi = its upper 16 bits and lo = the rest, which
//     occupy rows r and RP + r of A; the two partial results are added at the end.  The relative
//     error of hi + lo is below 2^-16.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// Keys per lane and step of the bf16-value kernel.  The kernel runs one wavefront per SIMD (all 512
// vector registers of a lane): measured faster than two wavefronts with half the registers each,
// because a step's values (16 KB per 64 keys at d = 128) stay in flight in registers during the whole
// score phase without spilling.  Up to d = 128 a lane carries two keys, so that every scalar query
// chunk, every wave-wide maximum and every accumulator rescale serves 128 keys.
template <int KPL>
constexpr int prob_row() { return KPL * kWave + 8; }  // bf16 per probability row in LDS: keys + 8 pad

template <class P, int KPL>
struct DecodeSmemMfma {
    DecodeTables<P> tb;
    __attribute__((aligned(16))) uint16_t pbuf[kDecodeWaves][16][prob_row<KPL>()];
};

// Optional 1-bit QJL residual (Sec. 3.6).  The correction of a key is a product with signs, sum_j sigma_j q2_j per
// query row: 16 keys x 16 operand rows x 32 coordinates at a time on v_mfma_f32_16x16x32_bf16, the signs as bf16 +-1
// (exact) and each q2 as the sum of three bf16 numbers (24 bits: exact as well, up to numbers far below the row's size).
//   * B: lane (n, g) = (l % 16, l / 16) holds the sign words of group g of key n of each block of 16 keys, loaded in that
//     form from the side-car.  Bits i and i + 16 of a word become one register of two bf16 numbers with a shift and an
//     and-or (their sign bits under a constant 1.0).
//   * A: operand rows as in LDS below: with up to four query rows the three parts are rows r, 4 + r and 8 + r of one
//     operand, with eight the leading parts and first remainders are rows r and 8 + r of one operand and the second
//     remainders rows r of another one that adds to the same accumulators.
//   * the parts of a key's sum sit in lane groups of the accumulators of its block; three to five exchanges of lane rows
//     per register add them up and leave every lane with the sums of its own key.
// This took the place of a table of signed sums per byte of signs (d / 8 x 256 x rows floats), which cost d / 8 random
// 16-byte LDS reads and their additions per key, limited the row group to what fitted LDS (4 at d = 128, 2 at d = 256: more
// rows read the keys again) and was rebuilt for every work item: 0.243 -> 0.233 ms for 16 x 32768 tokens x 8 KV heads at
// d = 128, b = 3 with four query heads per KV head, where the kernel is now bound by memory as without the residual.
template <int D, int RG>
struct QjlOperands {
    static constexpr int WORDS = D / 32;                        // sign words per key
    static constexpr int WPL = WORDS < 4 ? 1 : WORDS / 4;       // sign words per lane and key
    static constexpr int STEPS = D / 32;                        // k-steps of 32 coordinates
    static constexpr int SETS = RG <= 4 ? 1 : 2;                // A operands per k-step
    uint4 a[SETS][STEPS][4][16];                                // [set][k-step][lane group][operand row]
    // word i of a lane's (at d = 64 two lane groups share a word)
    static __device__ __forceinline__ int word(int g, int i) { return WORDS < 4 ? g >> 1 : g * WPL + i; }
    // coordinate of element j of lane group g in k-step s
    static __device__ __forceinline__ int coordinate(int g, int s, int j) {
        const int pair = (j >> 1) + 16 * (j & 1);
        if constexpr (D == 64) return 32 * (g >> 1) + 8 * (g & 1) + 4 * s + pair;
        else return 32 * (g * WPL + s / 4) + 4 * (s % 4) + pair;
    }
};

// SCORES: also store the scaled scores (a second instantiation, so that the usual one carries none of
// the addressing state of that store through its loop).
// QJL: add the 1-bit QJL residual correction of Sec. 3.6 to every score (side-car `qjl`, second rotated
// queries `q2`).
// PAGED: `cache` and `v` are pools of 64-token pages, [page][KV head] tiles each (a key tile in the device
// layout of the contiguous cache, a value tile of 64 rows), and logical tile j of sequence s lives in page
// pt_table[s * pt_stride + j] (ids outside [0, pt_pages) are clamped: a bad table reads wrong pages, never
// outside the pools).  The page ids of a step are read one step before its loads are issued.
template <class P, int RG, bool SCORES, bool QJL, bool PAGED = false>
__global__ __launch_bounds__(kDecodeWaves *kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void decode_kernel_mfma(
    DeviceBooks books, DecodeShape shp, const float *__restrict__ q_rot, const uint4 *__restrict__ cache,
    const uint32_t *__restrict__ v, const int32_t *__restrict__ seq_lens, float *__restrict__ part_ml,
    float *__restrict__ part_acc, float *__restrict__ scores_out,
    const unsigned char *__restrict__ qjl, const float *__restrict__ q2, const int32_t *__restrict__ pt_table,
    int32_t pt_stride, int32_t pt_pages) {
    // (the table as a restrict-qualified kernel argument of its own: its loads are then known not to be
    // clobbered by the kernel's stores and become scalar loads)
    constexpr int D = P::D;
    constexpr int KPL = decode_keys_per_lane<D>();
    constexpr bool AHEAD = D <= 128;       // P.V runs one step behind the scores, inside the next score pass
    constexpr int KS = 2 * KPL;            // k-steps of 32 keys per step
    constexpr int CPL = D / 16;            // channels per lane chunk = N-blocks
    constexpr int CW = CPL / 2;            // 32-bit words per chunk
    constexpr int RP = RG < 4 ? 4 : RG;    // probability rows padded to a multiple of 4
    constexpr int ROWB = D * 2;            // bytes per value row
    constexpr int TILEB = P::GRANULES * kWave * 16;  // bytes per cache tile
    constexpr int PROW = prob_row<KPL>();
    constexpr int QW = D / 32;             // sign words per key of the QJL side-car
    constexpr int TQ = kWave * (D / 8 + 2);  // side-car bytes per tile
    // static, so that table addresses are compile-time constants that fold into the LDS instructions
    constexpr bool MX = mx_scores<P>();    // scores on the matrix cores (every plan up to 3 bits per coordinate)
    // fewer registers for the score pass where it would spill (one row, 3 bits, 16 x 32768 tokens, 8 KV heads, spilling 231 us, so 203)
    // (eight rows without the residual keep the two-instruction lookups: 16 x 1500 tokens 22.5 -> 22.2, 16 x 32768 208.4 -> 207.8;
    // not at two classes, over pages they spill)
    constexpr bool LEAN = QJL || RG == 8 || RG == 1 || P::NCLASS == 2;
    __shared__ DecodeSmemMfma<P, KPL> sm;
    using QO = QjlOperands<D, RG>;
    __shared__ __attribute__((aligned(16))) uint4 qjl_store[QJL ? sizeof(QO) / 16 : 1];
    __shared__ __attribute__((aligned(16))) uint2 qop_store[MX ? sizeof(QueryOperands<P, RG>) / 8 : 1];
    const QueryOperands<P, RG> &qop = *reinterpret_cast<const QueryOperands<P, RG> *>(&qop_store[0]);
    // the wavefronts' results at the end of a segment; at its start the rotated queries lie there (MX)
    __shared__ __attribute__((aligned(16))) float seg_acc[kDecodeWaves][RG][D];
    __shared__ float seg_ml[kDecodeWaves][RG][2];
    static_assert(P::QS + D <= kDecodeWaves * D, "both rotations fit");
    float (*q_rows)[P::QS] = reinterpret_cast<float (*)[P::QS]>(&seg_acc[0][0][0]);
    float (*q2_rows)[D] = reinterpret_cast<float (*)[D]>(&seg_acc[0][0][0] + RG * P::QS);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept in a scalar register
    BookLevels<P> levels;
    levels.load(lane);
    WorkSpan<KPL, kDecodeWaves> span;
    span.open(shp, seq_lens, lane);
    if (__builtin_expect(shp.out != nullptr, 0)) zero_empty_pair<D, RG>(shp, seq_lens, tid, kDecodeWaves * kWave);
    if (span.pos >= span.end) return;   // (whole workgroup, before any barrier)
    levels.store(sm.tb, tid);           // (kept in registers until the tables are built they are live through the steps)
    // The tables are built inside the segment loop, after the first segment's first loads have been issued:
    // those do not depend on the tables, and their latency covers the build.
    bool tables_built = false;

    // per segment (set in the segment loop below; the helpers capture them by reference)
    WaveWork ww;
    const float *qg = q_rot;
    const char *k_region = reinterpret_cast<const char *>(cache);
    const char *v_pair = reinterpret_cast<const char *>(v);
    const int n16 = lane & 15, g4 = lane >> 4;
    const uint32_t k_lane = lane * 16u;
    // A value row is read in pieces of 16 lanes x LANEB bytes, each piece contiguous (whole cache lines per
    // load instruction: with the non-temporal hint a line touched by two instructions may be fetched twice).
    // Lane n16 holds bytes [n16 LANEB, (n16 + 1) LANEB) of every piece: at d = 256 its 16 channels are
    // 8 n16 .. + 7 and 128 + 8 n16 .. + 7, and N-block c of the P.V product is channel
    // (c / 8) 128 + 8 n16 + c % 8.
    constexpr int LANEB = CPL * 2 < 16 ? CPL * 2 : 16;
    // Byte offsets of this lane's channels in its rows 32 ks + 4 j + g4: one register per JB values of j,
    // the others reached by immediate offsets (below 4096).
    constexpr int JB = 4096 / (4 * ROWB) < 8 ? 4096 / (4 * ROWB) : 8;
    int v_lane[KS][8 / JB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int h = 0; h < 8 / JB; ++h) v_lane[ks][h] = (32 * ks + 4 * JB * h + g4) * ROWB + n16 * LANEB;
    const int ppos = (lane & 32) + 8 * (lane & 3) + ((lane & 31) >> 2);  // slot of key `lane` in a pbuf row

    // Only the words that hold record bytes are loaded: a register written by a load but never read
    // may be reused at once by the compiler, which then has to wait for that load first.
    auto load_record = [&](int64_t tile, uint32_t (&w)[P::NWORDS]) {
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
        constexpr int USED = (P::RECORD_BYTES + 3) / 4;
        const char *src = k_region + tile * TILEB;
#pragma unroll
        for (int g = 0; g < P::GRANULES; ++g) {
            const char *gp = src + g * (kWave * 16) + k_lane;
            constexpr int kFull = 4;
            const int n = (USED - 4 * g) < kFull ? (USED - 4 * g) : kFull;
            // (global address space said explicitly: the laundered base pointer below would otherwise make these
            // flat loads, which count against the LDS / scalar wait counter as well)
            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
            typedef const u32x4_t __attribute__((address_space(1))) *g4_t;
            typedef const u32x3_t __attribute__((address_space(1))) *g3_t;
            typedef const u32x2_t __attribute__((address_space(1))) *g2_t;
            typedef const uint32_t __attribute__((address_space(1))) *g1_t;
            if (n == 4) {
                const u32x4_t x = __builtin_nontemporal_load((g4_t)(gp));
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = x.z; w[4 * g + 3] = x.w;
            } else if (n == 3) {
                const u32x3_t x = __builtin_nontemporal_load((g3_t)(gp));
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = x.z; w[4 * g + 3] = 0u;
            } else if (n == 2) {
                const u32x2_t x = __builtin_nontemporal_load((g2_t)(gp));
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = 0u; w[4 * g + 3] = 0u;
            } else {
                w[4 * g] = __builtin_nontemporal_load((g1_t)(gp));
                w[4 * g + 1] = 0u; w[4 * g + 2] = 0u; w[4 * g + 3] = 0u;
            }
        }
    };
    // The records of a step; a tile past the sequence's last one is replaced by the last one (its keys
    // are masked out by position), so that nothing outside the tiles that hold tokens is read.
    auto load_records = [&](int step, uint32_t (&w)[KPL][P::NWORDS]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) load_record(min(step * KPL + k, ww.n_tiles - 1), w[k]);
    };
    // PAGED: the page ids of the tiles of a step (the last tile's for tiles past it) are read as they are, one
    // step ahead; the position in the pools (in tiles) is computed from them when the step's loads are issued,
    // so that nothing waits for the table right after asking it.
    // The ids come through the vector memory path (every lane reads the same entry), asked for before the
    // step's other loads: the wait for them one step later then covers only loads that are long complete.  As
    // scalar loads they shared a counter with the query chunks, whose first wait of a step also waited for a
    // table entry that had missed the scalar cache.
    int lane_zero = 0;
    if constexpr (PAGED) asm volatile("" : "+v"(lane_zero));
    auto page_ids = [&](int step, int (&page)[KPL]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            const int tile = max(min(step * KPL + k, ww.n_tiles - 1), 0);
            page[k] = pt_table[static_cast<int64_t>(ww.seq) * pt_stride + tile + lane_zero];
        }
    };
    auto page_slots = [&](const int (&page)[KPL], int64_t (&slot)[KPL]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            const int id = __builtin_amdgcn_readfirstlane(page[k]);
            slot[k] = static_cast<int64_t>(min(max(id, 0), pt_pages - 1)) * shp.n_kv_heads + ww.kvh;
        }
    };
    auto load_records_at = [&](const int64_t (&slot)[KPL], uint32_t (&w)[KPL][P::NWORDS]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) load_record(slot[k], w[k]);
    };
    int64_t slot_cur[KPL];   // PAGED: pool positions of the step being worked on
    int page_nxt[KPL];       // PAGED: page ids of the wave's next step
    // QJL side-car of a tile, layout [word][key] uint32 (bit set: negative), then [key] fp16 residual norms.  Lane (n, g)
    // holds the words of group g of keys 16 b + n, b = 0 .. 3, and the norm of its own key.
    const char *j_region = reinterpret_cast<const char *>(qjl);
    auto load_signs = [&](const char *src, uint32_t (&sc)[4 * QO::WPL + 1]) {
#pragma unroll
        for (int i = 0; i < QO::WPL; ++i)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                sc[4 * i + b] = *reinterpret_cast<const uint32_t *>(src + QO::word(g4, i) * (kWave * 4) + (16 * b + n16) * 4);
        sc[4 * QO::WPL] = *reinterpret_cast<const uint16_t *>(src + QW * (kWave * 4) + lane * 2);
    };
    auto load_sidecar = [&](int step, uint32_t (&sc)[KPL][4 * QO::WPL + 1]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k)
            load_signs(j_region + static_cast<int64_t>(min(step * KPL + k, ww.n_tiles - 1)) * TQ, sc[k]);
    };
    // PAGED: the side-car is a pool of [page][KV head] tiles like the keys'; slot = page * n_kv_heads + KV head
    auto load_sidecar_at = [&](const int64_t (&slot)[KPL], uint32_t (&sc)[KPL][4 * QO::WPL + 1]) {
#pragma unroll
        for (int k = 0; k < KPL; ++k) load_signs(j_region + slot[k] * TQ, sc[k]);
    };
    // q2 . sigma per query row of this lane's key
    auto qjl_dot = [&](const uint32_t (&sc)[4 * QO::WPL + 1], float (&corr)[RG]) __attribute__((always_inline)) {
        const uint4 *a_lane = &qjl_store[g4 * 16 + n16];
        f32x4_t cacc[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) cacc[b] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        uint32_t wrd[4 * QO::WPL];
#pragma unroll
        for (int e = 0; e < 4 * QO::WPL; ++e) wrd[e] = D == 64 ? sc[e] << (8 - 8 * (g4 & 1)) : sc[e];
        // the A operands one k-step ahead; the barriers keep the compiler from expanding all signs first (spills)
        union AOp { uint4 u; bf16x8_t b; };
        AOp qa[2][QO::SETS];
#pragma unroll
        for (int t = 0; t < QO::SETS; ++t) qa[0][t].u = a_lane[t * QO::STEPS * 64];
#pragma unroll
        for (int st = 0; st < QO::STEPS; ++st) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < QO::SETS; ++t)
                if (st + 1 < QO::STEPS) qa[(st + 1) & 1][t].u = a_lane[(t * QO::STEPS + st + 1) * 64];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                union { uint32_t u[4]; bf16x8_t b; } sg;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int sh = D == 64 ? 7 - 4 * st - jj : 15 - 4 * (st % 4) - jj;
                    const uint32_t moved = wrd[D == 64 ? b : 4 * (st / 4) + b] << sh;
                    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(sg.u[jj]) : "v"(moved), "s"(0x80008000u), "v"(0x3f803f80u));
                }
#pragma unroll
                for (int t = 0; t < QO::SETS; ++t)
                    cacc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[st & 1][t].b, sg.b, cacc[b], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x0 = cacc[0][i], x1 = cacc[1][i], x2 = cacc[2][i], x3 = cacc[3][i];
            if constexpr (RG <= 4) {
                // lane groups of a block: [leading, first remainder, second remainder, 0]
                swap16(x0, x1);            // x0: leading parts of blocks 0, 1, then second remainders; x1: first remainders
                swap16(x2, x3);
                float a = x0 + x1, b = x2 + x3;
                swap32(a, b);              // a: (leading + first) of blocks 0 .. 3, b: second remainders of blocks 0 .. 3
                if (i < RG) corr[i < RG ? i : 0] = a + b;
            } else {
                // lane groups of a block: [rows 0-3, rows 4-7, first remainders of rows 0-3, of rows 4-7]
                swap32(x0, x2);            // x0: rows of blocks 0 and 2, x2: their remainders
                swap32(x1, x3);
                float a = x0 + x2, b = x1 + x3;
                swap16(a, b);              // a: rows 0-3 of blocks 0 .. 3, b: rows 4-7
                corr[i] = a;
                corr[RG > 4 ? 4 + i : 0] = b;
            }
        }
    };
    float m_run[RG], l_lane[RG];
    f32x4_t acc[CPL];

    // Values come through a buffer descriptor that covers a step's rows up to the sequence's last token
    // (rows past it read as zero; their probabilities are zero too); the descriptor of a step that does
    // not exist is empty, its loads move nothing.
    auto values_of = [&](int step, bool exists) {
        const int t0 = step * (KPL * kWave);
        const int n_valid = exists ? min(KPL * kWave, ww.len - t0) : 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(v_pair + static_cast<int64_t>(t0) * ROWB), 0,
                                                 n_valid * ROWB, 0x00020000);
    };
    // PAGED: tile k of a step has a descriptor of its own.  The lanes address rows relative to the step's
    // first row, so the descriptor starts 64 k rows before the tile (nothing below the tile is addressed
    // through it) and ends with the tile's last token.
    auto values_at = [&](int step, int k, int64_t slot, bool exists) {
        // (wave-uniform by construction; said so explicitly, or the descriptor may end up in vector registers
        // and every load through it in a loop over its distinct values)
        const int n_valid =
            __builtin_amdgcn_readfirstlane(exists ? min(max(ww.len - (step * KPL + k) * kWave, 0), kWave) : 0);
        const int64_t off = (slot - k) * (kWave * ROWB);
        const uint32_t off_lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(off));
        const uint32_t off_hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(static_cast<uint64_t>(off) >> 32));
        const char *base = v_pair + static_cast<int64_t>((static_cast<uint64_t>(off_hi) << 32) | off_lo);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0,
                                                 n_valid > 0 ? (k * kWave + n_valid) * ROWB : 0, 0x00020000);
    };
    // Values and records are read once and never again: the loads carry the non-temporal hint (bit 1 of the
    // buffer intrinsic's cache policy, the nt bit of a global load), which keeps the stream from displacing
    // what the caches hold.  Measured on the Llama-shaped batch: 0.243 -> 0.205 ms for the whole kernel.
    // this lane's part of k-step ks: 8 rows x CPL channels
    auto load_values = [&](__amdgpu_buffer_rsrc_t rsrc, int ks, uint32_t (&vk)[8][CW]) {
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if constexpr (CW == 2) {
                const u32x2_t x =
                    __builtin_amdgcn_raw_buffer_load_b64(rsrc, v_lane[ks][j / JB] + (j % JB) * (4 * ROWB), 0, kStreamPolicy);
                vk[j][0] = x.x; vk[j][1] = x.y;
            } else {
#pragma unroll
                for (int q4 = 0; q4 < CW / 4; ++q4) {
                    const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(
                        rsrc, v_lane[ks][j / JB] + (j % JB) * (4 * ROWB) + 16 * LANEB * q4, 0, kStreamPolicy);
                    vk[j][4 * q4] = x.x; vk[j][4 * q4 + 1] = x.y; vk[j][4 * q4 + 2] = x.z; vk[j][4 * q4 + 3] = x.w;
                }
            }
        }
    };
    uint32_t vr[KS][8][CW];  // values: of the previous step until its P.V piece has run, then of the current step
    // P.V of one step is cut into KS * CW pieces: piece (ks, q) multiplies the probabilities of k-step ks with
    // the two channel blocks 2 q and 2 q + 1, whose B operands are byte permutes of word q of the k-step's
    // eight value registers.  A piece's A operand (16 bytes of the probability rows in LDS) is read one
    // piece ahead.
    constexpr int NPIECE = KS * CW;
    auto pv_operand = [&](int ks) {
        return *reinterpret_cast<const uint4 *>(&sm.pbuf[wave][n16][32 * ks + 8 * g4]);
    };
    auto pv_piece = [&](auto pp, const uint4 &pa_bits) __attribute__((always_inline)) {
        constexpr int ks = decltype(pp)::value / CW, q = decltype(pp)::value % CW;
        union { uint4 u; bf16x8_t b; } pa;
        pa.u = pa_bits;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            union { uint32_t u[4]; bf16x8_t b; } vb;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                vb.u[jj] = __builtin_amdgcn_perm(vr[ks][2 * jj + 1][q], vr[ks][2 * jj][q], h ? 0x07060302u : 0x05040100u);
            acc[2 * q + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa.b, vb.b, acc[2 * q + h], 0, 0, 0);
        }
    };
    // One step.  Up to d = 128 the step is software pipelined with P.V one step behind the scores: the score
    // pass of step n carries, spread over its chunks, the P.V pieces of step n - 1 (whose probabilities sit in
    // LDS since the end of that step) and, as soon as the last piece of a k-step has read its value registers,
    // the loads of step n's own values into them.  Matrix-core work thus overlaps the vector arithmetic of the
    // scores, and -- what matters more with a single in-order wavefront per SIMD -- the value loads enter the
    // compute unit's memory pipeline a k-step at a time at the pace of the arithmetic, not in one burst per step
    // whose issue stalls the wavefront.  The first step of a segment multiplies zeros (the value registers are
    // cleared at the segment's start), the last step's P.V runs after the loop.  At d = 256 (registers: holding a
    // step's values across the score pass spills there) the values are requested at the top of the step and
    // P.V follows the softmax.  The records of the wave's next step are requested first thing
    // and are used one call later.  The step loop below is unrolled by two with the two record buffers
    // swapping roles, so that no register copies (and no full memory wait in front of them) carry the
    // prefetched records over.
    auto process_step = [&](int step, const uint32_t (&w)[KPL][P::NWORDS], uint32_t (&w_next)[KPL][P::NWORDS],
                            uint32_t (&sc)[KPL][4 * QO::WPL + 1], uint32_t (&sc_next)[KPL][4 * QO::WPL + 1])
                            __attribute__((always_inline)) {
        const int t0 = step * (KPL * kWave);
        const int n_valid = min(KPL * kWave, ww.len - t0);
        // always issued (the wave's last step re-reads its own records): a branch here would make the compiler
        // wait for every outstanding load first
        const int step_nx = min(step + ww.step_stride, ww.step_last);
        __amdgpu_buffer_rsrc_t v_cur[KPL];   // this step's values, per tile of the step (all the same unless PAGED)
        int64_t slot_nxt[KPL];
        if constexpr (PAGED) {
            page_slots(page_nxt, slot_nxt);
            page_ids(min(step_nx + ww.step_stride, ww.step_last), page_nxt);   // used one step from here
        }
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            if constexpr (PAGED) v_cur[k] = values_at(step, k, slot_cur[k], true);
            else v_cur[k] = values_of(step, true);
        }
        if constexpr (!AHEAD) {   // d = 256: the registers hold one step's values only while it is worked on
            // ... and its side-car, asked for before them: held across the previous step it made the residual kernels spill,
            // as did the wide form of the score pass (4 x 16384 tokens, 8 KV heads: b = 3, one row 98 -> 69 us, four rows
            // 103 -> 74; b = 2.5, eight rows 129 -> 83)
            if constexpr (QJL) {
                if constexpr (PAGED) load_sidecar_at(slot_cur, sc);
                else load_sidecar(step, sc);
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) load_values(v_cur[ks / 2], ks, vr[ks]);
        }
        if constexpr (PAGED) {
            load_records_at(slot_nxt, w_next);
            if constexpr (QJL && AHEAD) load_sidecar_at(slot_nxt, sc_next);
#pragma unroll
            for (int k = 0; k < KPL; ++k) slot_cur[k] = slot_nxt[k];
        } else {
            load_records(step_nx, w_next);
            if constexpr (QJL && AHEAD) load_sidecar(min(step + ww.step_stride, ww.step_last), sc_next);
        }
        // The loads above feed the NEXT step, which sits behind a branch in the unrolled loop; without this
        // barrier the compiler sinks them into that branch, i.e. to the top of the step that uses them, and
        // every second step waits for a full memory round trip.
        asm volatile("" ::: "memory");
        // D2-D4: scores (queries carry the softmax scale already).  The query offset (always 0) is
        // laundered per step: otherwise the loop-invariant scalar loads of the whole query are hoisted
        // out of the step loop and hundreds of scalar registers spill.
        float s[KPL][RG];
        int q_off = 0;
        asm volatile("" : "+s"(q_off));
        if constexpr (AHEAD) {
            // chunk c runs pieces [c NPIECE / NCH, (c + 1) NPIECE / NCH) and reads the A operands of chunk c + 1's
            constexpr int NCH = MX ? mx_units<P, KPL, LEAN>() : score_chunks<P, RG, KPL>();
            uint4 pa_bits[NPIECE];
            static_for<0, NPIECE / NCH>([&](auto pp) { pa_bits[decltype(pp)::value] = pv_operand(decltype(pp)::value / CW); });
            auto pv_in_chunk = [&](auto cc) __attribute__((always_inline)) {
                constexpr int ci = decltype(cc)::value;
                constexpr int lo = ci * NPIECE / NCH, hi = (ci + 1) * NPIECE / NCH;
                constexpr int hi_next = ci + 1 < NCH ? (ci + 2) * NPIECE / NCH : hi;
                static_for<hi, hi_next>([&](auto pp) { pa_bits[decltype(pp)::value] = pv_operand(decltype(pp)::value / CW); });
                static_for<lo, hi>([&](auto pp) {
                    constexpr int pi = decltype(pp)::value;
                    pv_piece(pp, pa_bits[pi]);
                    if constexpr (pi % CW == CW - 1) load_values(v_cur[(pi / CW) / 2], pi / CW, vr[pi / CW]);
                });
            };
            if constexpr (MX) tile_scores_mx<P, RG, KPL, decltype(pv_in_chunk), 2, LEAN, !LEAN || (RG == 8 && !QJL && P::NCLASS == 1)>(w, qop, sm.tb, lane, s, pv_in_chunk);
            else tile_scores<P, RG, KPL>(w, qg + q_off, sm.tb, lane, s, pv_in_chunk);
            // the probabilities of the previous step have been read: the new ones may overwrite them
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            if constexpr (MX) tile_scores_mx<P, RG, KPL, NoChunkHook, 2, QJL>(w, qop, sm.tb, lane, s);
            else tile_scores<P, RG, KPL>(w, qg + q_off, sm.tb, lane, s);
        }
#pragma unroll
        for (int k = 0; k < KPL; ++k) {
            const float gamma = __uint_as_float(w[k][0]);
            const bool valid = k * kWave + lane < n_valid;
            if constexpr (QJL) {
                // Sec. 3.6: q . k = gamma (q_rot . u^ + gamma_r q2 . sigma), the estimator's constant is in q2
                float corr[RG];
                qjl_dot(sc[k], corr);
                const float gamma_r = __half2float(__ushort_as_half(static_cast<unsigned short>(sc[k][4 * QO::WPL])));
#pragma unroll
                for (int r = 0; r < RG; ++r) s[k][r] = fmaf(gamma_r, corr[r], s[k][r]);
            }
#pragma unroll
            for (int r = 0; r < RG; ++r) s[k][r] = valid ? s[k][r] * gamma : -INFINITY;
            if constexpr (SCORES) {
                // the kernel with the residual is built once; it looks at the pointer
                if (valid && (!QJL || scores_out != nullptr))
                    store_scores<RG>(shp, ww, scores_out, t0 + k * kWave + lane, s[k]);
            }
        }
        // D5: online softmax, one running maximum per row for the whole wave
        float alpha[RG], mx[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            mx[r] = s[0][r];
#pragma unroll
            for (int k = 1; k < KPL; ++k) mx[r] = fmaxf(mx[r], s[k][r]);
        }
        wave_max_of(mx);
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const float m_new = fmaxf(m_run[r], mx[r]);
            alpha[r] = exp2_raw((m_run[r] - m_new) * kLog2e);
            m_run[r] = m_new;
            float psum = 0.0f;
#pragma unroll
            for (int k = 0; k < KPL; ++k) {
                const float p = exp2_raw((s[k][r] - m_new) * kLog2e);
                psum += p;
                const uint32_t pb = __float_as_uint(p);
                const float lo = p - __uint_as_float(pb & 0xffff0000u);
                sm.pbuf[wave][r][k * kWave + ppos] = static_cast<uint16_t>(pb >> 16);
                sm.pbuf[wave][RP + r][k * kWave + ppos] = static_cast<uint16_t>(__float_as_uint(lo) >> 16);
            }
            l_lane[r] = fmaf(l_lane[r], alpha[r], psum);
        }
        // accumulator rows of this lane: m = 4 * g4 + i, probability row r = m % RP
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a;
            if constexpr (RP == 4) {
                a = i < RG ? alpha[i < RG ? i : 0] : 1.0f;
            } else {
                // (copies: a choice between the array's elements themselves keeps it in memory, which the compiler puts in
                // LDS and addresses through the dispatch packet -- in host memory, 15 us away for the last workgroups)
                const float lower = alpha[i], upper = alpha[RG > 4 ? 4 + i : 0];
                a = (g4 & 1) ? upper : lower;
            }
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[c][i] *= a;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if constexpr (!AHEAD) {
            // D6: P.V of this step
            static_for<0, NPIECE>([&](auto pp) { pv_piece(pp, pv_operand(decltype(pp)::value / CW)); });
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    uint32_t w_a[KPL][P::NWORDS], w_b[KPL][P::NWORDS];
    uint32_t sc_a[KPL][4 * QO::WPL + 1], sc_b[KPL][4 * QO::WPL + 1];
    while (span.next(shp, seq_lens, wave, lane, &ww)) {
        qg = q_rot + ww.group_id * (P::QS * RG);
        SegmentQueries<P, RG, kDecodeWaves> sq;
        if constexpr (MX) sq.load(shp, ww, wave, lane);
        if constexpr (QJL) j_region = reinterpret_cast<const char *>(qjl) + (PAGED ? 0 : ww.pair * (shp.t_capacity / kWave) * TQ);
        // Addresses are a wave-uniform base (scalar registers) plus a small per-lane byte offset.
        if constexpr (PAGED) {
            k_region = reinterpret_cast<const char *>(cache);
            v_pair = reinterpret_cast<const char *>(v);
        } else {
            k_region = reinterpret_cast<const char *>(cache) + ww.pair * shp.t_capacity * (P::GRANULES * 16);
            v_pair = reinterpret_cast<const char *>(v) + ww.pair * shp.t_capacity * ROWB;
        }
        // The record pointer loses its "read-only, never aliased" provenance here: loads known to be invariant
        // may be moved across any barrier, and the compiler then sinks the prefetch of the next step's records
        // into the (conditional) step that uses them.
        // (not at d = 256: holding the next step's records through a whole step spills registers there)
        if constexpr (AHEAD) {
            const uint64_t bits = reinterpret_cast<uint64_t>(k_region);
            uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits));
            uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bits >> 32));
            asm volatile("" : "+s"(lo), "+s"(hi));
            k_region = reinterpret_cast<const char *>((static_cast<uint64_t>(hi) << 32) | lo);
        }
#pragma unroll
        for (int r = 0; r < RG; ++r) { m_run[r] = -INFINITY; l_lane[r] = 0.0f; }
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

        if (ww.step_begin < ww.step_end) {
            if constexpr (PAGED) {
                int page_first[KPL];
                page_ids(ww.step_begin, page_first);
                page_ids(min(ww.step_begin + ww.step_stride, ww.step_last), page_nxt);
                page_slots(page_first, slot_cur);
                load_records_at(slot_cur, w_a);
                if constexpr (QJL && AHEAD) load_sidecar_at(slot_cur, sc_a);
            } else {
                load_records(ww.step_begin, w_a);
                if constexpr (QJL && AHEAD) load_sidecar(ww.step_begin, sc_a);
            }
        }
        // (the rows of the operand that hold no probabilities stay zero)
#pragma unroll 1
        for (int e = lane; e < 16 * PROW / 8; e += kWave) reinterpret_cast<uint4 *>(&sm.pbuf[wave][0][0])[e] = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (AHEAD) {
            // The first step's P.V pieces multiply zeros by zeros.  The zero values come from loads through an empty descriptor, which move nothing: the wavefront
            // then enters the step loop with the same sequence of outstanding loads as a later iteration has,
            // and the wait counts the compiler derives for the loop are those of the steady state (it takes the
            // stricter of the two ways into the loop).
            const __amdgpu_buffer_rsrc_t v_none = values_of(0, false);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) load_values(v_none, ks, vr[ks]);
        }
        if (!tables_built) {   // workgroup-uniform
            build_tables<P, MX>(sm.tb, tid, kDecodeWaves * kWave);
            tables_built = true;
        }
        // The segment's rotated queries as matrix-core operands.  Every wavefront has left the step loop of the previous
        // segment and read its results (the barriers at its end).
        if constexpr (MX) {
            sq.store(shp, ww, wave, lane, q_rows, QJL ? q2_rows : nullptr);
            __syncthreads();
            build_query_operands<P, RG>(&qop_store[0], q_rows, tid, kDecodeWaves * kWave);
        }
        if constexpr (QJL) {   // ... and the A operands of the residual's correction
            const float *q2s = MX ? &q2_rows[0][0] : q2 + ww.group_id * (RG * D);
            constexpr int ENTRIES = QO::SETS * QO::STEPS * 64;
#pragma unroll 1
            for (int e = tid; e < ENTRIES; e += kDecodeWaves * kWave) {
                const int m = e % 16, g = (e / 16) % 4, st = (e / 64) % QO::STEPS, set = e / (64 * QO::STEPS);
                // query row and part (0 leading, 1 and 2 the remainders) of operand row m
                const int r = RG <= 4 ? m % 4 : m % 8, part = RG <= 4 ? m / 4 : (set == 0 ? m / 8 : (m < 8 ? 2 : 3));
                uint32_t h[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    float x = (r < RG && part < 3) ? q2s[r * D + QO::coordinate(g, st, j)] : 0.0f;
                    h[j] = bf16_rne(x);
                    for (int t = 0; t < part; ++t) {
                        x -= __uint_as_float(h[j] << 16);
                        h[j] = bf16_rne(x);
                    }
                }
                qjl_store[e] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
            }
        }
        if constexpr (MX || QJL) __syncthreads();
        for (int step = ww.step_begin; step < ww.step_end; step += 2 * ww.step_stride) {
            process_step(step, w_a, w_b, sc_a, sc_b);
            if (step + ww.step_stride < ww.step_end) process_step(step + ww.step_stride, w_b, w_a, sc_b, sc_a);
        }
        if constexpr (AHEAD) {   // D6 of the wave's last step
            static_for<0, NPIECE>([&](auto pp) { pv_piece(pp, pv_operand(decltype(pp)::value / CW)); });
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }

        // D7: add the hi and lo partial results (lane groups RP/4 apart); the wavefronts' results are merged in LDS
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float hi = acc[c][i], lo = acc[c][i];
                if constexpr (RP == 4) swap16(hi, lo); else swap32(hi, lo);   // lo: in the lane groups of the hi parts
                acc[c][i] += lo;
            }
        if (g4 < RP / 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    if (i < RG) seg_acc[wave][4 * g4 + i][(c / (LANEB / 2)) * (8 * LANEB) + n16 * (LANEB / 2) + c % (LANEB / 2)] = acc[c][i];
        }
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const float l = wave_sum(l_lane[r]);
            if (lane == 0) {
                seg_ml[wave][r][0] = m_run[r];
                seg_ml[wave][r][1] = l;
            }
        }
        __syncthreads();
        merge_waves<D, RG, kDecodeWaves>(shp, ww, &seg_acc[0][0][0], RG * D, &seg_ml[0][0][0], 2 * RG, part_ml, part_acc, tid);
        __syncthreads();   // (the next segment's queries, or results, take the place)
    }
}

// ---- fp32 values: P.V on the vector ALUs --------------------------------------------------------
// The probabilities go through LDS to a mapping with 8 channels per lane; lanes with the same
// lane / (d / 8) walk the same keys.
template <class P, int RG>
struct DecodeSmemValu {
    DecodeTables<P> tb;
    float pbuf[kDecodeWaves][kWave][RG];
    __attribute__((aligned(16))) float seg_acc[kDecodeWaves][RG][P::D];   // the wavefronts' results at the end of a segment
    float seg_ml[kDecodeWaves][RG][2];
};

// VQ: the values are group-quantised rows (Sec. 4, "value-side group size"; the "value dequantization" of
// Alg. 2): per token [v_bits-bit codes, channel j at bit v_bits * j][per group of v_group channels: fp32
// scale, fp32 zero point], dequantised as zero + scale * code while they are accumulated.
template <class P, int RG, bool VQ = false>
__global__ __launch_bounds__(kDecodeWaves *kWave) void decode_kernel_valu(
    DeviceBooks books, DecodeShape shp, const float *__restrict__ q_rot, const uint4 *__restrict__ cache,
    const float4 *__restrict__ v, const int32_t *__restrict__ seq_lens, float *__restrict__ part_ml,
    float *__restrict__ part_acc, float *__restrict__ scores_out, int v_bits, int v_group) {
    constexpr int D = P::D;
    constexpr int LPR = D / 8;          // lanes per value row (8 channels per lane)
    constexpr int KPL = kWave / LPR;    // value rows per wave-wide load
    extern __shared__ __align__(16) unsigned char smem_raw[];
    DecodeSmemValu<P, RG> &sm = *reinterpret_cast<DecodeSmemValu<P, RG> *>(smem_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    BookLevels<P> levels;
    levels.load(lane);
    WorkSpan<1, kDecodeWaves, false> span;   // (registers to spare)
    span.open(shp, seq_lens, lane);
    if (__builtin_expect(shp.out != nullptr, 0)) zero_empty_pair<D, RG>(shp, seq_lens, tid, kDecodeWaves * kWave);
    if (span.pos >= span.end) return;   // (whole workgroup, before any barrier)
    levels.store(sm.tb, tid);           // (kept in registers until the tables are built they are live through the steps)
    build_tables<P>(sm.tb, tid, kDecodeWaves * kWave);
    const int rl = lane % LPR, ko = lane / LPR;
    WaveWork ww;
    while (span.next(shp, seq_lens, wave, lane, &ww)) {
    const float *qg = q_rot + ww.group_id * (P::QS * RG);
    const uint4 *region = cache + ww.pair * (shp.t_capacity * P::GRANULES);
    const int64_t v_row0 = ww.pair * shp.t_capacity;

    float m_run[RG], l_lane[RG], acc[RG][8];
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        m_run[r] = -INFINITY;
        l_lane[r] = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[r][c] = 0.0f;
    }

    // A step is a tile.  (Nothing of a tile waits for the one before but the running maximum, so two of them in a step, as in the
    // kernel over bf16 values, only made a short call's longest chain twice as long: two / one, one head over 4096
    // tokens 19.7 -> 17.8 us, 8 KV heads of four rows over 1000 26.7 -> 23.1, 2 x 9000 38.8 -> 35.5, 16 x 8192 133.9 -> 133.6.)
    for (int tile = ww.step_begin; tile < ww.step_end; tile += ww.step_stride) {
        const int t0 = tile * kWave;
        const int n_valid = min(kWave, ww.len - t0);
        uint32_t w1[1][P::NWORDS];
        uint32_t (&w)[P::NWORDS] = w1[0];
        const uint4 *src = region + static_cast<int64_t>(tile) * (P::GRANULES * kWave) + lane;
#pragma unroll
        for (int g = 0; g < P::GRANULES; ++g) {
            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
            const u32x4_t x = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + g * kWave));   // streamed
            w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = x.z; w[4 * g + 3] = x.w;
        }
        // VQ: the tile's quantised value words are requested here, so that they arrive during the scores.
        // This lane's 8 channels of a row are 8 * v_bits bits at byte rl * v_bits, fetched as the two aligned
        // words around them (the second may reach into the row's own metadata); rows past the last token
        // are re-reads of the last one (their probabilities are zero).
        constexpr int NIT = VQ ? kWave / KPL : 1;   // key rows per lane and tile
        uint32_t q_lo[NIT], q_hi[NIT];
        float2 q_meta[NIT];
        if constexpr (VQ) {
            const int code_bytes = v_bits * (D / 8);
            const int row_bytes = code_bytes + (D / v_group) * 8;
            const int boff = rl * v_bits;
            const unsigned char *base = reinterpret_cast<const unsigned char *>(v) + (v_row0 + t0) * row_bytes;
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
                const unsigned char *row = base + static_cast<int64_t>(min(i * KPL + ko, n_valid - 1)) * row_bytes;
                const uint32_t *wp = reinterpret_cast<const uint32_t *>(row) + (boff >> 2);
                q_lo[i] = wp[0];
                q_hi[i] = wp[1];
                q_meta[i] = *reinterpret_cast<const float2 *>(row + code_bytes + ((rl * 8) / v_group) * 8);
            }
        }
        // fp32 values: a lane's rows of the tile in batches of VB row loads, the first batch on its way during the scores
        // (one load at a time, each waited for, was most of the kernel: one head over 4096 tokens, 16 -> 14 us with the loads of 16 rows in flight).  Rows past
        // the last token are re-reads of it, replaced by zeros when they are used.
        constexpr int VIT = kWave / KPL;                      // rows per lane and tile
        constexpr int VBATCH = VQ ? 1 : (VIT < 16 ? VIT : 16);
        float4 vbuf[VBATCH][2];
        auto request_rows = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < VBATCH; ++i) {
                const int64_t vrow = v_row0 + t0 + min((i0 + i) * KPL + ko, n_valid - 1);
                vbuf[i][0] = v[vrow * (D / 4) + 2 * rl];
                vbuf[i][1] = v[vrow * (D / 4) + 2 * rl + 1];
            }
        };
        if constexpr (!VQ) {
            request_rows(0);
            asm volatile("" ::: "memory");   // (or the loads are moved to their use)
        }
        float s1[1][RG];
        float (&s)[RG] = s1[0];
        int q_off = 0;
        asm volatile("" : "+s"(q_off));
        tile_scores<P, RG, 1>(w1, qg + q_off, sm.tb, lane, s1);
        const float gamma = __uint_as_float(w[0]);
        const bool valid = lane < n_valid;
#pragma unroll
        for (int r = 0; r < RG; ++r) s[r] = valid ? s[r] * gamma : -INFINITY;
        if (scores_out != nullptr && valid) store_scores<RG>(shp, ww, scores_out, t0 + lane, s);
        float alpha[RG], mx[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) mx[r] = s[r];
        wave_max_of(mx);
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const float m_new = fmaxf(m_run[r], mx[r]);
            alpha[r] = exp2_raw((m_run[r] - m_new) * kLog2e);
            m_run[r] = m_new;
            const float p = exp2_raw((s[r] - m_new) * kLog2e);
            l_lane[r] = fmaf(l_lane[r], alpha[r], p);
            sm.pbuf[wave][lane][r] = p;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[r][c] *= alpha[r];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if constexpr (VQ) {
            const uint32_t mask = (1u << v_bits) - 1u;
            const uint32_t sh = static_cast<uint32_t>((rl * v_bits) & 3);
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
                const int key = i * KPL + ko;           // probabilities of lanes past n_valid are zero
                float pv[RG];
#pragma unroll
                for (int r = 0; r < RG; ++r) pv[r] = sm.pbuf[wave][key][r];
                const uint32_t bits = __builtin_amdgcn_alignbyte(q_hi[i], q_lo[i], sh);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float val = fmaf(q_meta[i].x, static_cast<float>((bits >> (c * v_bits)) & mask), q_meta[i].y);
#pragma unroll
                    for (int r = 0; r < RG; ++r) acc[r][c] = fmaf(pv[r], val, acc[r][c]);
                }
            }
        } else {
#pragma unroll
            for (int i0 = 0; i0 < VIT; i0 += VBATCH) {
                if (i0 > 0) request_rows(i0);
#pragma unroll
                for (int i = 0; i < VBATCH; ++i) {
                    const int key = (i0 + i) * KPL + ko;
                    float pv[RG];
#pragma unroll
                    for (int r = 0; r < RG; ++r) pv[r] = sm.pbuf[wave][key][r];
                    const float4 a = vbuf[i][0], b = vbuf[i][1];
                    const bool in = key < n_valid;
                    const float vals[8] = {in ? a.x : 0.0f, in ? a.y : 0.0f, in ? a.z : 0.0f, in ? a.w : 0.0f,
                                           in ? b.x : 0.0f, in ? b.y : 0.0f, in ? b.z : 0.0f, in ? b.w : 0.0f};
#pragma unroll
                    for (int r = 0; r < RG; ++r)
#pragma unroll
                        for (int c = 0; c < 8; ++c) acc[r][c] = fmaf(pv[r], vals[c], acc[r][c]);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // D7: fold the KPL lane groups; the wavefronts' results are merged in LDS
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[r][c] += __shfl_xor(acc[r][c], o, kWave);
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        const float l = wave_sum(l_lane[r]);
        if (lane == 0) { sm.seg_ml[wave][r][0] = m_run[r]; sm.seg_ml[wave][r][1] = l; }
        if (ko == 0) {
#pragma unroll
            for (int c = 0; c < 8; ++c) sm.seg_acc[wave][r][rl * 8 + c] = acc[r][c];
        }
    }
    __syncthreads();
    merge_waves<D, RG, kDecodeWaves>(shp, ww, &sm.seg_acc[0][0][0], RG * D, &sm.seg_ml[0][0][0], 2 * RG, part_ml, part_acc, tid);
    __syncthreads();
    }   // segments
}

// ---- launch helpers -----------------------------------------------------------------------------
template <class P>
int launch_decode_mq(const octopus_codebooks_t &cb, const DecodeShape &s, const void *cache, const void *v,
                     const int32_t *seq_lens, float *part_ml, float *part_acc, hipStream_t stream,
                     PageTable pt = PageTable{nullptr, 0, 0});   // pt: cache and v are pools of pages

// bf16 values: the matrix-core kernels.  SCORES: the instantiation that also writes the scores (built in
// a translation unit of its own).
template <class P, int RG, bool SCORES>
int launch_decode_mfma_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                          const void *v, const int32_t *seq_lens, float *part_ml, float *part_acc, float *scores_out,
                          hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    // one workgroup per compute unit; they share the steps of the call
    hipLaunchKernelGGL((decode_kernel_mfma<P, RG, SCORES, false>), dim3(kDecodeWorkgroups), dim3(kDecodeWaves * kWave),
                       0, stream, books, s, q_rot, static_cast<const uint4 *>(cache), static_cast<const uint32_t *>(v),
                       seq_lens, part_ml, part_acc, scores_out, nullptr, nullptr, nullptr, 0, 0);
    return static_cast<int>(hipGetLastError());
}

// Row groups of one and two rows that the host shapes a call for (least_rows in octopus_host.cpp); those of four and eight
// are built for every plan.
template <class P, bool QJL = false>
constexpr bool row_group_built(int rows) {
    return rows >= 4 || mx_scores<P>() || P::D > 128 || (P::D == 64 && (rows == 1 || !QJL));
}

// Paged pools (bf16 values, row groups of at most 8 rows).
template <class P, int RG>
int launch_decode_paged_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *k_pool,
                           const void *v_pool, const PageTable &pt, const int32_t *seq_lens, float *part_ml,
                           float *part_acc, hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    hipLaunchKernelGGL((decode_kernel_mfma<P, RG, false, false, true>), dim3(kDecodeWorkgroups),
                       dim3(kDecodeWaves * kWave), 0, stream, books, s, q_rot, static_cast<const uint4 *>(k_pool),
                       static_cast<const uint32_t *>(v_pool), seq_lens, part_ml, part_acc, nullptr, nullptr,
                       nullptr, pt.table, pt.stride, pt.n_pages);
    return static_cast<int>(hipGetLastError());
}

template <class P>
int launch_decode_paged_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                             const void *k_pool, const void *v_pool, const PageTable &pt, const int32_t *seq_lens,
                             float *part_ml, float *part_acc, hipStream_t stream) {
    switch (s.rows_per_pass) {
        case 1: if constexpr (row_group_built<P>(1)) return launch_decode_paged_rg<P, 1>(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream); break;
        case 2: if constexpr (row_group_built<P>(2)) return launch_decode_paged_rg<P, 2>(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream); break;
        case 4: return launch_decode_paged_rg<P, 4>(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 8: return launch_decode_paged_rg<P, 8>(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 128:
        case 256:
        case 512:   // the many-row kernel (d <= 128), which takes the page table as an argument
            if constexpr (P::D <= 128) return launch_decode_mq<P>(cb, s, k_pool, v_pool, seq_lens, part_ml, part_acc, stream, pt);
            return static_cast<int>(hipErrorInvalidValue);
        default: break;
    }
    return static_cast<int>(hipErrorInvalidValue);   // (a row group that is not built)
}

// Paged pools with the QJL side-car in pages as well (a pool of [page][KV head] side-car tiles).
template <class P, int RG>
int launch_decode_paged_qjl_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                               const void *k_pool, const void *qjl_pool, const float *q2, const void *v_pool,
                               const PageTable &pt, const int32_t *seq_lens, float *part_ml, float *part_acc,
                               hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    hipLaunchKernelGGL((decode_kernel_mfma<P, RG, true, true, true>), dim3(kDecodeWorkgroups),
                       dim3(kDecodeWaves * kWave), 0, stream, books, s, q_rot, static_cast<const uint4 *>(k_pool),
                       static_cast<const uint32_t *>(v_pool), seq_lens, part_ml, part_acc, nullptr,
                       static_cast<const unsigned char *>(qjl_pool), q2, pt.table, pt.stride, pt.n_pages);
    return static_cast<int>(hipGetLastError());
}

template <class P>
int launch_decode_paged_qjl_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                                 const void *k_pool, const void *qjl_pool, const float *q2, const void *v_pool,
                                 const PageTable &pt, const int32_t *seq_lens, float *part_ml, float *part_acc,
                                 hipStream_t stream) {
    switch (s.rows_per_pass) {
        case 1: if constexpr (row_group_built<P, true>(1)) return launch_decode_paged_qjl_rg<P, 1>(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream); break;
        case 2: if constexpr (row_group_built<P, true>(2)) return launch_decode_paged_qjl_rg<P, 2>(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream); break;
        case 4: return launch_decode_paged_qjl_rg<P, 4>(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 8: return launch_decode_paged_qjl_rg<P, 8>(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        default: break;
    }
    return static_cast<int>(hipErrorInvalidValue);
}

template <class P, bool SCORES>
int launch_decode_mfma_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                            const void *cache, const void *v, const int32_t *seq_lens, float *part_ml,
                            float *part_acc, float *scores_out, hipStream_t stream) {
    if ((scores_out != nullptr) != SCORES) return static_cast<int>(hipErrorInvalidValue);
    switch (s.rows_per_pass) {
        case 1: return launch_decode_mfma_rg<P, 1, SCORES>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 2: return launch_decode_mfma_rg<P, 2, SCORES>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 4: return launch_decode_mfma_rg<P, 4, SCORES>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 8: return launch_decode_mfma_rg<P, 8, SCORES>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 128:
        case 256:
        case 512:   // the many-row kernel: rows per workgroup
            if constexpr (P::D <= 128 && !SCORES)
                return launch_decode_mq<P>(cb, s, cache, v, seq_lens, part_ml, part_acc, stream);
            return static_cast<int>(hipErrorInvalidValue);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

// fp32 values: P.V on the vector units
template <class P, int RG>
int launch_decode_valu_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                          const void *v, const int32_t *seq_lens, float *part_ml, float *part_acc, float *scores_out,
                          hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    const size_t smem = sizeof(DecodeSmemValu<P, RG>);
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(&decode_kernel_valu<P, RG>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem));
    if (err != hipSuccess) return static_cast<int>(err);
    hipLaunchKernelGGL((decode_kernel_valu<P, RG>), dim3(kDecodeWorkgroups), dim3(kDecodeWaves * kWave), smem, stream,
                       books, s, q_rot, static_cast<const uint4 *>(cache), static_cast<const float4 *>(v), seq_lens,
                       part_ml, part_acc, scores_out, 0, 0);
    return static_cast<int>(hipGetLastError());
}

template <class P>
int launch_decode_valu_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                            const void *cache, const void *v, const int32_t *seq_lens, float *part_ml,
                            float *part_acc, float *scores_out, hipStream_t stream) {
    switch (s.rows_per_pass) {
        case 1: return launch_decode_valu_rg<P, 1>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 2: return launch_decode_valu_rg<P, 2>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 4: return launch_decode_valu_rg<P, 4>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 8: return launch_decode_valu_rg<P, 8>(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

// Decode attention over group-quantised values.
template <class P, int RG>
int launch_decode_vq_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                        const void *vq, int v_bits, int v_group, const int32_t *seq_lens, float *part_ml,
                        float *part_acc, float *scores_out, hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    const size_t smem = sizeof(DecodeSmemValu<P, RG>);
    hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(&decode_kernel_valu<P, RG, true>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem));
    if (err != hipSuccess) return static_cast<int>(err);
    hipLaunchKernelGGL((decode_kernel_valu<P, RG, true>), dim3(kDecodeWorkgroups), dim3(kDecodeWaves * kWave), smem,
                       stream, books, s, q_rot, static_cast<const uint4 *>(cache), static_cast<const float4 *>(vq),
                       seq_lens, part_ml, part_acc, scores_out, v_bits, v_group);
    return static_cast<int>(hipGetLastError());
}

template <class P>
int launch_decode_vq_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                          const void *vq, int v_bits, int v_group, const int32_t *seq_lens, float *part_ml,
                          float *part_acc, float *scores_out, hipStream_t stream) {
    switch (s.rows_per_pass) {
        case 1: return launch_decode_vq_rg<P, 1>(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream);
        case 2: return launch_decode_vq_rg<P, 2>(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream);
        case 4: return launch_decode_vq_rg<P, 4>(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream);
        case 8: return launch_decode_vq_rg<P, 8>(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

// bf16 values with the QJL residual.
template <class P, int RG>
int launch_decode_qjl_rg(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                         const void *qjl, const float *q2, const void *v, const int32_t *seq_lens, float *part_ml,
                         float *part_acc, float *scores_out, hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    hipLaunchKernelGGL((decode_kernel_mfma<P, RG, true, true>), dim3(kDecodeWorkgroups),
                       dim3(kDecodeWaves * kWave), 0, stream, books, s, q_rot, static_cast<const uint4 *>(cache),
                       static_cast<const uint32_t *>(v), seq_lens, part_ml, part_acc, scores_out,
                       static_cast<const unsigned char *>(qjl), q2, nullptr, 0, 0);
    return static_cast<int>(hipGetLastError());
}

template <class P>
int launch_decode_qjl_plan(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot,
                           const void *cache, const void *qjl, const float *q2, const void *v,
                           const int32_t *seq_lens, float *part_ml, float *part_acc, float *scores_out,
                           hipStream_t stream) {
    switch (s.rows_per_pass) {
        case 1: if constexpr (row_group_built<P, true>(1)) return launch_decode_qjl_rg<P, 1>(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream); break;
        case 2: if constexpr (row_group_built<P, true>(2)) return launch_decode_qjl_rg<P, 2>(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream); break;
        case 4: return launch_decode_qjl_rg<P, 4>(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 8: return launch_decode_qjl_rg<P, 8>(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream);
        default: break;
    }
    return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace octopus

#endif
