// Decode attention for many query rows per KV head (a chunk of queries against the whole cache, e.g. the
// 3600 queries of a video frame): Alg. 2 with the roles of a dense attention kernel.  Here the work per
// key is a dense contraction over hundreds of rows, so both products run on the matrix cores; the keys
// are still decoded on the fly from the packed records, once per block of 128, 256 or 512 query rows, into an LDS
// tile and never reach memory.
//
// A workgroup of 4 or 8 wavefronts owns 128, 256 or 512 query rows of one (sequence, KV head) (one or two blocks of 32 per
// wavefront) and a range of 64-token tiles.  Per tile:
//   * stage (all wavefronts, one tile ahead, double-buffered LDS): lane = key; the record is unpacked,
//     gamma * rho^ * n^ is looked up and multiplied, split into two bf16 numbers (hi = upper 16 bits,
//     lo = the rest) and written to the key tile [key][coordinate]; the values of the tile are written
//     transposed [channel][key];
//   * S^T = K^ Q^T (keys x rows) with v_mfma_f32_32x32x16_bf16, three products per k-step (hi hi, hi lo,
//     lo hi: relative error below 2^-16); a lane then holds 32 scores of ONE query row, so the softmax
//     statistics of a row live in one lane (and its partner lane + 32);
//   * O^T += V^T P^T (channels x rows): the probabilities go from the accumulators of the first product
//     straight into the B operand of the second (k-slot j of lane group h is key 4h + j, or 8 + 4h + j - 4
//     for j >= 4, of each group of 16 keys, which is how the first product left them), again as hi + lo.
// The partial (m, l, acc) of each row goes to the split-K workspace and through the same merge kernel as
// the single-query path.
#ifndef OCTOPUS_DECODE_MQ_HPP_
#define OCTOPUS_DECODE_MQ_HPP_

#include "octopus_decode.hpp"

namespace octopus {

// Query rows per workgroup: NW = 4 wavefronts (128 rows) or NW = 8 (256 rows, two wavefronts per SIMD within 256 registers
// each), RB = 1 or (d = 64, 512 rows) 2 blocks of 32 rows per wavefront, one after the other on each tile.  The keys of a tile
// are decoded once per workgroup, so more rows mean less decoding; the host picks what the call is fastest with
// (many_rows_splits).
// 512 rows: a tile takes 4.1 us, two of 256 rows 4.5 (3600 queries x 24 heads, 75600 tokens, b = 4: 3930 -> 3710 us; 800 x 24, 9000
// tokens 169 -> 144).  Tried and slower: the blocks interleaved so that one's scores are computed during the other's exponentials
// (registers: 6300 us and more), the remainders of the queries in LDS (4220), the two blocks sharing each read of keys and values, 32
// keys at a time (3700: the reads are not what bounds it), last blocks of few rows started after all others (3950).
// What bounds it: the issue of products and vector instructions.  On one SIMD, per wavefront of several, 64 multiply-adds take 152
// cycles, 64 exponentials 520, 8 products 256, and the products with the multiply-adds 306: a product keeps others from issuing for
// about 19 of its 32 cycles.  Per tile and 32 rows a wavefront issues 40 products, 32 exponentials, 150 other vector instructions
// and 85 - 100 for staging, shared by its blocks: 40 x 19 + 32 x 8 + 245 x 2.4 cycles, 3200 for 256 rows by two wavefronts per SIMD, of the
// 4500 that a tile takes (2.25 us; the clock falls to about 2 GHz under this load: busy cycles over the kernel's time).  Three wavefronts per SIMD (384 rows by twelve, 160 registers) take as long per row as 512 rows, so
// it is not latency; the way down is fewer vector instructions per score.

typedef __attribute__((ext_vector_type(16))) float f32x16_t;
constexpr uint32_t kXcds = 8;   // accelerator dies of the chip; consecutive workgroups go to consecutive dies

template <class P>
struct MqSmem {
    static constexpr int D = P::D;
    static constexpr int KST = D + 8;       // bf16 per row of the key tile: 16-byte reads of 8 lanes hit 8 bank groups
    static constexpr int VST = kWave + 4;   // bf16 per row of the transposed value tile (8-byte aligned rows)
    float4 dir0[1 << (2 * P::BD0)];
    float4 dir1[P::NCLASS == 2 ? 1 << (2 * P::BD1) : 1];
    float c_xi[2][kMaxLevels];
    float c_rho[2][kMaxLevels];
    uint16_t kh[2][kWave][KST];
    uint16_t kl[2][kWave][KST];
    uint16_t vt[2][D][VST];
};

// Which work a workgroup has.  The blocks of rows of one (sequence, KV head, split), a unit, read the same keys and values: they follow
// each other in the order of the work, and each accelerator die (workgroup b runs on die b % 8, each with its own L2) takes an
// eighth of that order, so that the tiles are fetched from memory once and not once per die, and no die has more workgroups than an
// eighth of them, rounded up.  (Whole units of blocks per die before: 23 units of 11 blocks were two rounds of workgroups on seven dies of 32
// compute units; 2776 rows of one KV head over 22097 tokens, d = 64, 87 us of this kernel.)
__host__ __device__ inline uint32_t mq_position(uint32_t workgroup, uint32_t n_work) {
    return (workgroup % kXcds) * ((n_work + kXcds - 1) / kXcds) + workgroup / kXcds;
}
struct MqWork {
    uint32_t pair, split, grp;   // pair: sequence n_kv_heads + KV head
};
// In a row, a die has whole sequences, and with sequences of different lengths some dies have most of the tiles (24 KV heads of 528 rows
// over 4376 and 226 tokens, d = 128, b = 4, took 198 us, as long as over twice 4376).  So the order may take every eighth pair, then every
// eighth from the next one on: a die has pairs of every sequence.  With fewer KV heads than dies it takes the units so, and as the first
// splits of a short sequence have its tiles, the splits of a pair are turned so that its first goes to another die than its neighbours'.
// Whole units per die, by unit % 8 / in a row / spread: that call 164 / 198 / 119 us, 16 ragged to 1167, 24 KV heads x 48, d = 128, b = 4 150 / 111 /
// 85, d = 64, 16 ragged to 8000, 8 x 64 85 / 82 / 69, 32 to 4000 93 / 83 / 69, 8 to 6000, 4 KV heads x 512, d = 128 128 / 114 / 106.
// What it costs is that a die reads from every sequence, 1 - 2 us.  That is more than it gives where every workgroup has a compute unit of
// its own and few tiles (d = 64, 16 ragged to 6352, one KV head of 196 rows 27.9 in a row / 30.3, d = 128, 5 to 3697, 2 x 238 32.4 / 34.3), from
// about 16 tiles on it is less; of equal sequences in more than one round it is up to 3 % (d = 64, 16 x 105, 24 KV heads of 222 rows 58.5 / 60.1).
__host__ __device__ inline bool mq_spreads(int32_t n_seq, int32_t n_splits, int32_t max_len, uint32_t n_work) {
    return n_seq > 1 && (n_work > 256 || max_len / n_splits >= 16 * kWave);
}
// Every eighth of 0 .. n - 1, then every eighth from the next one on: number i of that order.
__host__ __device__ inline uint32_t mq_spread(uint32_t i, uint32_t n) {
    const uint32_t each = n / kXcds, more = n % kXcds;   // numbers of a residue, residues with one more
    if (i < more * (each + 1)) {
        const uint32_t residue = i / (each + 1);
        return kXcds * (i - residue * (each + 1)) + residue;
    }
    const uint32_t rest = i - more * (each + 1), residue = rest / each;
    return kXcds * (rest - residue * each) + more + residue;
}
__host__ __device__ inline MqWork mq_work(uint32_t position, uint32_t n_seq, uint32_t n_kv_heads, uint32_t n_splits, uint32_t n_row_groups,
                                          bool spread) {
    const uint32_t i = position / n_row_groups, grp = position - i * n_row_groups, n_pairs = n_seq * n_kv_heads;
    uint32_t pair = i / n_splits, split = i - pair * n_splits;
    if (spread) {
        if (n_kv_heads >= kXcds) {
            pair = mq_spread(pair, n_pairs);
        } else {
            const uint32_t unit = mq_spread(i, n_pairs * n_splits);
            pair = unit / n_splits;
            const uint32_t at = unit - pair * n_splits;
            const uint32_t turn = n_splits >= kXcds ? (pair * (1u - n_splits)) % kXcds : (pair * n_splits / kXcds) % n_splits;
            split = at >= turn ? at - turn : at + n_splits - turn;
        }
    }
    return MqWork{pair, split, grp};
}

template <class P, int NW, int RB>
__global__ __launch_bounds__(kWave *NW) __attribute__((amdgpu_waves_per_eu(P::D <= 64 || NW == 8 ? 2 : 1))) void decode_kernel_mq(DeviceBooks books, DecodeShape shp,
                                                         const uint4 *__restrict__ cache,
                                                         const uint16_t *__restrict__ v,
                                                         const int32_t *__restrict__ seq_lens,
                                                         float *__restrict__ part_ml, float *__restrict__ part_acc,
                                                         PageTable pt) {
    // pt.table (or NULL): `cache` and `v` are pools of 64-token pages, [page][KV head] each a key tile and 64 value
    // rows; logical tile j of sequence s lives in page pt.table[s * pt.stride + j] (clamped to the pool)
    constexpr int D = P::D;
    constexpr int KK = D / 16;               // k-steps of the score product
    constexpr int NB = D / 32;               // 32-channel blocks of the output
    constexpr int ROWB = D * 2;              // bytes per value row
    constexpr int TILEB = P::GRANULES * kWave * 16;
    constexpr int ROWS = 32 * NW * RB;       // query rows per workgroup: row 32 (NW b + w) + n is row n of wavefront w's block b
    constexpr bool REF_BY_PRODUCT = RB == 2;
    constexpr int VP = D / 8 / NW;           // 16-byte value pieces per thread and tile
    using S = MqSmem<P>;
    __shared__ S sm;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;

    // work: (sequence, KV head, block of ROWS rows, split) and the split's tiles
    const uint32_t n_work = static_cast<uint32_t>(shp.n_seq * shp.n_kv_heads) * static_cast<uint32_t>(shp.n_splits * shp.n_row_groups);
    const uint32_t work = mq_position(blockIdx.x, n_work);
    if (work >= n_work) return;   // (whole workgroup, before any barrier)
    const MqWork mine = mq_work(work, static_cast<uint32_t>(shp.n_seq), static_cast<uint32_t>(shp.n_kv_heads), static_cast<uint32_t>(shp.n_splits),
                                static_cast<uint32_t>(shp.n_row_groups), mq_spreads(shp.n_seq, shp.n_splits, shp.max_len, n_work));
    const int grp = static_cast<int>(mine.grp), split = static_cast<int>(mine.split);
    const int64_t pair = mine.pair;
    const int seq = static_cast<int>(mine.pair / static_cast<uint32_t>(shp.n_kv_heads));
    const int kvh = static_cast<int>(mine.pair % static_cast<uint32_t>(shp.n_kv_heads));
    const int len = min(max(seq_lens[seq], 0), shp.max_len);
    const int n_tiles = (len + kWave - 1) / kWave;
    const int base = n_tiles / shp.n_splits, rem = n_tiles % shp.n_splits;
    const int tile_begin = split * base + min(split, rem);
    const int tile_end = tile_begin + base + (split < rem ? 1 : 0);
    if (tile_begin >= tile_end) return;   // (a split past the sequence's last tile: nothing of it is written, and the merge does not read it)

    const bool paged = pt.table != nullptr;
    const char *k_region = reinterpret_cast<const char *>(cache) + (paged ? 0 : pair * shp.t_capacity * (P::GRANULES * 16));
    const char *v_pair = reinterpret_cast<const char *>(v) + (paged ? 0 : pair * shp.t_capacity * ROWB);

    // Q^T operands of this wave's 32 rows: lane (n, h) holds coordinates 16 kk + 8 h .. + 8 of row n as bf16 hi and lo.
    union BF8 { uint32_t u[4]; bf16x8_t b; };
    BF8 qh[RB][KK], ql[RB][KK];
    // The rows are asked for here and rotated in place (rotate_queries below).
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    u32x4_t q_raw[KK], q_more[KK];   // bf16 queries: the words of q_raw, two each
    uint32_t q_neg[KK];
    const int q_row = grp * ROWS + wave * 32 + n;
    // blocks of this wavefront that have rows: the others' products are left out
    const int live = __builtin_amdgcn_readfirstlane(min(RB, (max(shp.rows_per_kv - grp * ROWS - wave * 32, 0) + 32 * NW - 1) / (32 * NW)));
    auto load_queries = [&](int rb) __attribute__((always_inline)) {
        typedef uint32_t u32x4a_t __attribute__((ext_vector_type(4), aligned(4)));   // (queries are aligned to 4 bytes)
        const int row = min(q_row + 32 * NW * rb, shp.rows_per_kv - 1);
        const int qi = row / shp.heads_per_kv, head = kvh * shp.heads_per_kv + row % shp.heads_per_kv;
        const int64_t base_q = ((static_cast<int64_t>(seq) * shp.n_q + qi) * shp.n_q_heads + head) * D + 8 * h;
        const int es = shp.q_is_bf16 ? 2 : 4, second = shp.q_is_bf16 ? 0 : 16;   // (one path: the arrays written by two are kept in scratch memory)
        const char *src = static_cast<const char *>(shp.q) + base_q * es;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            q_raw[kk] = *reinterpret_cast<const u32x4a_t *>(src + 16 * kk * es);
            q_more[kk] = *reinterpret_cast<const u32x4a_t *>(src + 16 * kk * es + second);
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) q_neg[kk] = shp.signs[kvh * (D / 8) + 2 * kk + h];
    };
    // q_rot = scale H (s . q) of the 32 rows at once, all in registers (the same additions as rotate_queries_kernel's: the
    // butterflies of the element index's bits in ascending order, bit 3 is the lane's half).  The rotation was a launch of its own whose
    // 4-byte stores lay ROWS x 4 bytes apart: 53 us of 4005 for 3600 queries x 24 heads at d = 64, 19 of 325 for 509 x 32 at d = 128.
    auto rotate_queries = [&](auto block) __attribute__((always_inline)) {
        constexpr int rb = decltype(block)::value;
        float x[KK][8];
        const bool there = q_row + 32 * NW * rb < shp.rows_per_kv;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const u32x4_t lower = q_raw[kk], upper = q_more[kk];
                const uint32_t pair_word = lower[e / 2], own_word = e < 4 ? lower[e & 3] : upper[e & 3];
                const uint32_t bits = shp.q_is_bf16 ? ((e & 1) ? pair_word & 0xffff0000u : pair_word << 16) : own_word;
                x[kk][e] = there ? __uint_as_float(bits ^ ((q_neg[kk] << (31 - e)) & 0x80000000u)) : 0.0f;
            }
#pragma unroll
        for (int m = 1; m < 8; m <<= 1)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if ((e & m) == 0) {
                        const float a = x[kk][e], b = x[kk][e | m];
                        x[kk][e] = a + b;
                        x[kk][e | m] = a - b;
                    }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                float a = x[kk][e], b = x[kk][e + 1];
                swap32(a, b);                       // a: lower halves' of elements e | e + 1, b: the upper halves'
                float sum = a + b, diff = a - b;
                swap32(sum, diff);
                x[kk][e] = sum;
                x[kk][e + 1] = diff;
            }
#pragma unroll
        for (int m = 1; m < KK; m <<= 1)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
                if ((kk & m) == 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float a = x[kk][e], b = x[kk | m][e];
                        x[kk][e] = a + b;
                        x[kk | m][e] = a - b;
                    }
                }
        const float norm = shp.scale * (D == 64 ? 0.125f : 0.08838834764831845f);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // (in units of log2: the scores come out as exponents of two)
                const float a = x[kk][2 * e] * norm * kLog2e, b = x[kk][2 * e + 1] * norm * kLog2e;
                const uint32_t ab = __float_as_uint(a), bb = __float_as_uint(b);
                qh[rb][kk].u[e] = __builtin_amdgcn_perm(bb, ab, 0x07060302u);
                const float al = a - __uint_as_float(ab & 0xffff0000u), bl = b - __uint_as_float(bb & 0xffff0000u);
                ql[rb][kk].u[e] = __builtin_amdgcn_perm(__float_as_uint(bl), __float_as_uint(al), 0x07060302u);
            }
    };

    // ---- staging: global -> registers -> LDS tile ---------------------------------------------------
    uint32_t w[P::NWORDS];          // this lane's record of the tile being staged
    uint4 vp[VP];                   // its value pieces: key `lane`, channels 8 (wave + NW i) .. + 8
    auto load_tile = [&](int tile) __attribute__((always_inline)) {
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
        constexpr int USED = (P::RECORD_BYTES + 3) / 4;
        // position of the tile in the cache (in tiles): the logical tile, or its page's tile of this KV head
        int64_t slot = tile;
        if (paged) {
            const int page = pt.table[static_cast<int64_t>(seq) * pt.stride + tile];
            slot = static_cast<int64_t>(min(max(page, 0), pt.n_pages - 1)) * shp.n_kv_heads + kvh;
        }
        const char *src = k_region + slot * TILEB + lane * 16;
#pragma unroll
        for (int g = 0; g < P::GRANULES; ++g) {
            const char *gp = src + g * (kWave * 16);
            const int nw = (USED - 4 * g) < 4 ? (USED - 4 * g) : 4;
            if (nw == 4) {
                const uint4 x = *reinterpret_cast<const uint4 *>(gp);
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = x.z; w[4 * g + 3] = x.w;
            } else if (nw == 3) {
                const u32x3_t x = *reinterpret_cast<const u32x3_t *>(gp);
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = x.z; w[4 * g + 3] = 0u;
            } else if (nw == 2) {
                const u32x2_t x = *reinterpret_cast<const u32x2_t *>(gp);
                w[4 * g] = x.x; w[4 * g + 1] = x.y; w[4 * g + 2] = 0u; w[4 * g + 3] = 0u;
            } else {
                w[4 * g] = *reinterpret_cast<const uint32_t *>(gp);
                w[4 * g + 1] = 0u; w[4 * g + 2] = 0u; w[4 * g + 3] = 0u;
            }
        }
        // value rows past the sequence's end are replaced by its last row (their probabilities are zero)
        // (that row is in the same tile, hence in the same page)
        const int row = min(tile * kWave + lane, len - 1);
        const char *vrow = v_pair + (slot * kWave + (row - tile * kWave)) * ROWB;
#pragma unroll
        for (int i = 0; i < VP; ++i) vp[i] = *reinterpret_cast<const uint4 *>(vrow + (wave + NW * i) * 16);
    };
    // Wave wv writes the coordinates [wv * D / NW, (wv + 1) * D / NW) of its lane's key: it decodes the triplets
    // that cover them (one or two of them are decoded by the neighbouring wave as well) and writes whole
    // 16-byte pieces of the key tile.  (Two-byte writes, one per coordinate, land on 8 banks for the 64 lanes
    // of a wavefront and were a third of this kernel's time.)
    auto stage_block = [&](auto ww, int buf) __attribute__((always_inline)) {
        constexpr int wv = decltype(ww)::value;
        constexpr int CW = D / NW;                      // coordinates per wave: D / 4 or D / 8 (8, 16 or 32)
        constexpr int T_LO = (wv * CW) / 3, T_HI = ((wv + 1) * CW - 1) / 3;
        constexpr int NT = T_HI - T_LO + 1;
        float val[3 * NT];
        static_for<0, NT>([&](auto jj) {
            constexpr int i = T_LO + decltype(jj)::value;
            constexpr int c = P::cls(i);
            constexpr int bd = P::bdir(i), bn = P::bnrm(i);
            const uint32_t code = field<P::dir_bit(i), 2 * bd>(w);
            const uint32_t nrm = field<P::nrm_bit(i), bn>(w);
            const float4 dir = (c ? sm.dir1 : sm.dir0)[code];
            const float g = __uint_as_float(w[0]) * sm.c_rho[c][nrm];
            val[3 * decltype(jj)::value] = g * dir.x;
            val[3 * decltype(jj)::value + 1] = g * dir.y;
            val[3 * decltype(jj)::value + 2] = g * dir.z;
        });
#pragma unroll
        for (int g8 = 0; g8 < CW / 8; ++g8) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = wv * CW + 8 * g8 + 2 * k - 3 * T_LO;      // index into val of the pair's first value
                const uint32_t b0 = __float_as_uint(val[j]), b1 = __float_as_uint(val[j + 1]);
                const float l0 = val[j] - __uint_as_float(b0 & 0xffff0000u);
                const float l1 = val[j + 1] - __uint_as_float(b1 & 0xffff0000u);
                hi[k] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                lo[k] = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
            }
            *reinterpret_cast<uint4 *>(&sm.kh[buf][lane][wv * CW + 8 * g8]) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4 *>(&sm.kl[buf][lane][wv * CW + 8 * g8]) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
    };
    auto stage_tile = [&](int buf) __attribute__((always_inline)) {
        switch (wave) {
            case 0: stage_block(std::integral_constant<int, 0>{}, buf); break;
            case 1: stage_block(std::integral_constant<int, 1>{}, buf); break;
            case 2: stage_block(std::integral_constant<int, 2>{}, buf); break;
            case 3: stage_block(std::integral_constant<int, 3>{}, buf); break;
            default:
                if constexpr (NW == 8) {
                    switch (wave) {
                        case 4: stage_block(std::integral_constant<int, 4>{}, buf); break;
                        case 5: stage_block(std::integral_constant<int, 5>{}, buf); break;
                        case 6: stage_block(std::integral_constant<int, 6>{}, buf); break;
                        default: stage_block(std::integral_constant<int, 7>{}, buf); break;
                    }
                }
                break;
        }
#pragma unroll
        for (int i = 0; i < VP; ++i) {
            const int c0 = (wave + NW * i) * 8;
            const uint32_t x[4] = {vp[i].x, vp[i].y, vp[i].z, vp[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sm.vt[buf][c0 + 2 * e][lane] = static_cast<uint16_t>(x[e] & 0xffffu);
                sm.vt[buf][c0 + 2 * e + 1][lane] = static_cast<uint16_t>(x[e] >> 16);
            }
        }
    };

    // The row's reference exponent: probabilities are 2^(score - m_ref).  Its negative is what the first product's
    // accumulators start from, so the scores arrive with the subtraction done; it is moved (and everything summed so far
    // rescaled) only when a score exceeds it by more than kHeadroom, which after the first tile is rare: a probability may
    // then be up to 2^kHeadroom, which floating point does not mind.
    constexpr float kHeadroom = 8.0f;
    float m_ref[RB], l_run[RB];
    f32x16_t oacc[RB][NB];
    f32x16_t c_ref[REF_BY_PRODUCT ? 1 : RB];
    // REF_BY_PRODUCT: 16 registers a block are too many; the accumulators start from a product of ones with three bf16 numbers
    // that add up to the reference (24 bits: exactly), in its first slots.
    BF8 minus_ref[RB], ones;
#pragma unroll
    for (int k = 0; k < 4; ++k) ones.u[k] = h == 0 ? (k == 0 ? 0x3f803f80u : (k == 1 ? 0x00003f80u : 0u)) : 0u;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_ref[rb] = l_run[rb] = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) minus_ref[rb].u[k] = 0u;
        if constexpr (!REF_BY_PRODUCT) {
#pragma unroll
            for (int e = 0; e < 16; ++e) c_ref[rb][e] = 0.0f;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[rb][nb][e] = 0.0f;
    }

    // Start: queries and first tile are asked for, then the tables (one copy: the lookups are a small part of this kernel) are
    // built and the queries rotated.
    load_queries(0);
    load_tile(tile_begin);
    if (wave < 4) {   // a level per lane, of one array per wavefront
        typedef const float __attribute__((address_space(4))) *arg_t;
        static_assert(kMaxLevels == kWave && offsetof(DeviceBooks, c_rho) == offsetof(DeviceBooks, c_xi) + 2 * kMaxLevels * sizeof(float), "four arrays in a row");
        const float level = ((arg_t)__builtin_amdgcn_kernarg_segment_ptr())[offsetof(DeviceBooks, c_xi) / 4 + wave * kMaxLevels + lane];
        (wave < 2 ? sm.c_xi[wave] : sm.c_rho[wave - 2])[lane] = level;
    }
    __syncthreads();
    build_dir_lut<P::BD0>(sm.dir0, sm.c_xi[0], tid, kWave * NW);
    if constexpr (P::NCLASS == 2) build_dir_lut<P::BD1>(sm.dir1, sm.c_xi[1], tid, kWave * NW);
    rotate_queries(std::integral_constant<int, 0>{});
    if constexpr (RB == 2) {
        load_queries(1);
        rotate_queries(std::integral_constant<int, 1>{});
    }
    __syncthreads();                       // tables complete
    stage_tile(0);
    load_tile(min(tile_begin + 1, tile_end - 1));
    __syncthreads();

    // With 8 wavefronts (two per SIMD: w and w + 4) the upper four stage the next tile BEFORE they work on
    // the current one, the lower four after: the two wavefronts of a SIMD are then in opposite phases, one
    // on the matrix cores while the other decodes keys on the vector units.
    const bool stage_first = NW == 8 && wave >= 4;
    for (int tile = tile_begin; tile < tile_end; ++tile) {
        const int buf = (tile - tile_begin) & 1;
        if (stage_first && tile + 1 < tile_end) {
            stage_tile(buf ^ 1);
            load_tile(min(tile + 2, tile_end - 1));
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb >= live) break;   // (uniform)
            __builtin_amdgcn_sched_barrier(0);   // (or registers spill)
            // S^T = K^ Q^T for the tile's two blocks of 32 keys
            f32x16_t sacc[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                if constexpr (REF_BY_PRODUCT) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) sacc[mb][e] = 0.0f;
                    sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones.b, minus_ref[rb].b, sacc[mb], 0, 0, 0);
                } else {
                    sacc[mb] = c_ref[rb];
                }
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    BF8 ah, al;
                    *reinterpret_cast<uint4 *>(ah.u) = *reinterpret_cast<const uint4 *>(&sm.kh[buf][32 * mb + n][16 * kk + 8 * h]);
                    *reinterpret_cast<uint4 *>(al.u) = *reinterpret_cast<const uint4 *>(&sm.kl[buf][32 * mb + n][16 * kk + 8 * h]);
                    sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah.b, qh[rb][kk].b, sacc[mb], 0, 0, 0);
                    sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah.b, ql[rb][kk].b, sacc[mb], 0, 0, 0);
                    sacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al.b, qh[rb][kk].b, sacc[mb], 0, 0, 0);
                }
            }
            // keys past the end of the sequence (last tile only): element e of block mb is key
            // 32 mb + 8 (e / 4) + 4 h + e % 4
            const int n_valid = len - tile * kWave;
            if (n_valid < kWave) {
                const int valid = n_valid - 4 * h;
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (32 * mb + 8 * (e / 4) + (e % 4) >= valid) sacc[mb][e] = -INFINITY;
            }
            // online softmax of this lane's row (its other 32 keys of the tile are in lane + 32)
            float mx = sacc[0][0];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int e = mb == 0 ? 1 : 0; e < 16; e += 2) mx = fmaxf(fmaxf(mx, sacc[mb][e]), sacc[mb][e + 1 < 16 ? e + 1 : e]);
            {
                float other = mx, own = mx;
                swap32(own, other);                    // the row's other half of the tile is in lane ^ 32
                mx = fmaxf(own, other);
            }
            const bool first = tile == tile_begin;
            if (first || __ballot(mx > kHeadroom) != 0) {
                const float delta = first ? mx : fmaxf(mx, 0.0f);
                m_ref[rb] += delta;
                if constexpr (REF_BY_PRODUCT) {
                    const float r0 = -m_ref[rb], r1 = r0 - __uint_as_float(__float_as_uint(r0) & 0xffff0000u);
                    const float r2 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
                    minus_ref[rb].u[0] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
                    minus_ref[rb].u[1] = __float_as_uint(r2) >> 16;
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e) c_ref[rb][e] = -m_ref[rb];
                }
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) sacc[mb][e] -= delta;
                if (!first) {
                    const float alpha = exp2_raw(-delta);
                    l_run[rb] *= alpha;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int e = 0; e < 16; ++e) oacc[rb][nb][e] *= alpha;
                }
            }
            float psum = 0.0f;
            BF8 ph[4], pl[4];   // per group of 16 keys: the 8 k-slots of this lane, hi and lo
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    const float p0 = exp2_raw(sacc[mb][e]), p1 = exp2_raw(sacc[mb][e + 1]);
                    psum += p0 + p1;
                    // (the remainders as v_dot2_f32_bf16 of the packed pair with (-1, 0): one instruction instead of two, and slower)
                    const uint32_t b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
                    const float l0 = p0 - __uint_as_float(b0 & 0xffff0000u), l1 = p1 - __uint_as_float(b1 & 0xffff0000u);
                    ph[2 * mb + e / 8].u[(e % 8) / 2] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                    pl[2 * mb + e / 8].u[(e % 8) / 2] = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
                }
            l_run[rb] += psum;
            // O^T += V^T P^T
#pragma unroll
            for (int g16 = 0; g16 < 4; ++g16)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    BF8 va;
                    const uint16_t *vrow = &sm.vt[buf][32 * nb + n][16 * g16 + 4 * h];
                    const uint2 x0 = *reinterpret_cast<const uint2 *>(vrow), x1 = *reinterpret_cast<const uint2 *>(vrow + 8);
                    va.u[0] = x0.x; va.u[1] = x0.y; va.u[2] = x1.x; va.u[3] = x1.y;
                    oacc[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va.b, ph[g16].b, oacc[rb][nb], 0, 0, 0);
                    oacc[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va.b, pl[g16].b, oacc[rb][nb], 0, 0, 0);
                }
        }
        // stage the next tile into the other buffer, request the one after
        if (!stage_first && tile + 1 < tile_end) {
            stage_tile(buf ^ 1);
            load_tile(min(tile + 2, tile_end - 1));
        }
        __syncthreads();
    }

    // partial of each row: element e of block nb is channel 32 nb + 8 (e / 4) + 4 h + e % 4 of row n
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = grp * ROWS + 32 * NW * rb + wave * 32 + n;
        if (row >= shp.rows_per_kv) continue;
        const int64_t prow = (pair * shp.rows_per_kv + row) * shp.n_splits + split;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<float4 *>(part_acc + prow * D + 32 * nb + 8 * q4 + 4 * h) =
                    make_float4(oacc[rb][nb][4 * q4], oacc[rb][nb][4 * q4 + 1], oacc[rb][nb][4 * q4 + 2], oacc[rb][nb][4 * q4 + 3]);
        const float l = l_run[rb] + __shfl_xor(l_run[rb], 32, kWave);
        if (h == 0) {
            part_ml[prow * 2] = m_ref[rb];   // in units of log2
            part_ml[prow * 2 + 1] = l;
        }
    }
}

template <class P>
int launch_decode_mq(const octopus_codebooks_t &cb, const DecodeShape &s, const void *cache, const void *v,
                     const int32_t *seq_lens, float *part_ml, float *part_acc, hipStream_t stream, PageTable pt) {
    const DeviceBooks books = device_books(cb);
    const int64_t work = static_cast<int64_t>(s.n_seq) * s.n_kv_heads * s.n_splits * s.n_row_groups;
    const int64_t wgs = (work + kXcds - 1) / kXcds * kXcds;   // see the kernel's work mapping
    if (wgs * std::min(s.rows_per_pass, 256) * 2 > UINT32_MAX) return static_cast<int>(hipErrorInvalidValue);   // (threads of a launch)
    auto go = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(wgs)), dim3(kWave * waves), 0, stream, books, s,
                           static_cast<const uint4 *>(cache), static_cast<const uint16_t *>(v), seq_lens, part_ml, part_acc,
                           pt);
    };
    if (s.rows_per_pass == 128) {
        go(decode_kernel_mq<P, 4, 1>, 4);
    } else if (s.rows_per_pass == 256) {
        go(decode_kernel_mq<P, 8, 1>, 8);
    } else if (P::D <= 64 && s.rows_per_pass == 512) {
        if constexpr (P::D <= 64) go(decode_kernel_mq<P, 8, 2>, 8);
    } else {
        return static_cast<int>(hipErrorInvalidValue);
    }
    return static_cast<int>(hipGetLastError());
}

}  // namespace octopus

#endif
