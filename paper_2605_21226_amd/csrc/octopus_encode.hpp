// Online key encoder (Alg. 1 with the local 3x3 candidate set): a workgroup of 4 or 8 wavefronts takes one to
// eight consecutive 64-token cache tiles of one (sequence, KV head), one after the other.  With the library's own
// direction codebooks the winner of the nine candidates is found among four (CornerGrid).
#ifndef OCTOPUS_ENCODE_HPP_
#define OCTOPUS_ENCODE_HPP_

#include <cstddef>

#include "octopus_device.hpp"

namespace octopus {

constexpr int kURow = 65;  // words per coordinate row of the rotated tile (64 keys + 1 pad)

template <int D>
constexpr float inv_sqrt_dim() {
    return D == 64 ? 0.125f : (D == 128 ? 0.08838834764831845f : 0.0625f);
}

// Seed search (Alg. 1, searchsorted on B_xi) through a uniform grid of cells over [-1, 1]: a cell
// stores how many boundaries lie in lower cells and the boundary inside the cell (+inf if none).  The
// host refuses codebooks with two boundaries in one cell, so one compare finishes the count exactly:
// the cell index is monotone in x, hence boundaries of lower cells are below x and those of higher
// cells above it.
template <int BD>
struct SeedGrid {
    static constexpr int K = 1 << BD;
    static constexpr int NCELL = 8 * K;
    __device__ static __forceinline__ int cell_of(float x) {
        // floor((x + 1) * NCELL / 2), clamped: the scaling by a power of two is exact, so one fused multiply-add
        // rounds as the sum does, and the conversion's truncation is the floor wherever the clamp lets it through
        const int c = static_cast<int>(fmaf(x, 0.5f * NCELL, 0.5f * NCELL));
        return min(max(c, 0), NCELL - 1);
    }
};

// CORNERS.  The winner of Alg. 1's nine candidates is one of four for every Lloyd-Max direction codebook this library
// builds (corner_levels; other codebooks take the nine): with |xi| and |eta| in the place of xi and eta, the four corners of
// the bracket between two neighbouring positive levels on either axis (below the second level: the first bracket, above
// the last but one: the last), in the quadrant that the signs of the key's x and y name.  Why: on a face of the octahedron the
// point is a linear function of (xi, eta), so a candidate that loses to one corner at every vertex of a convex piece of the
// square loses on all of it.  Cut by the brackets, by the seeds and by the face, every piece has such a corner for each
// other candidate, by at least 2.9e-6 of the triplet's norm (the rounding errors of two scores stay below 1e-6) where |p_x|
// and |p_y| are above near_axis().  Next to an axis two mirrored candidates tie, and the first of the nine wins: a
// wavefront with such a key in it (one in 300; zero and non-finite keys as well) also looks at the nine.
// Equal scores of two corners are decided in the order of Alg. 1's loop, which runs towards the axis where the
// coordinate is negative.  Signs cost nothing (the products take |x| and |y|), the corners lie at constant offsets from the
// first one, so there is no table of neighbours: 4 lookups a triplet instead of 15, 61 vector instructions instead of 115.
//
// The bracket is a rounded polynomial of the coordinate (linear up to 4 direction bits, whose levels are nearly evenly
// spaced; a square term at 5): its steps need not lie on the levels, the winner is a corner of either bracket where they part
// (by the same margins; tests/test_encoder_brackets.py takes the steps as they are).  For the same reason the coordinates
// need no more than the hardware's reciprocal.  Before, a grid of cells in LDS gave the bracket: a lookup and a compare more per axis
// (71 vector instructions a triplet) and a table to build.  With the closed form of lone coordinates (TWO_PADS below): 16 x 32768 tokens x
// 8 KV heads, d = 128, b = 3 561 -> 521 us; 4 sequences at b = 2 / b = 4 143 -> 131.5 / 203 -> 183; d = 64, 8 x 32768 x 8, b = 3 / 4 151 -> 134 /
// 287 -> 197; d = 256, 4 x 16384 x 8, b = 2.5 223 -> 210.
constexpr int log2_of(int x) { return x <= 1 ? 0 : 1 + log2_of(x / 2); }
template <int BD>
struct CornerGrid {
    static constexpr int K = 1 << BD, H = K / 2;
    // steps of the bracket: w = |xi| - 1 / 2 -> round(w (kSlope - kBend |w|) + H / 2 - 1), in 0 .. H - 2 for |w| <= kReach
    static constexpr float kSlope = BD <= 3 ? 4.25f : (BD == 4 ? 8.4f : 17.2f), kBend = BD == 5 ? 1.8f : 0.0f;
    static constexpr float kReach = BD <= 3 ? 0.34f : (BD == 4 ? 0.41f : 0.455f);
    static constexpr uint32_t kOne = 0x4B000000u;   // the bits of 2^23: added to a number below 2^22 it leaves its integer in the low bits
    // H + bracket, above it the bits of kOne; any w, NaN included
    __device__ static __forceinline__ uint32_t bracket(float w) { return bracket_within(__builtin_amdgcn_fmed3f(w, -kReach, kReach)); }
    // the same for |w| <= kReach (the host's tests take the steps from here)
    __host__ __device__ static __forceinline__ uint32_t bracket_within(float w) {
        const float slope = kBend != 0.0f ? fmaf(fabsf(w), -kBend, kSlope) : kSlope;
        return __builtin_bit_cast(uint32_t, fmaf(w, slope, 8388608.0f + static_cast<float>(H + H / 2 - 1)));
    }
    // the margins next to an axis shrink with the levels: 2 |p_x| times the first level, and less where z < 0
    static constexpr float near_axis() { return BD <= 3 ? 1e-5f : 1.25e-6f * K; }
    // What lane l adds to bracket(x) REP * 16 + bracket(y) H * REP * 16, modulo 2^32, for the byte offset of the bracket's first corner
    // in its copy of the quadrant table.  (Opaque: taken apart, its large part keeps the table's address out of the LDS
    // instructions' offsets.)
    template <int REP>
    static constexpr uint32_t kCornerStart = 0u - (kOne + H) * (REP * 16u) - (kOne + H) * (H * REP * 16u);
    template <int REP>
    __device__ static __forceinline__ uint32_t corner_start(int lane) {
        uint32_t at = kCornerStart<REP> + (static_cast<uint32_t>(lane) & (REP - 1)) * 16u;
        asm volatile("" : "+v"(at));
        return at;
    }
};

// The direction table holds ONE QUADRANT of the code grid: a Lloyd-Max codebook of the symmetric marginal is
// antisymmetric (C_xi[K - 1 - j] = -C_xi[j], checked on the host), and Oct^-1(-xi, eta) is Oct^-1(xi, eta) with
// its first component negated, bit for bit (likewise eta and the second component).  Entry (fx, fy), fx, fy <
// K / 2, is Oct^-1(C_xi[fx], C_xi[fy]); a code (jx, jy) reads entry (min(jx, K-1-jx), min(jy, K-1-jy)) and negates
// the key's x (y) coordinate instead of the entry's when jx (jy) lies in the upper half -- the products, and so
// the scores, are the same numbers.  A quarter of the entries pays for four times the copies: copy r of entry
// e sits at index e * REP + r and lane l reads copy l % REP, so with 8 copies of 16 bytes any 8 neighbouring lanes
// read 8 different groups of banks whatever their codes (two copies of the full table left the candidate reads
// with about one conflict cycle per useful cycle).  For 6-bit direction codes four copies fit the budget; at
// d = 256, where the rotated tile alone takes 67 KB, four copies up to 3-bit codes and two above, so that two
// workgroups still fit a compute unit at 3 bits per coordinate.  The seed grid keeps two copies up to d = 128.
template <int D, int BD = 1>
constexpr int encode_table_rep() { return (D <= 128 && BD <= 5) ? 8 : (D <= 128 || BD <= 3 ? 4 : 2); }
constexpr int quadrant_entries(int bd) { return bd <= 1 ? 1 : (1 << (2 * (bd - 1))); }

// Wavefronts per workgroup.  LDS (the rotated tile, above all) decides how many workgroups a compute unit holds:
// three at d = 128 up to 3 bits per coordinate, two at 4 bits and at d = 256, one at d = 256 and 4 bits; with four
// wavefronts each a SIMD then has three, two or one to choose from, and the kernel waits on LDS and barriers.  Eight
// wavefronts share a tile from d = 128 on (measured, same records: d = 128 b = 3 -4 %, b = 4 -15 %; d = 256 b = 3
// -8 %, b = 4 -28 %; at d = 64 four workgroups fit anyway and eight wavefronts gain nothing).
template <class P>
constexpr int encode_waves() { return P::D >= 128 ? 8 : 4; }
template <class P>
constexpr int encode_threads() { return encode_waves<P>() * kWave; }

// float2 entries of a class's grid (rep: its copies, lane l reads copy l mod rep) and of a neighbour table.
constexpr int grid_cells(int bd, bool corners, int rep) { return bd < 1 || corners ? 1 : 8 * (1 << bd) * rep; }
constexpr int axis_entries(int bd, bool corners) { return bd < 1 || corners ? 1 : (1 << bd) * 3; }
template <class P, bool QJL, bool CORNERS>
struct EncodeSmem {
    float u[3 * P::NTRI][kURow];           // rotated coordinates [coordinate][key]
    __attribute__((aligned(16))) uint32_t rec[P::NWORDS][kWave];   // packed records [word][key]
    static constexpr int REP = encode_table_rep<P::D, (P::BD0 > P::BD1 ? P::BD0 : P::BD1)>();
    static constexpr int CREP = P::D <= 128 ? 2 : 1;   // copies of the grid
    static constexpr int NX = P::BD0 > 2 || P::BD1 > 2 ? 1 << (P::BD0 > P::BD1 ? P::BD0 : P::BD1) : 4;
    static constexpr int NR = 1 << (P::BN0 > P::BN1 ? P::BN0 : P::BN1);
    float4 lut0[quadrant_entries(P::BD0) * REP];
    float4 lut1[P::NCLASS == 2 ? quadrant_entries(P::BD1) * REP : 1];
    float2 cell0[grid_cells(P::BD0, CORNERS, CREP)];
    float2 cell1[grid_cells(P::BD1, CORNERS, CREP)];
    // neighbours of a seed index j on the x and on the y axis, [j][dx + 1]: {+-1 (the sign the key's coordinate
    // takes), byte offset of the candidate's row / column in the quadrant table}
    float2 nbx0[axis_entries(P::BD0, CORNERS)], nby0[axis_entries(P::BD0, CORNERS)];
    float2 nbx1[axis_entries(P::BD1, CORNERS)], nby1[axis_entries(P::BD1, CORNERS)];
    float c_xi[P::NCLASS][NX];
    float c_rho[P::NCLASS][NR];
    float bnd_xi[P::NCLASS][NX];           // boundaries, +inf padded
    __attribute__((aligned(16))) float bnd_rho[P::NCLASS][NR];   // (read four at a time where there are many)
    float sumsq[kWave];                    // squared norm of each key of the tile, then its scale factor 1 / (gamma sqrt(d))
    float res_sq[QJL ? encode_waves<P>() : 1][QJL ? kWave : 1];   // QJL side-car: squared residual norm, partial per wavefront
};

// Wavefronts per SIMD that the LDS footprint allows (160 KB per compute unit, 4 SIMDs): the register budget the
// kernel is compiled for, so that registers never cost a workgroup that LDS has room for.
template <class P, bool QJL, bool CORNERS>
constexpr int encode_waves_per_simd() {
    constexpr int groups = static_cast<int>((160 * 1024) / sizeof(EncodeSmem<P, QJL, CORNERS>));
    constexpr int waves = (groups < 1 ? 1 : groups) * encode_waves<P>() / 4;
    return waves > 6 ? 6 : waves;   // (the kernel does not fit the 64 registers of 8 wavefronts per SIMD)
}

// Entry (fx, fy) of the quadrant: the levels counted from the outermost negative one (FIRST 0), or for CORNERS from
// the least positive one (FIRST K / 2).
template <int BD, int REP, int FIRST>
__device__ __forceinline__ void build_quadrant(float4 *lut, const float *c_xi, int tid, int nthreads) {
    constexpr int H = BD <= 1 ? 1 : 1 << (BD - 1);
    // (with fewer entries than threads, nthreads / (H * H) threads share an entry: each computes it once and
    // writes its share of the copies)
    constexpr int Q = H * H;
    if (Q >= nthreads) {
        for (int e = tid; e < Q; e += nthreads) {
            const float4 n = oct_decode(c_xi[FIRST + e % H], c_xi[FIRST + e / H]);
#pragma unroll
            for (int r = 0; r < REP; ++r) lut[e * REP + r] = n;
        }
    } else {
        const int per_entry = nthreads / Q, e = tid % Q;
        const float4 n = oct_decode(c_xi[FIRST + e % H], c_xi[FIRST + e / H]);
        for (int r = tid / Q; r < REP; r += per_entry) lut[e * REP + r] = n;
    }
}

template <int BD, int REP, bool CORNERS>
__device__ __forceinline__ void build_encode_lut(float4 *lut, float2 *nbx, float2 *nby, const float *c_xi, int tid,
                                                 int nthreads) {
    constexpr int K = 1 << BD, H = BD <= 1 ? 1 : K / 2;
    build_quadrant<BD, REP, CORNERS ? K / 2 : 0>(lut, c_xi, tid, nthreads);
    if constexpr (!CORNERS) {
        for (int e = tid; e < 3 * K; e += nthreads) {
            const int j = min(max(e / 3 + e % 3 - 1, 0), K - 1);   // the clamped neighbour (Alg. 1's window at the rim)
            const int f = min(j, K - 1 - j);
            const float sign = j >= H && K > 1 ? -1.0f : 1.0f;
            nbx[e] = make_float2(sign, __uint_as_float(static_cast<uint32_t>(f * REP * 16)));
            nby[e] = make_float2(sign, __uint_as_float(static_cast<uint32_t>(f * H * REP * 16)));
        }
    }
}

// Oct^-1 of the centroids of a direction code, from the quadrant table.
template <int BD, int REP, bool CORNERS = false>
__device__ __forceinline__ float4 dir_lookup(const float4 *lut, uint32_t code, int lane) {
    constexpr int K = 1 << BD, H = BD <= 1 ? 1 : K / 2;
    const int jx = static_cast<int>(code & (K - 1)), jy = static_cast<int>(code >> BD);
    const int fx = CORNERS ? max(jx, K - 1 - jx) - H : min(jx, K - 1 - jx), fy = CORNERS ? max(jy, K - 1 - jy) - H : min(jy, K - 1 - jy);
    float4 n = lut[(fx + fy * H) * REP + (lane & (REP - 1))];
    if ((jx >= H) != CORNERS) n.x = -n.x;
    if ((jy >= H) != CORNERS) n.y = -n.y;
    return n;
}

// Two phases with a barrier between them: the cell of every boundary, one boundary per thread; then, per cell, how many
// boundaries lie in lower ones, four cells of boundaries per LDS read.  (Computing every boundary and its cell anew for
// every cell was 1900 cycles of a workgroup's start at 4-bit directions and 3900 at 5-bit ones.)
template <int BD>
__device__ __forceinline__ void build_boundaries(float *bnd, int *bnd_cell, const float *c_xi, int tid) {
    using G = SeedGrid<BD>;
    if (tid < (G::K > 4 ? G::K : 4)) {
        const float b = tid < G::K - 1 ? 0.5f * (c_xi[min(tid, G::K - 1)] + c_xi[min(tid + 1, G::K - 1)]) : INFINITY;
        bnd[tid] = b;
        if (bnd_cell != nullptr) bnd_cell[tid] = tid < G::K - 1 ? G::cell_of(b) : G::NCELL;
    }
}
template <int BD, int REP>
__device__ __forceinline__ void build_seed_grid(float2 *cell, const float *bnd, const int *bnd_cell, int tid, int nthreads) {
    using G = SeedGrid<BD>;
#pragma unroll 1
    for (int c = tid; c < G::NCELL; c += nthreads) {
        int below = 0;
#pragma unroll
        for (int k = 0; k < G::K; k += 4) {   // (entries past the last boundary are in no lower cell; at least four exist)
            const int4 at = *reinterpret_cast<const int4 *>(bnd_cell + k);
            below += (at.x < c ? 1 : 0) + (at.y < c ? 1 : 0) + (at.z < c ? 1 : 0) + (at.w < c ? 1 : 0);
        }
        const float first = bnd[below];       // +inf past the last one
#pragma unroll
        for (int r = 0; r < REP; ++r) cell[c * REP + r] = make_float2(__int_as_float(below), first);
    }
}

// number of boundaries strictly below x
template <int BD, int REP>
__device__ __forceinline__ int seed_index(const float2 *cell, const float *bnd, float x, int lane) {
    (void)bnd;
    const float2 e = cell[SeedGrid<BD>::cell_of(x) * REP + (lane & (REP - 1))];
    return __float_as_int(e.x) + (e.y < x ? 1 : 0);
}

// Sum over the LPR (8, 16 or 32) neighbouring lanes that hold one key row, left in all of them: an exchange-and-add
// butterfly over lane distances 1, 2, 4, 8 (and 16).  The first four go through the vector ALU's own lane permutes
// instead of LDS: after the distances 1 and 2 the four lanes of a quad hold the same sum, so the mirror of 8 lanes
// pairs each quad with its neighbour exactly as distance 4 does, and the mirror of 16 each half as distance 8 does
// (the same two operands in every addition, so the same bits).
template <int CTRL>
__device__ __forceinline__ float lane_permute(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
    static_assert(LPR == 8 || LPR == 16 || LPR == 32, "lanes per key row");
    v += lane_permute<0xB1>(v);    // quad permute [1, 0, 3, 2]
    v += lane_permute<0x4E>(v);    // quad permute [2, 3, 0, 1]
    if constexpr (LPR >= 16) v += lane_permute<0x141>(v);   // mirror within each 8 lanes
    if constexpr (LPR >= 32) v += lane_permute<0x140>(v);   // mirror within each 16 lanes
    // (the last addition in the order written, not as one instruction with the permute, which takes it
    // the other way round: of several NaNs in a key the same one is its norm in every kernel)
    float other = LPR == 8 ? lane_permute<0x141>(v) : (LPR == 16 ? lane_permute<0x140>(v) : __shfl_xor(v, 16, kWave));
    asm("" : "+v"(other));
    return v + other;
}

template <int R>
__device__ __forceinline__ void butterflies(float (&x)[R]) {
#pragma unroll
    for (int h = 1; h < R; h <<= 1) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if ((j & h) == 0) {
                const float a = x[j], b = x[j | h];
                x[j] = a + b;
                x[j | h] = a - b;
            }
        }
    }
}

// One triplet of one key: E4-E7 of the hot path.  Returns the packed direction field and norm index.
template <int BD, int BN, int REP, int CREP>
__device__ __forceinline__ void encode_triplet(float x, float y, float z, const float4 *lut, const float2 *cell,
                                               const float2 *nbx, const float2 *nby, const float *bnd_xi,
                                               const float *bnd_rho, int lane, uint32_t *dir_field,
                                               uint32_t *nrm_index) {
    constexpr int K = 1 << BD, M = 1 << BN;
    // Eq. (oct-encode)
    const float l1 = fabsf(x) + fabsf(y) + fabsf(z);
    // 1 / l1: the hardware reciprocal (1 ulp) refined by one Newton step, so that xi and eta carry the rounding of
    // a division rather than of an approximation (they are compared with the codebook boundaries below)
    const float l1c = fmaxf(l1, kEps);
    float inv = __builtin_amdgcn_rcpf(l1c);
    inv = fmaf(fmaf(-l1c, inv, 1.0f), inv, inv);
    const float px = x * inv, py = y * inv;
    float xi = px, eta = py;
    if (z < 0.0f) {
        const float fx = 1.0f - fabsf(py), fy = 1.0f - fabsf(px);
        xi = (px >= 0.0f) ? fx : -fx;
        eta = (py >= 0.0f) ? fy : -fy;
    }
    // scalar seed
    const int jx = seed_index<BD, CREP>(cell, bnd_xi, xi, lane);
    const int jy = seed_index<BD, CREP>(cell, bnd_xi, eta, lane);
    // local 3x3 joint rounding: dx outer, dy inner, the first maximum wins
    // the candidates' places in the quadrant table and the signs the key's coordinates take for them
    // (24-bit multiplies: full rate, unlike the 32-bit one)
    const float2 *rowx = reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(nbx) + __mul24(jx, 24));
    const float2 *rowy = reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(nby) + __mul24(jy, 24));
    float xa[3], yb[3];
    uint32_t ox[3], oy[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float2 ex = rowx[a], ey = rowy[a];
        xa[a] = x * ex.x;
        ox[a] = __float_as_uint(ex.y);
        yb[a] = y * ey.x;
        oy[a] = __float_as_uint(ey.y);
    }
    const char *base = reinterpret_cast<const char *>(lut) + (lane & (REP - 1)) * 16;
    // all nine scores, their maximum, then the first candidate that attains it
    float sc[9];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const float4 n = *reinterpret_cast<const float4 *>(base + ox[a] + oy[b]);
            sc[3 * a + b] = fmaf(z, n.z, fmaf(yb[b], n.y, xa[a] * n.x));
        }
    }
    // the maximum per dx, then overall; the winner is the first dx whose maximum attains it and, of that dx's three
    // candidates, the first that does (the order of Alg. 1's loop: dx outer, dy inner), found with two compares per
    // level instead of one per candidate
    const float row0 = fmaxf(fmaxf(sc[0], sc[1]), sc[2]), row1 = fmaxf(fmaxf(sc[3], sc[4]), sc[5]),
                row2 = fmaxf(fmaxf(sc[6], sc[7]), sc[8]);
    const float best = fmaxf(fmaxf(row0, row1), row2);
    const bool in0 = row0 == best, in1 = row1 == best;
    const int pick_x = in0 ? 0 : (in1 ? 1 : 2);
    const float first = in0 ? sc[0] : (in1 ? sc[3] : sc[6]), second = in0 ? sc[1] : (in1 ? sc[4] : sc[7]);
    const int pick_y = first == best ? 0 : (second == best ? 1 : 2);
    const int cx = min(max(jx + pick_x - 1, 0), K - 1);
    const int cy = min(max(jy + pick_y - 1, 0), K - 1);
    const uint32_t best_code = static_cast<uint32_t>(cx | (cy << BD));
    const float cs = fminf(fmaxf(best, 0.0f), 1.0f);
    int r = 0;
#pragma unroll
    for (int k = 0; k < M - 1; ++k) r += (bnd_rho[k] < cs) ? 1 : 0;
    *dir_field = best_code;
    *nrm_index = static_cast<uint32_t>(r);
}

// The same triplet with the four corners of its bracket as candidates; `valid`: the key is one that is stored (the others
// are zeros, which would send every wavefront of a short append through the nine candidates); `pads`: how many of the
// triplet's coordinates lie past the head dimension (y, z: zero).
// TWO_PADS: the plan's last triplet has one coordinate of its own (d = 64 and 256), and y = z = 0 there: the outermost level of
// x and, of the two next to eta = 0, the one that comes first.  (It lies on both axes, so every key looked at the nine: one
// triplet in 22 at d = 64.)
template <int BD, int BN, int REP, bool TWO_PADS>
__device__ __forceinline__ void encode_triplet_corners(float x, float y, float z, const float4 *lut, uint32_t corner_start,
                                                       const float *bnd_xi, const float *bnd_rho, int lane, bool valid, int pads,
                                                       uint32_t *dir_field, uint32_t *nrm_index) {
    using G = CornerGrid<BD>;
    constexpr int K = G::K, H = G::H, M = 1 << BN;
    const int neg_x = __float_as_int(x) >> 31, neg_y = __float_as_int(y) >> 31;   // 0 or -1
    const char *base = reinterpret_cast<const char *>(lut + (lane & (REP - 1)));
    float best;
    uint32_t best_code;
    uint32_t jx = G::kOne + H, jy = G::kOne + H;   // K / 2 + bracket
    bool known;   // the winner is among the four
    if (TWO_PADS && pads > 1) {
        const float n = *reinterpret_cast<const float *>(base + (H - 1) * REP * 16);
        best = fabsf(x) * n;
        best_code = (static_cast<uint32_t>(~neg_x) & (K - 1)) | ((H - 1) << BD);
        known = fabsf(x) > kEps && fabsf(x) < INFINITY;
        if constexpr (H > 1) jx = G::bracket(fabsf(x) * __builtin_amdgcn_rcpf(fmaxf(fabsf(x), kEps)) - 0.5f);   // (where it is not)
    } else {
    // Eq. (oct-encode), as in encode_triplet, but that the reciprocal is the hardware's (about one unit in the last place)
    const float l1 = fabsf(x) + fabsf(y) + fabsf(z);
    const float inv = __builtin_amdgcn_rcpf(fmaxf(l1, kEps));
    const float px = x * inv, py = y * inv;
    if constexpr (H == 1) {   // one level on either side: the signs are the code
        const float4 n = *reinterpret_cast<const float4 *>(base);
        best = fmaf(z, n.z, fmaf(fabsf(y), n.y, fabsf(x) * n.x));
        best_code = static_cast<uint32_t>((1 + neg_x) | ((1 + neg_y) << BD));
    } else {
        const float wx = fabsf(px) - 0.5f, wy = fabsf(py) - 0.5f;   // |xi| - 1 / 2 and |eta| - 1 / 2, where z < 0 folded over
        jx = G::bracket(z < 0.0f ? -wy : wx);
        jy = G::bracket(z < 0.0f ? -wx : wy);
        uint32_t off;   // (written out: the compiler makes three instructions of the two shift-adds)
        asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(off) : "v"(jy), "n"(log2_of(H * REP * 16)), "v"(corner_start));
        asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(off) : "v"(jx), "n"(log2_of(REP * 16)), "v"(off));
        const char *at = reinterpret_cast<const char *>(lut) + off;
        float sc[4];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float4 n = *reinterpret_cast<const float4 *>(at + (a * REP + b * (H * REP)) * 16);
                sc[2 * a + b] = fmaf(z, n.z, fmaf(fabsf(y), n.y, fabsf(x) * n.x));
            }
        // The upper end wins where its score is larger, or equal and the axis runs the other way.  A pair's larger score is
        // positive wherever it matters (the winner's angle to the key is far below 90 degrees), and then floats compare
        // as integers.
        const float row0 = fmaxf(sc[0], sc[1]), row1 = fmaxf(sc[2], sc[3]);
        best = fmaxf(row0, row1);
        const bool up_x = __float_as_int(row1) - neg_x > __float_as_int(row0);
        const float lower = up_x ? sc[2] : sc[0], upper = up_x ? sc[3] : sc[1];
        const bool up_y = __float_as_int(upper) - neg_y > __float_as_int(lower);
        // K / 2 + level on the positive side of an axis, its complement on the negative one
        const uint32_t code = (jx + (up_x ? 1u : 0u)) | ((jy + (up_y ? 1u : 0u)) << BD);
        uint32_t flip;
        asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(flip) : "n"(K - 1), "v"(neg_x), "v"(neg_y));
        best_code = (code ^ flip) & (K * K - 1u);
    }
    known = fminf(fminf(fabsf(px), fabsf(py)), l1 * (G::near_axis() / kEps)) > G::near_axis();
    }
    // next to an axis, below the divisor's clamp, or not a number: the nine candidates around the seed
    if (valid && !known) {
        if (pads > 1) y = 0.0f;   // (zero times a scale factor that is not a number)
        if (pads > 0) z = 0.0f;
        const float l1x = fmaxf(fabsf(x) + fabsf(y) + fabsf(z), kEps);
        float invx = __builtin_amdgcn_rcpf(l1x);
        invx = fmaf(fmaf(-l1x, invx, 1.0f), invx, invx);
        const float qx = x * invx, qy = y * invx;
        float xi = qx, eta = qy;
        if (z < 0.0f) {
            const float fx = 1.0f - fabsf(qy), fy = 1.0f - fabsf(qx);
            xi = (qx >= 0.0f) ? fx : -fx;
            eta = (qy >= 0.0f) ? fy : -fy;
        }
        // the seed (boundaries strictly below the coordinate) from the bracket: one boundary lies inside it
        auto seed = [&](float v, int j) __attribute__((always_inline)) {
            const float b = bnd_xi[H == 1 ? 1 : j];   // (one boundary in all, zero: the entry behind it is +inf)
            const int h = v > 0.0f ? j + (b < v ? 1 : 0) : j + (b <= -v ? 1 : 0);
            return v > 0.0f ? h : (v <= 0.0f ? K - 1 - h : 0);   // (not a number: the first)
        };
        const int sx = seed(xi, static_cast<int>(jx - G::kOne)), sy = seed(eta, static_cast<int>(jy - G::kOne));
        best = -INFINITY;
        best_code = static_cast<uint32_t>(min(sx + 1, K - 1) | (min(sy + 1, K - 1) << BD));   // (no candidate is a number)
#pragma clang loop unroll(disable)
        for (int dx = -1; dx <= 1; ++dx) {
            const int cx = min(max(sx + dx, 0), K - 1);
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                const uint32_t code = static_cast<uint32_t>(cx | (min(max(sy + dy, 0), K - 1) << BD));
                const float4 n = dir_lookup<BD, REP, true>(lut, code, lane);
                const float s = fmaf(z, n.z, fmaf(y, n.y, x * n.x));
                if (s > best) { best = s; best_code = code; }
            }
        }
    }
    // (thresholds lie in [0, 1), checked with the levels: no clamp of the score)
    int r = 0;
#pragma unroll
    for (int k = 0; k < M - 1; ++k) r += (bnd_rho[k] < best) ? 1 : 0;
    *dir_field = best_code;
    *nrm_index = static_cast<uint32_t>(r);
}

// The encoder-only rounding variants of App. E (same bitstream, same decoder); `mode` as in octopus.h:
// 0 seed only (Alg. 1 with the window {(0,0)}), 1 local 3x3, 2 full K x K grid, 3 three independent
// nearest-centroid rounds (the norm code from rho_i itself), 4 local 2x2 (the seed and its upper neighbour).
// Candidates are visited dx outer, dy inner (full grid: x index outer); the first maximum wins.
template <int BD, int BN, int REP, int CREP>
__device__ __forceinline__ void encode_triplet_any(float x, float y, float z, const float4 *lut, const float2 *cell,
                                                   const float *bnd_xi, const float *bnd_rho, int lane, int mode,
                                                   uint32_t *dir_field, uint32_t *nrm_index) {
    constexpr int K = 1 << BD, M = 1 << BN;
    const float l1 = fabsf(x) + fabsf(y) + fabsf(z);
    // 1 / l1: the hardware reciprocal (1 ulp) refined by one Newton step, so that xi and eta carry the rounding of
    // a division rather than of an approximation (they are compared with the codebook boundaries below)
    const float l1c = fmaxf(l1, kEps);
    float inv = __builtin_amdgcn_rcpf(l1c);
    inv = fmaf(fmaf(-l1c, inv, 1.0f), inv, inv);
    const float px = x * inv, py = y * inv;
    float xi = px, eta = py;
    if (z < 0.0f) {
        const float fx = 1.0f - fabsf(py), fy = 1.0f - fabsf(px);
        xi = (px >= 0.0f) ? fx : -fx;
        eta = (py >= 0.0f) ? fy : -fy;
    }
    const int jx = seed_index<BD, CREP>(cell, bnd_xi, xi, lane);
    const int jy = seed_index<BD, CREP>(cell, bnd_xi, eta, lane);
    float best = -INFINITY;
    uint32_t best_code = 0u;
    auto consider = [&](int ax, int ay) {
        const uint32_t code = static_cast<uint32_t>(ax | (ay << BD));
        const float4 n = dir_lookup<BD, REP>(lut, code, lane);
        const float sc = fmaf(z, n.z, fmaf(y, n.y, x * n.x));
        if (sc > best) { best = sc; best_code = code; }
    };
    // rolled loops on purpose: these variants are for ablations, and unrolling K x K candidates per
    // triplet of every class blows the code up
    if (mode == 2) {
#pragma clang loop unroll(disable)
        for (int c = 0; c < K * K; ++c) consider(c >> BD, c & (K - 1));
    } else {
        const int lo = (mode == 1) ? -1 : 0;
        const int hi = (mode == 1 || mode == 4) ? 1 : 0;
#pragma clang loop unroll(disable)
        for (int dx = lo; dx <= hi; ++dx)
#pragma clang loop unroll(disable)
            for (int dy = lo; dy <= hi; ++dy) consider(min(max(jx + dx, 0), K - 1), min(max(jy + dy, 0), K - 1));
    }
    const float radial = (mode == 3) ? sqrtf(fmaf(z, z, fmaf(y, y, x * x))) : best;
    const float cs = fminf(fmaxf(radial, 0.0f), 1.0f);
    int r = 0;
#pragma unroll
    for (int k = 0; k < M - 1; ++k) r += (bnd_rho[k] < cs) ? 1 : 0;
    *dir_field = best_code;
    *nrm_index = static_cast<uint32_t>(r);
}

// Consecutive fields of one stream of a key's record.  GATHER: gathered in a register and OR-ed into LDS a word at a time (the
// first and the last word of a wavefront's share are also its neighbours'); else each is OR-ed into LDS as it comes.  Bit
// positions are wave-uniform.
template <bool GATHER>
struct FieldWriter {
    uint32_t acc = 0u;
    int bit;   // position of the next field, from the start of the record
    __device__ __forceinline__ void put(uint32_t (*rec)[kWave], int key, int nbits, uint32_t v) {
        const int sh = bit & 31;
        if constexpr (GATHER) {
            acc |= v << sh;
            if (sh + nbits >= 32) {
                atomicOr(&rec[bit >> 5][key], acc);
                acc = sh + nbits > 32 ? v >> (32 - sh) : 0u;
            }
        } else {
            atomicOr(&rec[bit >> 5][key], v << sh);
            if (sh + nbits > 32) atomicOr(&rec[(bit >> 5) + 1][key], v >> (32 - sh));
        }
        bit += nbits;
    }
    __device__ __forceinline__ void finish(uint32_t (*rec)[kWave], int key) const {
        if (GATHER && (bit & 31)) atomicOr(&rec[bit >> 5][key], acc);
    }
};

// Consecutive cache tiles one workgroup takes, its tables built once for all of them: eight where that still leaves
// the launch several workgroups per place on the chip (a long prefill: the tables cost a fifth of a tile's time),
// fewer for shorter calls, down to one, so that a short chunk still spreads over the compute units.
inline int encode_tiles_per_group(int tiles, int n_kv_heads, int n_seq) {
    constexpr int64_t kEnough = 3072;   // 256 compute units x 3 resident workgroups x 4
    for (int t = 8; t > 1; t >>= 1)
        if (static_cast<int64_t>((tiles + t - 1) / t) * n_kv_heads * n_seq >= kEnough) return t;
    return 1;
}

// QJL: also write the optional side-car of Sec. 3.6 (1-bit QJL residual): the residual r = u - u^ of the
// rotated unit key replaces u in LDS as the triplets are encoded, a second sign-flipped Hadamard
// transform follows, and the signs of its output (bit set = negative) plus ||r|| as fp16 are stored per
// key: per tile of 64 tokens [d/32 words][64 keys] uint32, then [64 keys] fp16.
// ANY: the rounding mode is the run-time argument `mode` (the default encoder is built without it).
// CORNERS: four candidates per triplet (CornerGrid).
//
// Bound: the vector units (the nine-candidate form: LDS as well).  With four candidates, the transform's first three
// stages in the load phase and the others in one pass through LDS instead of two, the scale factor applied by the triplets and
// the fields of a record gathered in registers: 16 x 32768 tokens x 8 KV heads at d = 128, b = 3 923 -> 563 us (4.5 -> 7.4 G
// keys/s); 4 sequences at b = 2 / b = 4 241 -> 152 / 293 -> 202; d = 256, 4 x 16384 x 8, b = 2.5 / 4 353 -> 224 / 480 -> 324;
// d = 64, 8 x 32768 x 8, b = 3 252 -> 159; with the residual at d = 256 299 -> 162; 3001 keys of one sequence x 8 at b = 4
// 14.3 -> 11.5.
template <class P, bool BF16, bool QJL, bool ANY = false, bool CORNERS = false>
__global__ __launch_bounds__(encode_threads<P>())
__attribute__((amdgpu_waves_per_eu(encode_waves_per_simd<P, QJL, CORNERS>(), encode_waves_per_simd<P, QJL, CORNERS>())))
void encode_kernel(DeviceBooks books, const void *__restrict__ keys,
                                                      int64_t stride_seq, int64_t stride_tok, int64_t stride_head,
                                                      int32_t n_new, const uint8_t *__restrict__ signs,
                                                      uint4 *__restrict__ cache, int64_t t_capacity,
                                                      const int32_t *__restrict__ start_pos, int32_t n_kv_heads,
                                                      const uint8_t *__restrict__ signs2,
                                                      unsigned char *__restrict__ qjl, int32_t mode, PageTable pt,
                                                      int32_t tiles_per_group) {
    constexpr int D = P::D;
    constexpr int LPR = D / 8;        // threads per key row in the load phase
    constexpr int NWV = encode_waves<P>(), NT = encode_threads<P>();
    constexpr int RPP = NT / LPR;     // key rows per load pass
    using Smem = EncodeSmem<P, QJL, CORNERS>;
    constexpr int REP = Smem::REP, CREP = Smem::CREP;
    // static, so that table addresses are compile-time constants that fold into the LDS instructions
    __shared__ Smem sm;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in a scalar register
    const int kvh = blockIdx.y, seq = blockIdx.z;
    const int64_t start = start_pos ? max(start_pos[seq], 0) : 0;   // (a negative position would write before the cache)
    const int64_t tok_end = min(start + n_new, t_capacity);
    const int64_t first_tile = start / kWave + static_cast<int64_t>(blockIdx.x) * tiles_per_group;
    if (max(first_tile * kWave, start) >= tok_end) return;

    const int64_t head_base = seq * stride_seq + kvh * stride_head;
    const int col = (tid % LPR) * 8;
    const uint32_t sbits = signs[kvh * (D / 8) + col / 8];
    uint32_t flip[4];   // the sign bits of a thread's eight coordinates, two bf16 to a word
#pragma unroll
    for (int w = 0; w < 4; ++w) flip[w] = ((sbits >> (2 * w)) & 1u) << 15 | ((sbits >> (2 * w + 1)) & 1u) << 31;
    uint4 *region = cache + (static_cast<int64_t>(seq) * n_kv_heads + kvh) * (t_capacity * P::GRANULES);

    // A tile's key rows as loaded: 8 coordinates per thread and pass (bf16: one 16-byte word; fp32: two);
    // rows outside [start, tok_end) and tiles past the group's last one read as zeros.  The next tile's rows
    // are requested as soon as the current ones sit in LDS, so that they arrive during its transform and
    // triplet phases.
    constexpr int NPASS = kWave / RPP;
    uint4 raw[NPASS][BF16 ? 1 : 2];
    auto fetch_tile = [&](int64_t tile) {
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass) {
            const int64_t tok = tile * kWave + pass * RPP + tid / LPR;
            const bool valid = tok >= start && tok < tok_end;
#pragma unroll
            for (int h = 0; h < (BF16 ? 1 : 2); ++h) raw[pass][h] = make_uint4(0u, 0u, 0u, 0u);
            if (valid) {
                const int64_t off = head_base + (tok - start) * stride_tok + col;
                if constexpr (BF16) {
                    // 16 threads read one whole 256- or 512-byte row: streamed, read once (non-temporal)
                    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
                    const u32x4_t x = __builtin_nontemporal_load(
                        reinterpret_cast<const u32x4_t *>(static_cast<const uint16_t *>(keys) + off));
                    raw[pass][0] = make_uint4(x.x, x.y, x.z, x.w);
                } else {
                    raw[pass][0] = *reinterpret_cast<const uint4 *>(static_cast<const float *>(keys) + off);
                    raw[pass][BF16 ? 0 : 1] = *reinterpret_cast<const uint4 *>(static_cast<const float *>(keys) + off + 4);
                }
            }
        }
    };
    // the first tile's rows are requested before the tables are built, so that they arrive meanwhile
    fetch_tile(first_tile);
    // The codebooks' levels, one per lane, from the kernel's first argument and in flight with the rows: copied by
    // constant index they are a scalar load and a straight line of moves per level, 2000 cycles before the first table.
    // Together with the two phases of the tables below, at d = 128 and 8 KV heads: one key appended and decoded against
    // 24.4 -> 24.2 us; 3001 keys and values of a prompt at 4 bits (18.4 us) and long prefills the same within the noise.
    float book_xi[P::NCLASS], book_rho[P::NCLASS];
    {
        typedef const float __attribute__((address_space(4))) *arg_t;
        arg_t arg = (arg_t)__builtin_amdgcn_kernarg_segment_ptr();
#pragma unroll
        for (int c = 0; c < P::NCLASS; ++c) {
            book_xi[c] = arg[offsetof(DeviceBooks, c_xi) / 4 + c * kMaxLevels + lane];
            book_rho[c] = arg[offsetof(DeviceBooks, c_rho) / 4 + c * kMaxLevels + lane];
        }
    }

    // tables
    if (wave == 0) {
        static_assert(kMaxLevels == kWave, "a level per lane");
#pragma unroll
        for (int c = 0; c < P::NCLASS; ++c) {
            if (lane < Smem::NX) sm.c_xi[c][lane] = book_xi[c];
            if (lane < Smem::NR) sm.c_rho[c][lane] = book_rho[c];
        }
    }
    __syncthreads();
    int *bnd_cell = reinterpret_cast<int *>(&sm.rec[0][0]);   // (no record is being built yet)
    build_boundaries<P::BD0>(sm.bnd_xi[0], CORNERS ? nullptr : bnd_cell, sm.c_xi[0], tid);
    if constexpr (P::NCLASS == 2) build_boundaries<P::BD1>(sm.bnd_xi[1], CORNERS ? nullptr : bnd_cell + kMaxLevels, sm.c_xi[1], tid);
    build_encode_lut<P::BD0, REP, CORNERS>(sm.lut0, sm.nbx0, sm.nby0, sm.c_xi[0], tid, NT);
    if constexpr (P::NCLASS == 2) build_encode_lut<P::BD1, REP, CORNERS>(sm.lut1, sm.nbx1, sm.nby1, sm.c_xi[1], tid, NT);
    if constexpr (!CORNERS) {   // (with the corners the boundaries serve the keys next to an axis only)
        __syncthreads();
        build_seed_grid<P::BD0, CREP>(sm.cell0, sm.bnd_xi[0], bnd_cell, tid, NT);
        if constexpr (P::NCLASS == 2) build_seed_grid<P::BD1, CREP>(sm.cell1, sm.bnd_xi[1], bnd_cell + kMaxLevels, tid, NT);
    }
    if (tid < P::NCLASS * Smem::NR) {
        const int c = tid / Smem::NR, k = tid % Smem::NR;
        const int levels = 1 << (c ? (P::BN1 > 0 ? P::BN1 : 1) : P::BN0);
        sm.bnd_rho[c][k] = (k < levels - 1) ? 0.5f * (sm.c_rho[c][k] + sm.c_rho[c][k + 1]) : INFINITY;
    }
    for (int e = tid; e < (3 * P::NTRI - D) * kWave; e += NT) sm.u[D + e / kWave][e % kWave] = 0.0f;

    for (int tg = 0; tg < tiles_per_group; ++tg) {
        const int64_t tile = first_tile + tg;
        const int64_t tok_lo = max(tile * kWave, start);
        const int64_t tok_hi = min((tile + 1) * kWave, tok_end);
        if (tok_lo >= tok_hi) break;   // uniform over the workgroup
        // paged cache: the tile's page is asked for now and used when the tile is stored, phases later
        int page_asked = 0;
        if (pt.table != nullptr) page_asked = pt.table[static_cast<int64_t>(seq) * pt.stride + tile];
        __syncthreads();               // the previous tile's records have been stored; tables are complete
        // word 0 (gamma) is written whole by the transform phase below; the code words are OR-ed into
        for (int e = kWave + tid; e < P::NWORDS * kWave; e += NT) sm.rec[e / kWave][e % kWave] = 0u;

        // E1-E2: squared norm, sign flip
        [[maybe_unused]] float rows_sum = 0.0f;
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass) {
            const int key = pass * RPP + tid / LPR;
            float x[8];
            if constexpr (BF16) {
                const uint4 k = raw[pass][0];
                const uint4 r = make_uint4(k.x ^ flip[0], k.y ^ flip[1], k.z ^ flip[2], k.w ^ flip[3]);
                x[0] = bf16_lo(r.x); x[1] = bf16_hi(r.x); x[2] = bf16_lo(r.y); x[3] = bf16_hi(r.y);
                x[4] = bf16_lo(r.z); x[5] = bf16_hi(r.z); x[6] = bf16_lo(r.w); x[7] = bf16_hi(r.w);
            } else {
                const uint4 a = raw[pass][0], b = raw[pass][BF16 ? 0 : 1];
                x[0] = __uint_as_float(a.x); x[1] = __uint_as_float(a.y); x[2] = __uint_as_float(a.z);
                x[3] = __uint_as_float(a.w); x[4] = __uint_as_float(b.x); x[5] = __uint_as_float(b.y);
                x[6] = __uint_as_float(b.z); x[7] = __uint_as_float(b.w);
            }
            float ss = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
            ss = row_sum<LPR>(ss);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = !BF16 && ((sbits >> e) & 1u) ? -x[e] : x[e];
            butterflies<8>(x);   // E3, the first three stages: a thread holds eight coordinates of its row
#pragma unroll
            for (int e = 0; e < 8; ++e) sm.u[col + e][key] = x[e];
            if (tid % LPR == 0) sm.sumsq[key] = ss;
            if constexpr (BF16) rows_sum += ss;
        }
        // Rows that are not a number: their sum again, of the values before their signs were flipped, as a NaN's own sign is stored
        // (all lanes of a row are here).
        if constexpr (BF16) {
            if (__builtin_expect((__float_as_uint(rows_sum) & 0x7fffffffu) > 0x7f800000u, 0)) {
#pragma unroll 1
                for (int pass = 0; pass < NPASS; ++pass) {
                    uint4 k = raw[0][0];
#pragma unroll
                    for (int other = 1; other < NPASS; ++other)
                        if (pass == other) k = raw[other][0];
                    const uint32_t w[4] = {k.x, k.y, k.z, k.w};
                    float ss = 0.0f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float v = e & 1 ? bf16_hi(w[e / 2]) : bf16_lo(w[e / 2]);
                        ss = fmaf(v, v, ss);
                    }
                    ss = row_sum<LPR>(ss);
                    if (tid % LPR == 0) sm.sumsq[pass * RPP + tid / LPR] = ss;
                }
            }
        }
        if (tg + 1 < tiles_per_group) fetch_tile(tile + 1);
        __syncthreads();

        // E3: the other stages of the Walsh-Hadamard transform, one key per lane, in one pass through LDS.  The triplets take
        // the coordinates unscaled and multiply by the key's scale factor themselves.
        {
            constexpr int R = D / 8;
            // the norm of every key, once per key: by one wavefront, 64 keys at a time (the load phase has 4 to 32
            // lanes per key, and a square root and a division cost as much there for one active lane as for 64); the
            // scale factor replaces the sum of squares in LDS
            if (wave == NWV - 1) {
                const float gamma = sqrtf(sm.sumsq[lane]);
                sm.rec[0][lane] = __float_as_uint(gamma);
                sm.sumsq[lane] = (1.0f / fmaxf(gamma, kEps)) * inv_sqrt_dim<D>();
            }
            for (int lo = wave; lo < 8; lo += NWV) {
                float x[R];
#pragma unroll
                for (int e = 0; e < R; ++e) x[e] = sm.u[e * 8 + lo][lane];
                butterflies<R>(x);
#pragma unroll
                for (int e = 0; e < R; ++e) sm.u[e * 8 + lo][lane] = x[e];
            }
            __syncthreads();
        }

        // E4-E8: triplets, an equal share of them per wavefront, one key per lane
        {
            constexpr int CHUNK = (P::NTRI + NWV - 1) / NWV;
            const int i_end = min(P::NTRI, (wave + 1) * CHUNK);
            float rsq = 0.0f;
            // The norm thresholds of the default encoder in registers where they are few (up to 3 norm bits; the loop's
            // LDS atomics keep the compiler from hoisting the read itself, and LDS is this kernel's limit); with more
            // levels they stay in LDS, as registers are what six wavefronts per SIMD have least of.
            constexpr bool THR0_REG = P::BN0 <= 3, THR1_REG = P::NCLASS == 2 && P::BN1 >= 1 && P::BN1 <= 3;
            float thr0_reg[THR0_REG ? (1 << P::BN0) : 1], thr1_reg[THR1_REG ? (1 << P::BN1) : 1];
            if constexpr (THR0_REG) {
#pragma unroll
                for (int k = 0; k < (1 << P::BN0) - 1; ++k) thr0_reg[k] = sm.bnd_rho[0][k];
            }
            if constexpr (THR1_REG) {
#pragma unroll
                for (int k = 0; k < (1 << P::BN1) - 1; ++k) thr1_reg[k] = sm.bnd_rho[1][k];
            }
            const float *thr0 = THR0_REG ? thr0_reg : sm.bnd_rho[0];
            const float *thr1 = THR1_REG ? thr1_reg : sm.bnd_rho[P::NCLASS - 1];
            [[maybe_unused]] uint32_t corner0 = 0u, corner1 = 0u;
            using Grid1 = CornerGrid<(P::BD1 > 0 ? P::BD1 : 1)>;
            if constexpr (CORNERS) corner0 = CornerGrid<P::BD0>::template corner_start<REP>(lane);
            if constexpr (CORNERS && P::NCLASS == 2 && !QJL) corner1 = Grid1::template corner_start<REP>(lane);
            const float norm = sm.sumsq[lane];
            const bool valid = tile * kWave + lane >= tok_lo && tile * kWave + lane < tok_hi;
            // (gathered fields cost registers: with nine candidates those of two classes up to d = 128 spill, and of 32 norm levels and
            // more.  16 Ki keys x 8 KV heads over other codebooks, gathered / as they come: d = 128 at 1.5 bits, fp32 keys 73.9 / 64.2 us,
            // at 2.5 bits 76.3 / 72.0, 2 + 6 bits 122 / 94 (bf16 keys); the other way round at 3 bits 61.8 / 64.4, at d = 256 89.1 / 93.0)
            constexpr bool GATHER = CORNERS || ((P::NCLASS == 1 || D > 128) && P::BN0 < 5);
            FieldWriter<GATHER> dir, nrm;
            const int i_first = wave * CHUNK;
            dir.bit = (P::NCLASS == 1 || i_first < P::NT0) ? P::DIR0_BIT + i_first * 2 * P::BD0 : P::DIR1_BIT + (i_first - P::NT0) * 2 * P::BD1;
            nrm.bit = (P::NCLASS == 1 || i_first < P::NT0) ? P::NRM0_BIT + i_first * P::BN0 : P::NRM1_BIT + (i_first - P::NT0) * P::BN1;
            for (int i = i_first; i < i_end; ++i) {
                // (coordinates past the head dimension are zero: the scale factor of a key that is not finite is left out there)
                float x = sm.u[3 * i][lane] * norm, y = sm.u[3 * i + 1][lane] * (CORNERS || 3 * i + 1 < D ? norm : 1.0f),
                      z = sm.u[3 * i + 2][lane] * (CORNERS || 3 * i + 2 < D ? norm : 1.0f);
                asm("" : "+v"(x), "+v"(y), "+v"(z));   // (the rounded products: none is to be fused into a later sum)
                uint32_t dir_field, nrm_index;
                float4 nhat;
                float rho;
                if (P::NCLASS == 1 || i < P::NT0) {
                    if constexpr (ANY)
                        encode_triplet_any<P::BD0, P::BN0, REP, CREP>(x, y, z, sm.lut0, sm.cell0, sm.bnd_xi[0],
                                                                      sm.bnd_rho[0], lane, mode, &dir_field, &nrm_index);
                    else if constexpr (CORNERS)
                        encode_triplet_corners<P::BD0, P::BN0, REP, 3 * P::NTRI - D == 2>(x, y, z, sm.lut0, corner0, sm.bnd_xi[0], thr0, lane,
                                                                          valid, 3 * i + 3 - D, &dir_field, &nrm_index);
                    else
                        encode_triplet<P::BD0, P::BN0, REP, CREP>(x, y, z, sm.lut0, sm.cell0, sm.nbx0, sm.nby0,
                                                                  sm.bnd_xi[0], thr0, lane, &dir_field, &nrm_index);
                    dir.put(sm.rec, lane, 2 * P::BD0, dir_field);
                    nrm.put(sm.rec, lane, P::BN0, nrm_index);
                    if constexpr (QJL) { nhat = dir_lookup<P::BD0, REP, CORNERS>(sm.lut0, dir_field, lane); rho = sm.c_rho[0][nrm_index]; }
                } else {
                    if constexpr (P::NCLASS == 2) {
                        if constexpr (ANY)
                            encode_triplet_any<P::BD1, P::BN1, REP, CREP>(x, y, z, sm.lut1, sm.cell1, sm.bnd_xi[1],
                                                                          sm.bnd_rho[1], lane, mode, &dir_field, &nrm_index);
                        else if constexpr (CORNERS) {
                            if constexpr (QJL) {   // (a register less across the loop: it spills at d = 128, b = 2.5)
                                corner1 = corner0 + (Grid1::template kCornerStart<REP> - CornerGrid<P::BD0>::template kCornerStart<REP>);
                                asm volatile("" : "+v"(corner1));
                            }
                            encode_triplet_corners<P::BD1, P::BN1, REP, 3 * P::NTRI - D == 2>(x, y, z, sm.lut1, corner1, sm.bnd_xi[1], thr1, lane,
                                                                              valid, 3 * i + 3 - D, &dir_field, &nrm_index);
                        } else
                            encode_triplet<P::BD1, P::BN1, REP, CREP>(x, y, z, sm.lut1, sm.cell1, sm.nbx1, sm.nby1,
                                                                      sm.bnd_xi[1], thr1, lane, &dir_field, &nrm_index);
                        if (i == P::NT0 && i > i_first) {   // the second class has its own streams
                            dir.finish(sm.rec, lane);
                            nrm.finish(sm.rec, lane);
                            dir = FieldWriter<GATHER>{0u, P::DIR1_BIT};
                            nrm = FieldWriter<GATHER>{0u, P::NRM1_BIT};
                        }
                        dir.put(sm.rec, lane, 2 * P::BD1, dir_field);
                        nrm.put(sm.rec, lane, P::BN1, nrm_index);
                        if constexpr (QJL) { nhat = dir_lookup<P::BD1, REP, CORNERS>(sm.lut1, dir_field, lane); rho = sm.c_rho[1][nrm_index]; }
                    }
                }
                if constexpr (QJL) {
                    // r = u - rho^ n^ in place; the padded coordinates of the last triplet stay out of it
                    const float r0 = x - rho * nhat.x, r1 = y - rho * nhat.y, r2 = z - rho * nhat.z;
                    sm.u[3 * i][lane] = r0;
                    rsq = fmaf(r0, r0, rsq);
                    if (3 * i + 1 < D) { sm.u[3 * i + 1][lane] = r1; rsq = fmaf(r1, r1, rsq); }
                    if (3 * i + 2 < D) { sm.u[3 * i + 2][lane] = r2; rsq = fmaf(r2, r2, rsq); }
                }
            }
            dir.finish(sm.rec, lane);
            nrm.finish(sm.rec, lane);
            if constexpr (QJL) sm.res_sq[wave][lane] = rsq;
        }
        __syncthreads();

        // E8: store the tile, 16 bytes per (granule, key), coalesced over keys
        // pt.table (or NULL): `cache` is a pool of [page][KV head] tiles, logical tile j of sequence s is in page
        // pt.table[s * pt.stride + j] (clamped to the pool)
        uint4 *dst = region + tile * (P::GRANULES * kWave);
        if (pt.table != nullptr) {
            const int page = page_asked;
            dst = cache + (static_cast<int64_t>(min(max(page, 0), pt.n_pages - 1)) * n_kv_heads + kvh) * (P::GRANULES * kWave);
        }
        for (int e = tid; e < P::GRANULES * kWave; e += NT) {
            const int g = e / kWave, key = e % kWave;
            const int64_t tok = tile * kWave + key;
            if (tok >= tok_lo && tok < tok_hi) {
                // non-temporal: the records are not read again by this kernel, and lines left behind in the caches
                // (dirty, a whole prefill's worth) slow down whatever streams through memory next
                typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
                const u32x4_t rec4 = {sm.rec[4 * g][key], sm.rec[4 * g + 1][key], sm.rec[4 * g + 2][key],
                                      sm.rec[4 * g + 3][key]};
                __builtin_nontemporal_store(rec4, reinterpret_cast<u32x4_t *>(dst + e));
            }
        }

        if constexpr (QJL) {
            // sigma = sign(H diag(s2) r): the same two radix passes, signs applied on the way in, no scaling
            constexpr int R2 = D / 16;
            for (int g = wave; g < D / 16; g += NWV) {
                const uint32_t sb = signs2[kvh * (D / 8) + 2 * g] | (static_cast<uint32_t>(signs2[kvh * (D / 8) + 2 * g + 1]) << 8);
                float x[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float val = sm.u[g * 16 + e][lane];
                    x[e] = ((sb >> e) & 1u) ? -val : val;
                }
                butterflies<16>(x);
#pragma unroll
                for (int e = 0; e < 16; ++e) sm.u[g * 16 + e][lane] = x[e];
            }
            __syncthreads();
            for (int lo = wave; lo < 16; lo += NWV) {
                float x[R2];
#pragma unroll
                for (int e = 0; e < R2; ++e) x[e] = sm.u[e * 16 + lo][lane];
                butterflies<R2>(x);
#pragma unroll
                for (int e = 0; e < R2; ++e) sm.u[e * 16 + lo][lane] = x[e];
            }
            __syncthreads();
            constexpr int TQ = kWave * (D / 8 + 2);   // side-car bytes per tile
            unsigned char *qt = qjl + ((static_cast<int64_t>(seq) * n_kv_heads + kvh) * (t_capacity / kWave) + tile) * TQ;
            if (pt.table != nullptr) {   // the side-car in pages: a pool of [page][KV head] tiles, like the keys'
                const int page = page_asked;
                qt = qjl + (static_cast<int64_t>(min(max(page, 0), pt.n_pages - 1)) * n_kv_heads + kvh) * TQ;
            }
            const int64_t tok = tile * kWave + lane;
            const bool valid = tok >= tok_lo && tok < tok_hi;
            for (int wd = wave; wd < D / 32; wd += NWV) {
                uint32_t bits = 0u;
#pragma unroll
                for (int e = 0; e < 32; ++e) bits |= (sm.u[32 * wd + e][lane] < 0.0f ? 1u : 0u) << e;
                if (valid) reinterpret_cast<uint32_t *>(qt)[wd * kWave + lane] = bits;
            }
            if (wave == 0 && valid) {
                float n2 = 0.0f;
#pragma unroll
                for (int wv = 0; wv < NWV; wv += 4)
                    n2 += (sm.res_sq[wv][lane] + sm.res_sq[wv + 1][lane]) + (sm.res_sq[wv + 2][lane] + sm.res_sq[wv + 3][lane]);
                reinterpret_cast<__half *>(qt + (D / 8) * kWave)[lane] = __float2half_rn(sqrtf(n2));
            }
        }
    }
}

// One triplet without tables, for the append kernel below: the four corners (next to an axis: the nine candidates) by Oct^-1 of
// their levels, which is what the tables hold.  only_x: y and z lie past the head dimension (TWO_PADS above).
template <int BD, int BN>
__device__ __forceinline__ void encode_triplet_alone(float x, float y, float z, bool only_x, const float *c_xi, const float *c_rho,
                                                     uint32_t *dir_field, uint32_t *nrm_index) {
    using G = CornerGrid<BD>;
    constexpr int K = G::K, H = G::H, M = 1 << BN;
    const float l1 = fabsf(x) + fabsf(y) + fabsf(z);
    const float l1c = fmaxf(l1, kEps);
    float inv = __builtin_amdgcn_rcpf(l1c);
    inv = fmaf(fmaf(-l1c, inv, 1.0f), inv, inv);
    const float px = x * inv, py = y * inv;
    const int neg_x = __float_as_int(x) >> 31, neg_y = __float_as_int(y) >> 31;   // 0 or -1
    float best;
    uint32_t best_code;
    const float wx = fabsf(px) - 0.5f, wy = fabsf(py) - 0.5f;
    const int jx = H > 1 ? static_cast<int>(G::bracket(z < 0.0f ? -wy : wx) - G::kOne) : H;   // K / 2 + bracket
    const int jy = H > 1 ? static_cast<int>(G::bracket(z < 0.0f ? -wx : wy) - G::kOne) : H;
    const bool far = fminf(fminf(fabsf(px), fabsf(py)), l1 * (G::near_axis() / kEps)) > G::near_axis();
    if (only_x && l1 > kEps && l1 < INFINITY) {
        best = fabsf(x) * oct_decode(c_xi[K - 1], c_xi[H]).x;
        best_code = (static_cast<uint32_t>(~neg_x) & (K - 1)) | ((H - 1) << BD);
    } else if (far) {
        constexpr int ENDS = H > 1 ? 2 : 1;
        float sc[4];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (a >= ENDS || b >= ENDS) { sc[2 * a + b] = -INFINITY; continue; }
                const float4 n = oct_decode(c_xi[jx + a], c_xi[jy + b]);
                sc[2 * a + b] = fmaf(z, n.z, fmaf(fabsf(y), n.y, fabsf(x) * n.x));
            }
        const float row0 = fmaxf(sc[0], sc[1]), row1 = fmaxf(sc[2], sc[3]);
        best = fmaxf(row0, row1);
        const bool up_x = H > 1 && __float_as_int(row1) - neg_x > __float_as_int(row0);
        const float lower = up_x ? sc[2] : sc[0], upper = up_x ? sc[3] : sc[1];
        const bool up_y = H > 1 && __float_as_int(upper) - neg_y > __float_as_int(lower);
        const uint32_t code = static_cast<uint32_t>((jx + (up_x ? 1 : 0)) | ((jy + (up_y ? 1 : 0)) << BD));
        const uint32_t flip = (static_cast<uint32_t>(neg_x) & (K - 1)) | (static_cast<uint32_t>(neg_y) & ~(K - 1u));
        best_code = (code ^ flip) & (K * K - 1u);
    } else {
        float xi = px, eta = py;
        if (z < 0.0f) {
            const float fx = 1.0f - fabsf(py), fy = 1.0f - fabsf(px);
            xi = (px >= 0.0f) ? fx : -fx;
            eta = (py >= 0.0f) ? fy : -fy;
        }
        // the seeds (boundaries strictly below the coordinates) from the brackets, as in encode_triplet_corners
        auto seed = [&](float v, int j) __attribute__((always_inline)) {
            const float b = H > 1 ? 0.5f * (c_xi[j] + c_xi[H > 1 ? j + 1 : 0]) : INFINITY;
            const int h = v > 0.0f ? j + (b < v ? 1 : 0) : j + (b <= -v ? 1 : 0);
            return v > 0.0f ? h : (v <= 0.0f ? K - 1 - h : 0);
        };
        const int sx = seed(xi, jx), sy = seed(eta, jy);
        best = -INFINITY;
        best_code = static_cast<uint32_t>(min(sx + 1, K - 1) | (min(sy + 1, K - 1) << BD));   // (no candidate is a number)
#pragma clang loop unroll(disable)
        for (int c = 0; c < 9; ++c) {
            const int cx = min(max(sx + c / 3 - 1, 0), K - 1), cy = min(max(sy + c % 3 - 1, 0), K - 1);
            const float4 n = oct_decode(c_xi[cx], c_xi[cy]);
            const float s = fmaf(z, n.z, fmaf(y, n.y, x * n.x));
            if (s > best) { best = s; best_code = static_cast<uint32_t>(cx | (cy << BD)); }
        }
    }
    int r = 0;
#pragma unroll
    for (int k = 0; k < M - 1; ++k) r += (0.5f * (c_rho[k] + c_rho[k + 1]) < best) ? 1 : 0;
    *dir_field = best_code;
    *nrm_index = static_cast<uint32_t>(r);
}

// Few keys (a decode step appends one per sequence and KV head): one wavefront per key, a triplet per lane.  encode_kernel
// spends 9 us on such a call whatever it holds, tables and a chain of six triplets per wavefront, each with its LDS round
// trips; here nothing is built and every triplet is on its way at once.  Same codes bit for bit (the same operands in every
// addition of the transform and of the norm).  Bound by that chain: load, norm, 7 stages,
// triplet, store.  (A lone last coordinate, at d = 64 and 256, went through the nine candidates one after the other: 88 keys x 8 KV heads at
// d = 64 9.3 -> 4.9 us, one key x 2 at d = 256 8.1 -> 5.1.)
template <class P, bool BF16>
__global__ __launch_bounds__(kWave) void encode_few_kernel(DeviceBooks books, const void *__restrict__ keys, int64_t stride_seq,
                                                           int64_t stride_tok, int64_t stride_head, int32_t n_new,
                                                           const uint8_t *__restrict__ signs, uint4 *__restrict__ cache,
                                                           int64_t t_capacity, const int32_t *__restrict__ start_pos,
                                                           int32_t n_kv_heads, PageTable pt) {
    constexpr int D = P::D, LPR = D / 8;
    constexpr int NX = P::BD0 > 2 || P::BD1 > 2 ? 1 << (P::BD0 > P::BD1 ? P::BD0 : P::BD1) : 4;
    constexpr int NR = 1 << (P::BN0 > P::BN1 ? P::BN0 : P::BN1);
    __shared__ __attribute__((aligned(16))) float u[3 * P::NTRI + 16];
    __shared__ __attribute__((aligned(16))) uint32_t rec[P::NWORDS + 4];
    __shared__ float c_xi[P::NCLASS][NX], c_rho[P::NCLASS][NR];
    const int lane = threadIdx.x;
    const int kvh = blockIdx.y, seq = blockIdx.z;
    const int64_t start = start_pos ? max(start_pos[seq], 0) : 0;
    const int64_t tok = start + blockIdx.x;
    if (blockIdx.x >= static_cast<uint32_t>(n_new) || tok >= t_capacity) return;
    const int64_t tile = tok / kWave;
    int page = 0;
    if (pt.table != nullptr) page = pt.table[static_cast<int64_t>(seq) * pt.stride + tile];
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = 0.0f;
    uint32_t sbits = 0u;
    if (lane < LPR) {
        sbits = signs[kvh * LPR + lane];
        const int64_t off = seq * stride_seq + kvh * stride_head + static_cast<int64_t>(blockIdx.x) * stride_tok + lane * 8;
        if constexpr (BF16) {
            const uint4 r = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(keys) + off);
            x[0] = bf16_lo(r.x); x[1] = bf16_hi(r.x); x[2] = bf16_lo(r.y); x[3] = bf16_hi(r.y);
            x[4] = bf16_lo(r.z); x[5] = bf16_hi(r.z); x[6] = bf16_lo(r.w); x[7] = bf16_hi(r.w);
        } else {
            const float4 a = *reinterpret_cast<const float4 *>(static_cast<const float *>(keys) + off);
            const float4 b = *reinterpret_cast<const float4 *>(static_cast<const float *>(keys) + off + 4);
            x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
        }
    }
#pragma unroll
    for (int c = 0; c < P::NCLASS; ++c) {   // (levels by lane; the arguments hold kMaxLevels of each)
        typedef const float __attribute__((address_space(4))) *arg_t;
        arg_t arg = (arg_t)__builtin_amdgcn_kernarg_segment_ptr();
        const float xi = arg[offsetof(DeviceBooks, c_xi) / 4 + c * kMaxLevels + lane], rho = arg[offsetof(DeviceBooks, c_rho) / 4 + c * kMaxLevels + lane];
        if (lane < NX) c_xi[c][lane] = xi;
        if (lane < NR) c_rho[c][lane] = rho;
    }
    if (lane < P::NWORDS) rec[lane] = 0u;

    // E1-E3: norm, sign flip, transform (eight coordinates per lane, then lane by lane)
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
    ss = row_sum<LPR>(ss);
    const float gamma = sqrtf(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ss))));
    const float norm = (1.0f / fmaxf(gamma, kEps)) * inv_sqrt_dim<D>();
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = ((sbits >> e) & 1u) ? -x[e] : x[e];
    butterflies<8>(x);
    static_for<0, (D == 64 ? 3 : (D == 128 ? 4 : 5))>([&](auto bb) {
        constexpr int m = 1 << decltype(bb)::value;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float other = lane_xor<m>(x[e], lane);
            x[e] = (lane & m) ? other - x[e] : x[e] + other;
        }
    });
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < 8; ++e) u[lane * 8 + e] = x[e];
    }
    __syncthreads();

    // E4-E8
    for (int i = lane; i < P::NTRI; i += kWave) {
        float a = u[3 * i] * norm, b = 3 * i + 1 < D ? u[3 * i + 1] * norm : 0.0f, c = 3 * i + 2 < D ? u[3 * i + 2] * norm : 0.0f;
        asm("" : "+v"(a), "+v"(b), "+v"(c));   // (the rounded products: none is to be fused into a later sum)
        uint32_t dir, nrm;
        int dir_bit, nrm_bit, dir_bits, nrm_bits;
        if (P::NCLASS == 1 || i < P::NT0) {
            encode_triplet_alone<P::BD0, P::BN0>(a, b, c, 3 * i + 1 >= D, c_xi[0], c_rho[0], &dir, &nrm);
            dir_bits = 2 * P::BD0;
            nrm_bits = P::BN0;
            dir_bit = P::DIR0_BIT + i * dir_bits;
            nrm_bit = P::NRM0_BIT + i * nrm_bits;
        } else {
            constexpr int BD1 = P::BD1 > 0 ? P::BD1 : 1, BN1 = P::BN1 > 0 ? P::BN1 : 1;
            encode_triplet_alone<BD1, BN1>(a, b, c, 3 * i + 1 >= D, c_xi[P::NCLASS - 1], c_rho[P::NCLASS - 1], &dir, &nrm);
            dir_bits = 2 * BD1;
            nrm_bits = BN1;
            dir_bit = P::DIR1_BIT + (i - P::NT0) * dir_bits;
            nrm_bit = P::NRM1_BIT + (i - P::NT0) * nrm_bits;
        }
        atomicOr(&rec[dir_bit >> 5], dir << (dir_bit & 31));
        if ((dir_bit & 31) + dir_bits > 32) atomicOr(&rec[(dir_bit >> 5) + 1], dir >> (32 - (dir_bit & 31)));
        atomicOr(&rec[nrm_bit >> 5], nrm << (nrm_bit & 31));
        if ((nrm_bit & 31) + nrm_bits > 32) atomicOr(&rec[(nrm_bit >> 5) + 1], nrm >> (32 - (nrm_bit & 31)));
    }
    if (lane == 0) rec[0] = __float_as_uint(gamma);   // (no field reaches into word 0)
    __syncthreads();
    if (lane < P::GRANULES) {
        uint4 *dst = cache + (static_cast<int64_t>(seq) * n_kv_heads + kvh) * (t_capacity * P::GRANULES) + tile * (P::GRANULES * kWave);
        if (pt.table != nullptr)
            dst = cache + (static_cast<int64_t>(min(max(page, 0), pt.n_pages - 1)) * n_kv_heads + kvh) * (P::GRANULES * kWave);
        typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
        const u32x4_t rec4 = {rec[4 * lane], rec[4 * lane + 1], rec[4 * lane + 2], rec[4 * lane + 3]};
        __builtin_nontemporal_store(rec4, reinterpret_cast<u32x4_t *>(dst + lane * kWave + tok % kWave));
    }
}

// Calls that encode_few_kernel serves: its time goes with the keys, encode_kernel's with the tiles they fall into.  A tile kernel /
// this one, 8 KV heads: one key per sequence, 512 / 1024 / 2048 sequences, d = 128, b = 3 45.5 / 9.5, 87 / 13.9, 170 / 19.4 us
// (d = 256, b = 4 159 / 21, 315 / 32, 626 / 54; d = 64, b = 2 23 / 11.7, 40 / 18, 76 / 31); four keys, 256 sequences, d = 128
// 24.6 / 12.5 but d = 64, b = 2 13.9 / 18.5; 16 keys, 128 sequences 14.9 / 19.4.  In one sequence 512 keys are on a par (9 - 10 us) at
// d = 128 and behind at d = 256 (13 / 20), 128 keys ahead everywhere; alone on the chip one key takes 4.4 us instead of 7.5.
template <int D>
bool few_keys(int64_t n_seq, int64_t n_kv_heads, int64_t n_new) {
    return n_new <= (D >= 128 ? 4 : 2) || n_seq * n_kv_heads * n_new <= 1024;
}

template <class P>
int launch_encode_plan(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                       int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                       const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                       const uint8_t *signs2, void *qjl, hipStream_t stream, PageTable pt = PageTable{nullptr, 0, 0}) {
    const DeviceBooks books = device_books(cb);
    // a start that is not a multiple of 64 makes the new tokens straddle one more tile
    const int tiles = (n_new + kWave - 1) / kWave + (start_pos ? 1 : 0);
    const int tpg = encode_tiles_per_group(tiles, n_kv_heads, n_seq);
    const dim3 grid((tiles + tpg - 1) / tpg, n_kv_heads, n_seq);
    const bool bf16 = key_dtype == OCTOPUS_DTYPE_BF16;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(encode_threads<P>()), 0, stream, books, keys, stride_seq, stride_tok, stride_head, n_new,
                           signs, static_cast<uint4 *>(cache), t_capacity, start_pos, n_kv_heads, signs2,
                           static_cast<unsigned char *>(qjl), 1, pt, tpg);
    };
    // (four candidates per triplet where the winner is known to be among them, else nine)
    if (corner_levels(cb)) {
        if (qjl == nullptr && few_keys<P::D>(n_seq, n_kv_heads, n_new)) {
            auto few = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(n_new, n_kv_heads, n_seq), dim3(kWave), 0, stream, books, keys, stride_seq, stride_tok,
                                   stride_head, n_new, signs, static_cast<uint4 *>(cache), t_capacity, start_pos, n_kv_heads, pt);
            };
            if (bf16) few(encode_few_kernel<P, true>); else few(encode_few_kernel<P, false>);
        } else if (qjl != nullptr) {
            if (bf16) go(encode_kernel<P, true, true, false, true>); else go(encode_kernel<P, false, true, false, true>);
        } else {
            if (bf16) go(encode_kernel<P, true, false, false, true>); else go(encode_kernel<P, false, false, false, true>);
        }
    } else if (qjl != nullptr) {
        if (bf16) go(encode_kernel<P, true, true>); else go(encode_kernel<P, false, true>);
    } else {
        if (bf16) go(encode_kernel<P, true, false>); else go(encode_kernel<P, false, false>);
    }
    return static_cast<int>(hipGetLastError());
}

// The default encoder alone (local 3x3, no side-car, no pages): what the pairs of the App. D sweep are built with.
template <class P>
int launch_encode_basic_plan(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                             int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                             const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                             hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    const int tiles = (n_new + kWave - 1) / kWave + (start_pos ? 1 : 0);
    const int tpg = encode_tiles_per_group(tiles, n_kv_heads, n_seq);
    const dim3 grid((tiles + tpg - 1) / tpg, n_kv_heads, n_seq);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(encode_threads<P>()), 0, stream, books, keys, stride_seq, stride_tok, stride_head, n_new,
                           signs, static_cast<uint4 *>(cache), t_capacity, start_pos, n_kv_heads, nullptr, nullptr, 1,
                           PageTable{nullptr, 0, 0}, tpg);
    };
    if (key_dtype == OCTOPUS_DTYPE_BF16) go(encode_kernel<P, true, false>);
    else go(encode_kernel<P, false, false>);
    return static_cast<int>(hipGetLastError());
}

// The encoder with the rounding mode chosen at run time (no side-car).
template <class P>
int launch_encode_rounding_plan(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                                int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads,
                                int32_t n_new, const uint8_t *signs, void *cache, int64_t t_capacity,
                                const int32_t *start_pos, int32_t mode, hipStream_t stream) {
    const DeviceBooks books = device_books(cb);
    const int tiles = (n_new + kWave - 1) / kWave + (start_pos ? 1 : 0);
    const int tpg = encode_tiles_per_group(tiles, n_kv_heads, n_seq);
    const dim3 grid((tiles + tpg - 1) / tpg, n_kv_heads, n_seq);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(encode_threads<P>()), 0, stream, books, keys, stride_seq, stride_tok, stride_head, n_new,
                           signs, static_cast<uint4 *>(cache), t_capacity, start_pos, n_kv_heads, nullptr, nullptr, mode,
                           PageTable{nullptr, 0, 0}, tpg);
    };
    if (key_dtype == OCTOPUS_DTYPE_BF16) go(encode_kernel<P, true, false, true>);
    else go(encode_kernel<P, false, false, true>);
    return static_cast<int>(hipGetLastError());
}

}  // namespace octopus

#endif
