// The end of a decode call: the partial results of each output row merged, and, with a hybrid cache, the row's share of the
// native-precision window.
#ifndef OCTOPUS_MERGE_HPP_
#define OCTOPUS_MERGE_HPP_

#include "octopus_decode.hpp"

namespace octopus {

// A lane's N neighbouring channels (1, 2 or 4) of a row; the output is aligned to 4 bytes only.
template <int N>
__device__ __forceinline__ void load_channels(const float *p, float (&x)[N]) {
    typedef float vec_t __attribute__((ext_vector_type(N == 1 ? 2 : N)));
    if constexpr (N == 1) {
        x[0] = *p;
    } else {
        const vec_t v = *reinterpret_cast<const vec_t *>(p);
#pragma unroll
        for (int c = 0; c < N; ++c) x[c] = v[c];
    }
}
template <int N>
__device__ __forceinline__ void store_channels(float *p, const float (&x)[N]) {
    typedef float vec_t __attribute__((ext_vector_type(N == 1 ? 2 : N), aligned(4)));
    if constexpr (N == 1) {
        *p = x[0];
    } else {
        vec_t v;
#pragma unroll
        for (int c = 0; c < N; ++c) v[c] = x[c];
        *reinterpret_cast<vec_t *>(p) = v;
    }
}

// The window's part of a row (Sec. 4, default recipe: a short residual window of recent tokens kept uncompressed).  Its tokens
// follow the compressed ones of their sequence; their keys are read as stored, their scores are the plain scale * q . k, and its
// (m, l, acc) joins the split partials in the merge (flash-decoding identity, App. A).
//
// One wavefront per output row (sequence, query, query head).  Keys: [n_seq][n_kv_heads][w_capacity][D],
// values: rows seq_lens[s] + j of the value buffer [n_seq][n_kv_heads][t_capacity][D] (bf16 or fp32 each); with a
// page table (pt.table not NULL) token t of sequence s is row t % 64 of [page][KV head] of a pool of value pages,
// page = pt.table[s * pt.stride + t / 64] clamped to the pool, and t_capacity is what the table can address.
// Chunks of 64 window tokens, one token per lane for the scores (the query sits in LDS), then every lane
// accumulates its D / 64 channels over the chunk's tokens.
// Bound by latency and by the second-level cache (a window is a few kilobytes a row): the chunk's keys are asked for before the
// lengths are known, whole rows per instruction, and handed to their lanes through LDS (16 bytes per lane and row of 64 rows each
// fetched every cache line eight times: 13.3 us of 24 sequences x 64 heads x 32 tokens, so 8.0); the chunk's two pages as soon as
// the lengths are there, and up to 32 value rows, a lane's channels in one load, before the scores are computed.
// The window is worked on by the wavefront that merges the row, with the row's partial results on their way meanwhile: as a kernel of its
// own it cost a launch and a round trip of its result.  Calls with a window of 16 - 128, own kernel / here: 24 ragged sequences to 8000, 8 KV
// heads of eight rows 65.7 / 62.7 us, 1 x 41127, 8 of one 32.5 / 30.1, 1 x 3330, 2 of one, d = 64 18.6 / 14.4, 3 to 8596, 4 of eight, b = 4
// 42.5 / 40.7, 4 x 5000, 4 of four, d = 256 29.1 / 26.3.
template <int D, bool k_is_bf16, bool v_is_bf16>
struct WindowRow {
    static constexpr int CPT = D / kWave;      // channels per lane: CPT lane .. + CPT - 1
    static constexpr int KW = D / (k_is_bf16 ? 8 : 4);                       // 16-byte words of a key row
    static constexpr int VW = v_is_bf16 ? (CPT + 1) / 2 : CPT;               // 32-bit words of a lane's channels
    static constexpr int VB = D <= 128 ? 32 : 16;   // value rows in flight
    static constexpr bool STAGED = KW <= 32;   // (a longer row does not fit a lane's registers: read as it is used)
    static constexpr int RPI = kWave / KW > 0 ? kWave / KW : 1;   // key rows per load instruction
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    struct Smem {
        float qs[D];
        u32x4_t rows[STAGED ? kWave : 1][STAGED ? KW + 1 : 1];
    };
    const WindowCall &w;
    int lane;
    int64_t pair;
    const char *k_pair;
    u32x4_t key[STAGED ? KW : 1];   // the key rows of a chunk: RPI rows per instruction, those past the window's capacity are its last one

    __device__ __forceinline__ WindowRow(const WindowCall &call, int64_t pair_, int lane_)
        : w(call), lane(lane_), pair(pair_), k_pair(static_cast<const char *>(call.k_win) + pair_ * call.w_capacity * (KW * 16)) {}
    __device__ __forceinline__ void request_keys(int64_t j0) {   // (the buffer has at least one row per (sequence, KV head), whatever the lengths)
        if constexpr (STAGED) {
#pragma unroll
            for (int e = 0; e < KW; ++e) {
                const int64_t row = min(j0 + e * RPI + lane / KW, w.w_capacity - 1);
                key[e] = *reinterpret_cast<const u32x4_t *>(k_pair + row * (KW * 16) + (lane % KW) * 16);
            }
        }
    }
    __device__ __forceinline__ void load_query(const DecodeShape &shp, int64_t orow, Smem &sm) const {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int64_t i = orow * D + c * kWave + lane;
            const float x = shp.q_is_bf16 ? __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(shp.q)[i]) << 16)
                                          : static_cast<const float *>(shp.q)[i];
            sm.qs[c * kWave + lane] = x * shp.scale;
        }
        __syncthreads();
    }
    // request_keys(0) and load_query come first
    __device__ __forceinline__ void run(const DecodeShape &shp, Smem &sm, int64_t orow, int seq, int kvh, int asked_len, int asked_win,
                                        float &m_run, float &l_run, float (&acc)[CPT]) {
        const int64_t len = min(max(asked_len, 0), shp.max_len);   // clamped like every other kernel's
        // the window's tokens must fit behind the compressed ones in the value buffer
        const int64_t n_win = max(int64_t{0}, min(min(static_cast<int64_t>(asked_win), w.w_capacity), shp.t_capacity - len));

        m_run = -INFINITY;
        l_run = 0.0f;
#pragma unroll
        for (int c = 0; c < CPT; ++c) acc[c] = 0.0f;
        for (int64_t j0 = 0; j0 < n_win; j0 += kWave) {
            const int nj = static_cast<int>(min(static_cast<int64_t>(kWave), n_win - j0));
            if (j0 > 0) request_keys(j0);
            // where the chunk's value rows lie: 64 tokens are in at most two pages
            const int64_t t0 = len + j0;
            int64_t first = pair * shp.t_capacity + t0, second = first;   // row of token t0, and (less the tokens before) of the next page
            int split = kWave;                                            // tokens of the chunk in the first page
            if (w.pt.table != nullptr) {
                const int32_t *pages = w.pt.table + static_cast<int64_t>(seq) * w.pt.stride;
                const int page0 = pages[t0 / kWave], page1 = pages[(t0 + nj - 1) / kWave];
                split = kWave - static_cast<int>(t0 % kWave);
                first = (static_cast<int64_t>(min(max(page0, 0), w.pt.n_pages - 1)) * shp.n_kv_heads + kvh) * kWave + t0 % kWave;
                second = (static_cast<int64_t>(min(max(page1, 0), w.pt.n_pages - 1)) * shp.n_kv_heads + kvh) * kWave - split;
            }
            uint32_t x[VB][VW];
            auto request_values = [&](int jb) __attribute__((always_inline)) {   // (rows past the chunk's end: its last one)
#pragma unroll
                for (int u = 0; u < VB; ++u) {
                    if (u % 8 == 0 && jb + u >= nj) break;   // (uniform)
                    const int j = min(jb + u, nj - 1);
                    const int64_t row = (j < split ? first : second) + j;
                    if constexpr (v_is_bf16 && CPT == 1) {
                        x[u][0] = static_cast<const uint16_t *>(w.v)[row * D + lane];
                    } else {
                        const uint32_t *vp = static_cast<const uint32_t *>(w.v) + row * (D / (v_is_bf16 ? 2 : 1)) + lane * VW;
#pragma unroll
                        for (int c = 0; c < VW; ++c) x[u][c] = vp[c];
                    }
                }
            };
            request_values(0);
            asm volatile("" ::: "memory");   // (or the loads are moved to their use)
            if constexpr (STAGED) {
                if (j0 > 0) __syncthreads();
#pragma unroll
                for (int e = 0; e < KW; ++e) sm.rows[e * RPI + lane / KW][lane % KW] = key[e];
                __syncthreads();
            }
            float s = -INFINITY;
            if (lane < nj) {
                float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                const u32x4_t *own = STAGED ? &sm.rows[lane][0] : reinterpret_cast<const u32x4_t *>(k_pair + (j0 + lane) * (KW * 16));
#pragma unroll 16
                for (int e = 0; e < KW; ++e) {
                    const u32x4_t x4 = own[e];
                    const uint32_t w4[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        if constexpr (k_is_bf16) {
                            dot[h] = fmaf(sm.qs[8 * e + 2 * h], __uint_as_float(w4[h] << 16), dot[h]);
                            dot[h] = fmaf(sm.qs[8 * e + 2 * h + 1], __uint_as_float(w4[h] & 0xffff0000u), dot[h]);
                        } else {
                            dot[h] = fmaf(sm.qs[4 * e + h], __uint_as_float(w4[h]), dot[h]);
                        }
                    }
                }
                s = (dot[0] + dot[1]) + (dot[2] + dot[3]);
                if (w.scores_out != nullptr) w.scores_out[orow * shp.t_capacity + len + j0 + lane] = s;
            }
            const float m_new = fmaxf(m_run, wave_max(s));
            const float alpha = exp2_raw((m_run - m_new) * kLog2e);
            const float p = (lane < nj) ? exp2_raw((s - m_new) * kLog2e) : 0.0f;   // zero in lanes >= nj
            m_run = m_new;
            l_run = fmaf(l_run, alpha, wave_sum(p));
#pragma unroll
            for (int c = 0; c < CPT; ++c) acc[c] *= alpha;
            for (int jb = 0; jb < nj; jb += VB) {
                if (jb > 0) request_values(jb);
                auto add = [&](int u) __attribute__((always_inline)) {
                    const float wj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), jb + u));
#pragma unroll
                    for (int c = 0; c < CPT; ++c) {
                        const uint32_t word = x[u][v_is_bf16 ? c / 2 : c];
                        const float val = !v_is_bf16 ? __uint_as_float(word) : ((c & 1) ? bf16_hi(word) : bf16_lo(word));
                        acc[c] = fmaf(wj, val, acc[c]);
                    }
                };
                if (jb + VB <= nj) {
#pragma unroll
                    for (int u = 0; u < VB; ++u) add(u);
                } else {   // (rows past the end stay out: at weight zero an infinity in the last row would count again, as 0 * inf)
#pragma unroll
                    for (int u = 0; u < VB - 1; ++u) {
                        if (jb + u >= nj) break;
                        add(u);
                    }
                }
            }
        }
    }
};

// ---- D8: merge of the split partials, one wavefront per output row -----------------------------------
// out = sum_j w_j acc_j / sum_j w_j l_j with w_j = exp(m_j - max_j m_j) (the flash-decoding identity).
// A split without tokens has m = -inf, l = 0 and a zero accumulator, so it needs no special case.
// Bound by latency (one load for the lengths, then the partials, UN at a time): with one partial per segment instead of four per item
// of work, a long sequence has a quarter of the rows to read (one head over 4096 tokens: 11.6 us with 128 partials).
// UN: partial rows in flight per lane, 8 or, where the partials may be many, 32 (deep_merge).
// TWO: the call may be divided into blocks of two rounds (shp.two_round_blocks).
// WIN: one more partial per output row, of a native-precision window: 1 + (bf16 keys) + 2 (bf16 values); 0: no window.
template <int D, bool TWO, int WIN, int UN>
__global__ __launch_bounds__(kWave) void merge_kernel(DecodeShape shp, WindowCall window, const float *__restrict__ part_ml,
                                                      const float *__restrict__ part_acc,
                                                      const int32_t *__restrict__ seq_lens, float *__restrict__ out) {
    constexpr int CPT = D / kWave;  // channels per lane: CPT lane .. + CPT - 1
    __shared__ float wgt[kWave];
    const int lane = threadIdx.x;
    int lens = seq_lens[min(lane, shp.n_seq - 1)];   // asked for before anything is computed
    // (a launch has fewer than 2^32 threads, so a row's index fits 32 bits; divided as 64 bits it is 300 instructions)
    const uint32_t urow = blockIdx.x;  // (seq, qi, head)
    const int64_t orow = urow;
    const int head = static_cast<int>(urow % static_cast<uint32_t>(shp.n_q_heads));
    const uint32_t query = urow / static_cast<uint32_t>(shp.n_q_heads);
    const int qi = static_cast<int>(query % static_cast<uint32_t>(shp.n_q));
    const int seq = static_cast<int>(query / static_cast<uint32_t>(shp.n_q));
    const int kvh = head / shp.heads_per_kv;
    const int row = qi * shp.heads_per_kv + head % shp.heads_per_kv;
    const int grp = row / shp.rows_per_pass, r = row % shp.rows_per_pass;
    using Window = WindowRow<D, ((WIN - 1) & 1) != 0, ((WIN - 1) & 2) != 0>;
    __shared__ typename std::conditional<WIN != 0, typename Window::Smem, char>::type win_smem;
    Window win(window, static_cast<int64_t>(seq) * shp.n_kv_heads + kvh, lane);
    int own_len = 0, win_len = 0;
    if constexpr (WIN != 0) {
        win.request_keys(0);
        own_len = seq_lens[seq];
        win_len = window.win_lens[seq];
        win.load_query(shp, orow, win_smem);
    }
    // Partial j of this row is at prow0 + j * pstride, j < n_part.  The many-row kernel (blocks of 128 rows or more):
    // one partial per split that has tiles, adjacent.  Otherwise: one per segment of this row's (sequence, KV head, row group); the
    // segments' slots are consecutive, one per workgroup that has steps of the pair (the work distribution above).
    int64_t prow0;
    int n_part, pstride;
    if (shp.rows_per_pass >= 128) {
        prow0 = ((static_cast<int64_t>(seq) * shp.n_kv_heads + kvh) * shp.rows_per_kv + row) * shp.n_splits;
        // splits past the last tile have written nothing (max_len may be far above a sequence's length)
        const int asked = WIN != 0 ? own_len : (shp.n_seq <= kWave ? __builtin_amdgcn_readlane(lens, seq) : static_cast<int>(seq_lens[seq]));
        const int len = min(max(asked, 0), shp.max_len);
        n_part = min(shp.n_splits, (len + kWave - 1) / kWave);
        pstride = 1;
    } else {
        const uint64_t G = static_cast<uint64_t>(shp.n_kv_heads) * shp.n_row_groups;
        uint64_t total = 0, before = 0;
        uint32_t st = 0, own = 0;   // steps of sequence s0 + lane, and of this row's
        auto read = [&](int s0) {
            if (s0 > 0 || shp.n_seq > kWave) lens = seq_lens[min(s0 + lane, shp.n_seq - 1)];
            st = s0 + lane < shp.n_seq ? static_cast<uint32_t>(steps_of(lens, shp.max_len, shp.tiles_per_step)) : 0u;
        };
        auto add = [&](int s0, uint32_t x) {   // x: per lane, of sequences s0 ..
            const uint32_t sum = wave_scan(x);
            if (seq >= s0 && seq < s0 + kWave) {
                own = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(st), seq - s0));
                before = total + static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sum - x), seq - s0));
            }
            total += last_lane(sum);
        };
        for (int s0 = 0; s0 < shp.n_seq; s0 += kWave) {
            read(s0);
            add(s0, st);
        }
        const uint64_t sum = total;
        total *= G;
        Division div{kDivideEvenly, shp.item_waves == 8 ? 3 : 2, shp.tiles_per_step};
        if (__builtin_expect(shp.kind_known != 0 || !Division::surely_even<TWO>(shp, st, sum, total, div.waves_log2), 0)) {
            if (shp.kind_known != 0) div.kind = shp.kind_known;
            else div.template set<TWO>(shp, sum, [&](int s0) __attribute__((always_inline)) { read(s0); return st; });
            if (div.kind != kDivideEvenly) {
                total = 0;
                for (int s0 = 0; s0 < shp.n_seq; s0 += kWave) {
                    read(s0);
                    add(s0, div.units(st));
                }
                total *= G;
            }
        }
        const int g = kvh * shp.n_row_groups + grp;
        const uint64_t first = before * G + static_cast<uint64_t>(g) * div.units(own) + div.fixed();   // the pair's first quantum
        n_part = 0;
        int wg = 0;
        if (own > 0u) {
            wg = div.owner(total, first);
            n_part = div.owner(total, first + ((div.quanta(own) - 1u) << div.units_log2())) - wg + 1;
        }
        prow0 = (wg + static_cast<int64_t>(seq) * static_cast<int64_t>(G) + g) * shp.rows_per_pass + r;
        pstride = shp.rows_per_pass;
    }
    // The first (m, l) pairs and UN accumulator rows are requested before anything waits: with the usual handful of partials per row
    // this is all there is to read.
    float2 ml_first = make_float2(-INFINITY, 0.0f);
    if (lane < n_part) ml_first = *reinterpret_cast<const float2 *>(part_ml + (prow0 + static_cast<int64_t>(lane) * pstride) * 2);
    float x[UN][CPT];
    auto request = [&](int j0) __attribute__((always_inline)) {   // rows j0 .. + UN - 1, the last one's for those past it
        static_for<0, UN / 8>([&](auto gg) {
            constexpr int g = 8 * decltype(gg)::value;
            if (j0 + g >= n_part) return;   // (uniform)
#pragma unroll
            for (int u = g; u < g + 8; ++u)
                load_channels<CPT>(part_acc + (prow0 + static_cast<int64_t>(min(j0 + u, n_part - 1)) * pstride) * D + CPT * lane, x[u]);
        });
    };
    request(0);
    float m_win = -INFINITY, l_win = 0.0f, a_win[CPT];
    if constexpr (WIN != 0) {
        asm volatile("" ::: "memory");   // (or the loads are moved to their use)
        win.run(shp, win_smem, orow, seq, kvh, own_len, win_len, m_win, l_win, a_win);
    }
    float m = fmaxf(-INFINITY, ml_first.x);   // (a NaN stays out)
    for (int j = lane + kWave; j < n_part; j += kWave) m = fmaxf(m, part_ml[(prow0 + static_cast<int64_t>(j) * pstride) * 2]);
    m = wave_max(m);
    // the many-row kernel's maxima are in units of log2, the others' and the window's in natural ones
    const float unit = shp.rows_per_pass >= 128 ? 1.0f : kLog2e;
    if constexpr (WIN != 0) {
        m_win *= kLog2e / unit;
        m = fmaxf(m, m_win);
    }
    float a[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) a[c] = 0.0f;
    float l = 0.0f;
    if constexpr (WIN != 0) {
        const float f = (m_win == -INFINITY) ? 0.0f : exp2_raw((m_win - m) * unit);
        if (lane == 0) l = f * l_win;
#pragma unroll
        for (int c = 0; c < CPT; ++c) a[c] = f * a_win[c];
    }
    for (int j0 = 0; j0 < n_part; j0 += kWave) {
        const int j = j0 + lane;
        float f = 0.0f;
        if (j < n_part) {
            float2 ml = ml_first;
            if (j0 > 0) ml = *reinterpret_cast<const float2 *>(part_ml + (prow0 + static_cast<int64_t>(j) * pstride) * 2);
            f = (ml.x == -INFINITY) ? 0.0f : exp2_raw((ml.x - m) * unit);
            l += f * ml.y;
        }
        __syncthreads();
        wgt[lane] = f;
        __syncthreads();
        const int nj = min(kWave, n_part - j0);
        for (int jj = 0; jj < nj; jj += UN) {
            if (j0 + jj > 0) request(j0 + jj);
            auto take = [&](int u) __attribute__((always_inline)) {
                const float fj = wgt[jj + u];
#pragma unroll
                for (int c = 0; c < CPT; ++c) a[c] = fmaf(fj, x[u][c], a[c]);
            };
            if (jj + UN <= nj) {
#pragma unroll
                for (int u = 0; u < UN; ++u) take(u);
            } else {   // (partials past the last stay out: at weight zero an infinity in it would count again, as 0 * inf)
                static_for<0, UN / 8>([&](auto gg) {
                    constexpr int g = 8 * decltype(gg)::value;
                    if (jj + g >= nj) return;   // (uniform, as below)
                    static_for<g, g + 8>([&](auto uu) {
                        if (jj + decltype(uu)::value < nj) take(decltype(uu)::value);
                    });
                });
            }
        }
    }
    l = wave_sum(l);
#pragma unroll
    for (int c = 0; c < CPT; ++c) a[c] = (l > 0.0f) ? a[c] / l : 0.0f;
    store_channels<CPT>(out + orow * D + CPT * lane, a);
}

}  // namespace octopus

#endif
