// Native-precision window of a hybrid cache (Sec. 4, default recipe: a short residual window of recent
// tokens kept uncompressed).  The window's tokens follow the compressed ones of their sequence; their
// keys are read as stored, their scores are the plain scale * q . k, and the partial (m, l, acc) of the
// window joins the split partials of the compressed part in the merge (flash-decoding identity, App. A).
#ifndef OCTOPUS_WINDOW_HPP_
#define OCTOPUS_WINDOW_HPP_

#include "octopus_decode.hpp"

namespace octopus {

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
template <int D, bool k_is_bf16, bool v_is_bf16>
__global__ __launch_bounds__(kWave) void window_kernel(DecodeShape shp, const void *__restrict__ q, int q_is_bf16,
                                                       const void *__restrict__ k_win,
                                                       int64_t w_capacity, const int32_t *__restrict__ win_lens,
                                                       const void *__restrict__ v,
                                                       const int32_t *__restrict__ seq_lens, float scale,
                                                       float *__restrict__ win_ml, float *__restrict__ win_acc,
                                                       float *__restrict__ scores_out, PageTable pt) {
    constexpr int CPT = D / kWave;      // channels per lane: CPT lane .. + CPT - 1
    constexpr int KW = D / (k_is_bf16 ? 8 : 4);                       // 16-byte words of a key row
    constexpr int VW = v_is_bf16 ? (CPT + 1) / 2 : CPT;               // 32-bit words of a lane's channels
    constexpr int VB = D <= 128 ? 32 : 16;   // value rows in flight
    constexpr bool STAGED = KW <= 32;   // (a longer row does not fit a lane's registers: read as it is used)
    constexpr int RPI = kWave / KW > 0 ? kWave / KW : 1;   // key rows per load instruction
    __shared__ float qs[D];
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    __shared__ u32x4_t rows[STAGED ? kWave : 1][STAGED ? KW + 1 : 1];
    const int lane = threadIdx.x;
    const int64_t orow = blockIdx.x;  // (seq, qi, head)
    const int head = static_cast<int>(orow % shp.n_q_heads);
    const int seq = static_cast<int>(orow / (static_cast<int64_t>(shp.n_q_heads) * shp.n_q));
    const int kvh = head / shp.heads_per_kv;
    const int64_t pair = static_cast<int64_t>(seq) * shp.n_kv_heads + kvh;
    const int asked_len = seq_lens[seq], asked_win = win_lens[seq];
    // the key rows of a chunk: RPI rows per instruction, those past the window's capacity are its last one
    u32x4_t key[STAGED ? KW : 1];
    const char *k_pair = static_cast<const char *>(k_win) + pair * w_capacity * (KW * 16);
    auto request_keys = [&](int64_t j0) __attribute__((always_inline)) {
        if constexpr (STAGED) {
#pragma unroll
            for (int e = 0; e < KW; ++e) {
                const int64_t row = min(j0 + e * RPI + lane / KW, w_capacity - 1);
                key[e] = *reinterpret_cast<const u32x4_t *>(k_pair + row * (KW * 16) + (lane % KW) * 16);
            }
        }
    };
    request_keys(0);   // (the buffer has at least one row per (sequence, KV head), whatever the lengths)
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int64_t i = orow * D + c * kWave + lane;
        const float x = q_is_bf16 ? __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(q)[i]) << 16)
                                  : static_cast<const float *>(q)[i];
        qs[c * kWave + lane] = x * scale;
    }
    __syncthreads();

    const int64_t len = min(max(asked_len, 0), shp.max_len);   // clamped like every other kernel's
    // the window's tokens must fit behind the compressed ones in the value buffer
    const int64_t n_win = max(int64_t{0}, min(min(static_cast<int64_t>(asked_win), w_capacity), shp.t_capacity - len));

    float m_run = -INFINITY, l_run = 0.0f, acc[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) acc[c] = 0.0f;
    for (int64_t j0 = 0; j0 < n_win; j0 += kWave) {
        const int nj = static_cast<int>(min(static_cast<int64_t>(kWave), n_win - j0));
        if (j0 > 0) request_keys(j0);
        // where the chunk's value rows lie: 64 tokens are in at most two pages
        const int64_t t0 = len + j0;
        int64_t first = pair * shp.t_capacity + t0, second = first;   // row of token t0, and (less the tokens before) of the next page
        int split = kWave;                                            // tokens of the chunk in the first page
        if (pt.table != nullptr) {
            const int32_t *pages = pt.table + static_cast<int64_t>(seq) * pt.stride;
            const int page0 = pages[t0 / kWave], page1 = pages[(t0 + nj - 1) / kWave];
            split = kWave - static_cast<int>(t0 % kWave);
            first = (static_cast<int64_t>(min(max(page0, 0), pt.n_pages - 1)) * shp.n_kv_heads + kvh) * kWave + t0 % kWave;
            second = (static_cast<int64_t>(min(max(page1, 0), pt.n_pages - 1)) * shp.n_kv_heads + kvh) * kWave - split;
        }
        uint32_t x[VB][VW];
        auto request_values = [&](int jb) __attribute__((always_inline)) {   // (rows past the chunk's end: its last one)
#pragma unroll
            for (int u = 0; u < VB; ++u) {
                if (u % 8 == 0 && jb + u >= nj) break;   // (uniform)
                const int j = min(jb + u, nj - 1);
                const int64_t row = (j < split ? first : second) + j;
                if constexpr (v_is_bf16 && CPT == 1) {
                    x[u][0] = static_cast<const uint16_t *>(v)[row * D + lane];
                } else {
                    const uint32_t *vp = static_cast<const uint32_t *>(v) + row * (D / (v_is_bf16 ? 2 : 1)) + lane * VW;
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
            for (int e = 0; e < KW; ++e) rows[e * RPI + lane / KW][lane % KW] = key[e];
            __syncthreads();
        }
        float s = -INFINITY;
        if (lane < nj) {
            float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            const u32x4_t *own = STAGED ? &rows[lane][0] : reinterpret_cast<const u32x4_t *>(k_pair + (j0 + lane) * (KW * 16));
#pragma unroll 16
            for (int e = 0; e < KW; ++e) {
                const u32x4_t x4 = own[e];
                const uint32_t w4[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    if constexpr (k_is_bf16) {
                        dot[h] = fmaf(qs[8 * e + 2 * h], __uint_as_float(w4[h] << 16), dot[h]);
                        dot[h] = fmaf(qs[8 * e + 2 * h + 1], __uint_as_float(w4[h] & 0xffff0000u), dot[h]);
                    } else {
                        dot[h] = fmaf(qs[4 * e + h], __uint_as_float(w4[h]), dot[h]);
                    }
                }
            }
            s = (dot[0] + dot[1]) + (dot[2] + dot[3]);
            if (scores_out != nullptr) scores_out[orow * shp.t_capacity + len + j0 + lane] = s;
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
    if (lane == 0) {
        win_ml[orow * 2] = m_run;
        win_ml[orow * 2 + 1] = l_run;
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) win_acc[orow * D + CPT * lane + c] = acc[c];
}

}  // namespace octopus

#endif
