// Internal declarations shared by the host dispatch code and the HIP kernels.
#ifndef OCTOPUS_INTERNAL_H_
#define OCTOPUS_INTERNAL_H_

#include <stddef.h>
#include <stdint.h>

#include "octopus.h"

namespace octopus {

// Centroids handed to kernels by value (kernel argument space); boundaries are
// recomputed on the device as midpoints, exactly as the host computes them.
constexpr int kMaxLevels = OCTOPUS_MAX_LEVELS;   // 64: up to 6 bits per index (the pairs swept in App. D)
struct DeviceBooks {
    float c_xi[2][kMaxLevels];
    float c_rho[2][kMaxLevels];
};

inline DeviceBooks device_books(const octopus_codebooks_t &cb) {
    DeviceBooks books;
    for (int c = 0; c < 2; ++c)
        for (int k = 0; k < kMaxLevels; ++k) {
            books.c_xi[c][k] = cb.c_xi[c][k];
            books.c_rho[c][k] = cb.c_rho[c][k];
        }
    return books;
}

// Floats per rotated query row in the workspace: 3 * n_tri rounded up to 4.
inline int q_row_stride(int n_tri) { return (3 * n_tri + 3) & ~3; }

// How the decode kernels divide a call's steps (octopus_decode.hpp).
enum : int { kDivideEvenly, kBlockEach, kPairsWeighed, kPairEach };

// Paged cache: logical 64-token tile j of sequence s lives in page table[s * stride + j] of a pool of n_pages
// pages; table NULL: the contiguous cache.
struct PageTable {
    const int32_t *table;
    int32_t stride;
    int32_t n_pages;
};

// Native-precision window of a hybrid cache: the kernel that merges a row's partial results adds the window's (octopus_merge.hpp).
struct WindowCall {
    const void *k_win, *v;       // keys of the window; the value rows that follow the compressed tokens' (pt: in pages, t_capacity is what the table addresses)
    int64_t w_capacity;
    const int32_t *win_lens;
    float *scores_out;           // or NULL
    PageTable pt;
    int32_t k_is_bf16, v_is_bf16;
};

struct DecodeShape {
    int32_t n_seq, n_q_heads, n_kv_heads, n_q;
    int32_t heads_per_kv;   // n_q_heads / n_kv_heads
    int32_t rows_per_kv;    // n_q * heads_per_kv query rows sharing one KV head
    int32_t rows_per_pass;  // query rows one workgroup scores per key (1, 2, 4 or 8; 128, 256 or 512: many-row kernel)
    int32_t n_row_groups;   // ceil(rows_per_kv / rows_per_pass)
    int32_t n_splits;       // many-row kernel: workgroups sharing the tiles of one (sequence, KV head, row group)
    int32_t max_items;      // what the partials' part of the workspace is sized for (row groups of at most 8)
    int32_t max_len;        // host-side bound of the sequence lengths
    int32_t item_waves;     // wavefronts of the workgroup, which share a segment (4; 8: matrix-core kernel over quantised values up to d = 128 where its LDS fits)
    int32_t tiles_per_step; // 64-token tiles a wavefront takes per step (2 up to d = 128, else 1; 1: that kernel and decode_kernel_valu)
    int64_t t_capacity;
    // the call's queries, for the kernels that rotate the rows of their row group themselves (rotates_in_kernel)
    const void *q;
    const uint8_t *signs, *signs2;   // signs2: second rotation of the QJL residual, or NULL
    float scale;
    int32_t q_is_bf16;
    float *out;             // the call's output where every pair is one workgroup's and no merge follows, or NULL (direct_output)
    int32_t kind_known;     // kBlockEach or kPairEach where the host knows it whatever the lengths, else 0
    int32_t two_round_blocks;   // calls of one to two rounds of steps per workgroup go by blocks of two rounds (Division::set)
    int32_t pairs_fill;     // there may be as many (sequence, KV head, row group) pairs with tokens as workgroups (256)
    const WindowCall *window;   // host memory, for launch_merge: the call's window, or NULL
};

// Plans whose every class has a joint table (2 b_dir + b_nrm <= 10) score on the matrix cores where the kernel over bf16
// values or the matrix-core kernel over quantised values serves the call; those kernels rotate the queries themselves.
inline bool joint_plan(const octopus_plan_t &p) {
    for (int c = 0; c < p.n_class; ++c)
        if (2 * p.b_dir[c] + p.b_nrm[c] > 10) return false;
    return true;
}

// Workspace carve-up (all offsets multiples of 256 bytes).
struct Workspace {
    size_t q_rot_off, part_ml_off, part_acc_off, q2_off, total;
};

DecodeShape make_decode_shape(const octopus_plan_t &plan, int32_t n_seq, int32_t n_q_heads, int32_t n_kv_heads,
                              int32_t n_q, int64_t max_len, int64_t t_capacity, bool many_rows, int32_t rows_cap = 8,
                              int32_t vq_mfma_waves = 0, int32_t rows_min = 1, bool wide_rows = false);
// Row group the matrix-core kernel over quantised values would serve a call with (4 or 8 query rows), and
// whether such a kernel is built for the plan and value format (octopus_common.hip).
inline int32_t vq_mfma_rows(int32_t rows_per_kv) { return rows_per_kv <= 4 ? 4 : 8; }
// wavefronts per workgroup (4 or 8) of the matrix-core kernel over quantised values built for the shape, 0: none
int vq_mfma_available(const octopus_plan_t &plan, int32_t rows_per_pass, int32_t v_bits, int32_t v_group);
Workspace make_workspace(const octopus_plan_t &plan, const DecodeShape &s);

// Kernel launchers (defined in the .hip files).  Each returns a hipError_t cast to int.
// `q2` (NULL: not wanted): the queries rotated a second time with `signs2` for the QJL residual, [padded row][head_dim].
// (`work_plan`, and the rotation's `seq_lens`: not used; part of the launchers' signatures, which the host-side test drivers
// stub.)
int launch_rotate_queries(const octopus_plan_t &plan, const void *q, int q_dtype, const uint8_t *signs,
                          const DecodeShape &s, float scale, float *q_rot, const int32_t *seq_lens,
                          int32_t *work_plan, const uint8_t *signs2, float *q2, void *stream);
int launch_decode(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                  const void *v, int v_dtype, const int32_t *seq_lens, float *part_ml, float *part_acc,
                  float *scores_out, int32_t *work_plan, void *stream);
// bf16 values, row groups of at most qjl_rows_cap(plan)
int launch_decode_qjl(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                      const void *qjl, const float *q2, const void *v, const int32_t *seq_lens, float *part_ml,
                      float *part_acc, float *scores_out, int32_t *work_plan, void *stream);
// Query rows one workgroup of the QJL decode kernel serves at most (8); 0 if the plan is not built.
int qjl_rows_cap(const octopus_plan_t &plan);
// With s.window, of a native-precision window too.
int launch_merge(const octopus_plan_t &plan, const DecodeShape &s, const float *part_ml, const float *part_acc,
                 const int32_t *seq_lens, float *out, void *stream);
int launch_encode(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                  int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                  const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                  const uint8_t *signs2, void *qjl, void *stream);   // qjl NULL: no side-car

// Paged pools: the encoder writes each tile into its page of `k_pool` ([page][KV head] key tiles); the decode
// kernel reads key tiles from `k_pool` and bf16 value tiles ([page][KV head][64][head_dim]) from `v_pool`.
int launch_encode_paged(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                        int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                        const uint8_t *signs, void *k_pool, const PageTable &pt, const int32_t *start_pos,
                        void *stream, const uint8_t *signs2 = nullptr, void *qjl_pool = nullptr);   // qjl_pool: side-car pages
int launch_decode_paged(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *k_pool,
                        const void *v_pool, const PageTable &pt, const int32_t *seq_lens, float *part_ml,
                        float *part_acc, int32_t *work_plan, void *stream);
// ... with the QJL side-car in pages as well ([page][KV head] side-car tiles), q2 as for launch_decode_qjl
int launch_decode_paged_qjl(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *k_pool,
                            const void *qjl_pool, const float *q2, const void *v_pool, const PageTable &pt,
                            const int32_t *seq_lens, float *part_ml, float *part_acc, int32_t *work_plan, void *stream);

// The encoder with one of the rounding modes of App. E (OCTOPUS_ROUND_*), no side-car.
int launch_encode_rounding(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                           int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                           const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                           int32_t mode, void *stream);

// Value codec (group-quantised value rows) and decode attention over it.
int launch_encode_values(const void *v, int v_dtype, int64_t stride_seq, int64_t stride_tok, int64_t stride_head,
                         int32_t n_seq, int32_t n_kv_heads, int32_t n_new, int32_t head_dim, int32_t bits,
                         int32_t group, void *vq, int64_t t_capacity, const int32_t *start_pos, void *stream,
                         PageTable pt = PageTable{nullptr, 0, 0});   // pt: vq is a pool of [page][KV head][64] rows
int launch_decode_vq(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                     const void *vq, int v_bits, int v_group, const int32_t *seq_lens, float *part_ml,
                     float *part_acc, float *scores_out, int32_t *work_plan, void *stream,
                     PageTable pt = PageTable{nullptr, 0, 0});   // pt: cache and vq are pools of pages

// Measurement aid: plain streaming read of `bytes` bytes by n_blocks workgroups (non-temporal loads or not).
int launch_probe_read(const void *data, int64_t bytes, int nontemporal, int n_blocks, void *sink, void *stream);

// hipEventRecord(event, stream); returns a hipError_t cast to int.
int record_event(void *event, void *stream);

// True when every class's direction levels are those of the library's own codebook (to 2^-22 of a level) and its norm
// levels lie in [0, 1): the encoder then looks at four candidates per triplet instead of nine.
bool corner_levels(const octopus_codebooks_t &cb);

// True when every kernel family is instantiated for this plan (the six built bit widths of each head dimension).
bool plan_supported(const octopus_plan_t &plan);
// True for the extra (b_dir, b_nrm) pairs of the App. D sweep: plain encoder (local 3x3) and split-K decode over
// bf16 values only -- no score output, no QJL side-car, no quantised values, no pages, no many-row kernel.
bool plan_sweep_only(const octopus_plan_t &plan);

}  // namespace octopus

#endif
