// Dispatch by head dimension and the kernels that do not depend on the bit width.
#include "octopus_decode.hpp"
#include "octopus_merge.hpp"

namespace octopus {

bool plan_supported_d64(const octopus_plan_t &);
bool plan_supported_d128(const octopus_plan_t &);
bool plan_supported_d256(const octopus_plan_t &);
#define OCTOPUS_DECL(D)                                                                                            \
    int launch_decode_mfma_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *,     \
                                const void *, const int32_t *, float *, float *, float *, void *);                 \
    int launch_decode_mfma_scores_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *,            \
                                       const void *, const void *, const int32_t *, float *, float *, float *,     \
                                       void *);                                                                    \
    int launch_decode_valu_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *,     \
                                const void *, const int32_t *, float *, float *, float *, void *);                 \
    int launch_encode_d##D(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t, int32_t,     \
                           int32_t, int32_t, const uint8_t *, void *, int64_t, const int32_t *, const uint8_t *, void *, \
                           void *);                                                                                \
    int launch_decode_qjl_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *,      \
                               const void *, const float *, const void *, const int32_t *, float *, float *,       \
                               float *, void *);                                                                   \
    int qjl_rows_cap_d##D(const octopus_plan_t &);                                                                 \
    int vq_mfma_available_d##D(const octopus_plan_t &, int, int, int);                                             \
    int launch_decode_vq_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *,       \
                              const void *, int, int, const int32_t *, float *, float *, float *,                  \
                              void *, const PageTable &);                                                          \
    int launch_encode_rounding_d##D(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t,     \
                                    int32_t, int32_t, int32_t, const uint8_t *, void *, int64_t, const int32_t *,  \
                                    int32_t, void *);                                                              \
    int launch_decode_paged_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *,    \
                                 const void *, const PageTable &, const int32_t *, float *, float *,               \
                                 void *);                                                                          \
    int launch_encode_paged_d##D(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t,        \
                                 int32_t, int32_t, int32_t, const uint8_t *, void *, const PageTable &,            \
                                 const int32_t *, const uint8_t *, void *, void *);                                \
    int launch_decode_paged_qjl_d##D(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *, \
                                     const void *, const float *, const void *, const PageTable &, const int32_t *, \
                                     float *, float *, void *);
OCTOPUS_DECL(64)
OCTOPUS_DECL(128)
OCTOPUS_DECL(256)
#undef OCTOPUS_DECL

// Measurement aid: a plain streaming read of `bytes` bytes (16 bytes per lane, every workgroup walks its own
// contiguous share front to back, 8 loads in flight per lane), with or without the non-temporal hint.
template <bool NT>
__global__ __launch_bounds__(256) void probe_read_kernel(const uint32_t *__restrict__ p, int64_t units_per_block,
                                                         uint32_t *__restrict__ sink) {
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    const u32x4_t *base = reinterpret_cast<const u32x4_t *>(p) + static_cast<int64_t>(blockIdx.x) * units_per_block;
    uint32_t acc = 0;
    for (int64_t i = threadIdx.x; i < units_per_block; i += 256 * 8) {
        u32x4_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t j = min(i + u * 256, units_per_block - 1);
            x[u] = NT ? __builtin_nontemporal_load(base + j) : base[j];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += x[u].x ^ x[u].y ^ x[u].z ^ x[u].w;
    }
    if (acc == 0x9e3779b9u) sink[0] = acc;   // (keeps the loads alive; practically never taken)
}

int launch_probe_read(const void *data, int64_t bytes, int nontemporal, int n_blocks, void *sink, void *stream) {
    const int64_t units = bytes / 16 / n_blocks;
    if (nontemporal)
        hipLaunchKernelGGL(probe_read_kernel<true>, dim3(n_blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                           static_cast<const uint32_t *>(data), units, static_cast<uint32_t *>(sink));
    else
        hipLaunchKernelGGL(probe_read_kernel<false>, dim3(n_blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                           static_cast<const uint32_t *>(data), units, static_cast<uint32_t *>(sink));
    return static_cast<int>(hipGetLastError());
}

// the pairs of the App. D sweep (head dimension 128 only): plain encoder and bf16-value split-K decode
bool plan_supported_sweep_d128(const octopus_plan_t &);
int launch_decode_sweep_d128(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *, const void *,
                             const int32_t *, float *, float *, void *);
int launch_encode_sweep_d128(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t, int32_t, int32_t,
                             int32_t, const uint8_t *, void *, int64_t, const int32_t *, void *);

int record_event(void *event, void *stream) {
    return static_cast<int>(hipEventRecord(static_cast<hipEvent_t>(event), static_cast<hipStream_t>(stream)));
}

bool plan_sweep_only(const octopus_plan_t &plan) { return plan.head_dim == 128 && plan_supported_sweep_d128(plan); }

bool plan_supported(const octopus_plan_t &plan) {
    switch (plan.head_dim) {
        case 64: return plan_supported_d64(plan);
        case 128: return plan_supported_d128(plan);
        case 256: return plan_supported_d256(plan);
        default: return false;
    }
}

int launch_decode(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                  const void *v, int v_dtype, const int32_t *seq_lens, float *part_ml, float *part_acc,
                  float *scores_out, int32_t *, void *stream) {
    if (plan_sweep_only(cb.plan)) {
        if (v_dtype != OCTOPUS_DTYPE_BF16 || scores_out != nullptr) return static_cast<int>(hipErrorInvalidValue);
        return launch_decode_sweep_d128(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, stream);
    }
    // kernel family: 0 matrix cores, 1 matrix cores with score output, 2 vector units (fp32 values)
    const int family = v_dtype == OCTOPUS_DTYPE_BF16 ? (scores_out != nullptr ? 1 : 0) : 2;
#define OCTOPUS_GO(D)                                                                                                   \
    case D:                                                                                                             \
        return family == 0   ? launch_decode_mfma_d##D(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out,  \
                                                       stream)                                                          \
               : family == 1 ? launch_decode_mfma_scores_d##D(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc,       \
                                                              scores_out, stream)                            \
                             : launch_decode_valu_d##D(cb, s, q_rot, cache, v, seq_lens, part_ml, part_acc, scores_out,  \
                                                       stream);
    switch (cb.plan.head_dim) {
        OCTOPUS_GO(64)
        OCTOPUS_GO(128)
        OCTOPUS_GO(256)
        default: return static_cast<int>(hipErrorInvalidValue);
    }
#undef OCTOPUS_GO
}

int launch_decode_vq(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                     const void *vq, int v_bits, int v_group, const int32_t *seq_lens, float *part_ml,
                     float *part_acc, float *scores_out, int32_t *, void *stream, PageTable pt) {
    switch (cb.plan.head_dim) {
        case 64: return launch_decode_vq_d64(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream, pt);
        case 128: return launch_decode_vq_d128(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream, pt);
        case 256: return launch_decode_vq_d256(cb, s, q_rot, cache, vq, v_bits, v_group, seq_lens, part_ml, part_acc, scores_out, stream, pt);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int vq_mfma_available(const octopus_plan_t &plan, int32_t rows_per_pass, int32_t v_bits, int32_t v_group) {
    if (plan_sweep_only(plan)) return 0;
    switch (plan.head_dim) {
        case 64: return vq_mfma_available_d64(plan, rows_per_pass, v_bits, v_group);
        case 128: return vq_mfma_available_d128(plan, rows_per_pass, v_bits, v_group);
        case 256: return vq_mfma_available_d256(plan, rows_per_pass, v_bits, v_group);
        default: return 0;
    }
}

int qjl_rows_cap(const octopus_plan_t &plan) {
    switch (plan.head_dim) {
        case 64: return qjl_rows_cap_d64(plan);
        case 128: return qjl_rows_cap_d128(plan);
        case 256: return qjl_rows_cap_d256(plan);
        default: return 0;
    }
}

int launch_decode_qjl(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *cache,
                      const void *qjl, const float *q2, const void *v, const int32_t *seq_lens, float *part_ml,
                      float *part_acc, float *scores_out, int32_t *, void *stream) {
    switch (cb.plan.head_dim) {
        case 64: return launch_decode_qjl_d64(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 128: return launch_decode_qjl_d128(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream);
        case 256: return launch_decode_qjl_d256(cb, s, q_rot, cache, qjl, q2, v, seq_lens, part_ml, part_acc, scores_out, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int launch_encode(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                  int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                  const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                  const uint8_t *signs2, void *qjl, void *stream) {
    if (plan_sweep_only(cb.plan)) {
        if (qjl != nullptr) return static_cast<int>(hipErrorInvalidValue);
        return launch_encode_sweep_d128(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new,
                                        signs, cache, t_capacity, start_pos, stream);
    }
    switch (cb.plan.head_dim) {
        case 64: return launch_encode_d64(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, signs2, qjl, stream);
        case 128: return launch_encode_d128(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, signs2, qjl, stream);
        case 256: return launch_encode_d256(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, signs2, qjl, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int launch_decode_paged(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *k_pool,
                        const void *v_pool, const PageTable &pt, const int32_t *seq_lens, float *part_ml,
                        float *part_acc, int32_t *, void *stream) {
    switch (cb.plan.head_dim) {
        case 64: return launch_decode_paged_d64(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 128: return launch_decode_paged_d128(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 256: return launch_decode_paged_d256(cb, s, q_rot, k_pool, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int launch_encode_paged(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                        int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                        const uint8_t *signs, void *k_pool, const PageTable &pt, const int32_t *start_pos,
                        void *stream, const uint8_t *signs2, void *qjl_pool) {
    switch (cb.plan.head_dim) {
        case 64: return launch_encode_paged_d64(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, k_pool, pt, start_pos, signs2, qjl_pool, stream);
        case 128: return launch_encode_paged_d128(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, k_pool, pt, start_pos, signs2, qjl_pool, stream);
        case 256: return launch_encode_paged_d256(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, k_pool, pt, start_pos, signs2, qjl_pool, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int launch_decode_paged_qjl(const octopus_codebooks_t &cb, const DecodeShape &s, const float *q_rot, const void *k_pool,
                            const void *qjl_pool, const float *q2, const void *v_pool, const PageTable &pt,
                            const int32_t *seq_lens, float *part_ml, float *part_acc, int32_t *, void *stream) {
    switch (cb.plan.head_dim) {
        case 64: return launch_decode_paged_qjl_d64(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 128: return launch_decode_paged_qjl_d128(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        case 256: return launch_decode_paged_qjl_d256(cb, s, q_rot, k_pool, qjl_pool, q2, v_pool, pt, seq_lens, part_ml, part_acc, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

int launch_encode_rounding(const octopus_codebooks_t &cb, const void *keys, int key_dtype, int64_t stride_seq,
                           int64_t stride_tok, int64_t stride_head, int32_t n_seq, int32_t n_kv_heads, int32_t n_new,
                           const uint8_t *signs, void *cache, int64_t t_capacity, const int32_t *start_pos,
                           int32_t mode, void *stream) {
    switch (cb.plan.head_dim) {
        case 64: return launch_encode_rounding_d64(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, mode, stream);
        case 128: return launch_encode_rounding_d128(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, mode, stream);
        case 256: return launch_encode_rounding_d256(cb, keys, key_dtype, stride_seq, stride_tok, stride_head, n_seq, n_kv_heads, n_new, signs, cache, t_capacity, start_pos, mode, stream);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

template <int D>
static int rotate_d(const DecodeShape &s, float *q_rot, float *q2, hipStream_t stream) {
    constexpr int QS = (3 * ((D + 2) / 3) + 3) & ~3;
    const int64_t rows = static_cast<int64_t>(s.n_seq) * s.n_kv_heads * s.n_row_groups * s.rows_per_pass;
    hipLaunchKernelGGL((rotate_queries_kernel<D, QS>), dim3(static_cast<unsigned>(rows)), dim3(kWave), 0, stream, s, q_rot, q2);
    return static_cast<int>(hipGetLastError());
}

int launch_rotate_queries(const octopus_plan_t &plan, const void *q, int q_dtype, const uint8_t *signs,
                          const DecodeShape &s, float scale, float *q_rot, const int32_t *, int32_t *,
                          const uint8_t *signs2, float *q2, void *stream) {
    DecodeShape t = s;
    t.q = q;
    t.q_is_bf16 = q_dtype == OCTOPUS_DTYPE_BF16 ? 1 : 0;
    t.signs = signs;
    t.signs2 = signs2;
    t.scale = scale;
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (plan.head_dim) {
        case 64: return rotate_d<64>(t, q_rot, q2, st);
        case 128: return rotate_d<128>(t, q_rot, q2, st);
        case 256: return rotate_d<256>(t, q_rot, q2, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

// Partial rows in flight per wavefront of the merge: 8, or 32 where a row may have more than 8 partials and the rows are few enough
// to leave registers (more rows keep the memory busy with 8: 16288 rows of 4 partials take the same either way).  A row of many
// partials was a chain of round trips, one per 8: one KV head of four rows over 100000 tokens 31.7 -> 23.6 us, 8 of one row over 20000
// 19.1 -> 18.1, two of four over 40000 at d = 256 34.5 -> 31.6, one of eight rows over 41127 with a window 32.3 -> 30.6.  Calls of up to 8
// partials can be slower with the longer code (one fp32 row over 4096 tokens 17.3 -> 17.7), but how many a row has depends on the lengths:
// counted is what it has at most, a sequence of max_len tokens alone.  So calls of many equal pairs, two or three partials a row,
// take the longer code too, and pay nothing for it: 8 / 32 in flight, 16 x 32768 tokens, 8 KV heads of four rows 206.1 / 205.4 us, 32 x 8000
// 109.5 / 109.4, 8 x 8000, eight rows 37.6 / 37.2, d = 64, 24 x 8000, eight rows 53.8 / 54.3, d = 256, 32 x 8000, two rows 200.6 / 200.2.
static bool deep_merge(const DecodeShape &s, int64_t rows) {
    const int64_t round = static_cast<int64_t>(kWave) * s.tiles_per_step * s.item_waves * (s.two_round_blocks != 0 ? 2 : 1);
    const int64_t most = s.rows_per_pass >= 128 ? s.n_splits : (s.max_len + round - 1) / round;
    return rows <= 4096 && most > 8;
}

template <int D>
static int merge_d(const DecodeShape &s, const float *part_ml, const float *part_acc, const int32_t *seq_lens, float *out,
                   hipStream_t stream) {
    const int64_t rows = static_cast<int64_t>(s.n_seq) * s.n_q * s.n_q_heads;
    auto go = [&](auto kernel, const WindowCall &w) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(rows)), dim3(kWave), 0, stream, s, w, part_ml, part_acc, seq_lens, out);
    };
    // (with a window the values are bf16 or, over the vector-unit kernel's two-round blocks, fp32)
    const WindowCall *w = s.window;
    const bool two = s.two_round_blocks != 0;
    if (w != nullptr && two && w->v_is_bf16) return static_cast<int>(hipErrorInvalidValue);
    auto depth = [&](auto un) {
        constexpr int UN = decltype(un)::value;
        if (w == nullptr) {
            if (two) go(merge_kernel<D, true, 0, UN>, WindowCall{}); else go(merge_kernel<D, false, 0, UN>, WindowCall{});
        } else if (w->v_is_bf16) {
            if (w->k_is_bf16) go(merge_kernel<D, false, 4, UN>, *w); else go(merge_kernel<D, false, 3, UN>, *w);
        } else {
            if (w->k_is_bf16) go(merge_kernel<D, true, 2, UN>, *w); else go(merge_kernel<D, true, 1, UN>, *w);
        }
    };
    if (deep_merge(s, rows)) depth(std::integral_constant<int, 32>{}); else depth(std::integral_constant<int, 8>{});
    return static_cast<int>(hipGetLastError());
}

int launch_merge(const octopus_plan_t &plan, const DecodeShape &s, const float *part_ml, const float *part_acc,
                 const int32_t *seq_lens, float *out, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (plan.head_dim) {
        case 64: return merge_d<64>(s, part_ml, part_acc, seq_lens, out, st);
        case 128: return merge_d<128>(s, part_ml, part_acc, seq_lens, out, st);
        case 256: return merge_d<256>(s, part_ml, part_acc, seq_lens, out, st);
        default: return static_cast<int>(hipErrorInvalidValue);
    }
}

}  // namespace octopus
