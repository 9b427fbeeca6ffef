// Says which kernel shape the library's host side gives a decode call, without a GPU: the launchers are stubs that keep the
// shape they are handed.  Arguments, eight per call: kind, head_dim, bits per coordinate, n_seq, n_q_heads, n_kv_heads, n_q,
// max_len; one line per call: query rows per workgroup, row groups, splits, whether a merge is launched.  Kinds: 0 values in
// bf16, 1 the same over pages, 2 fp32 values, 3 / 4 quantised values by the matrix-core kernel of eight / four wavefronts, 5 the
// residual, 6 a window, 7 an output four bytes past its alignment; 13, 15 and 16 are 3, 5 and 6 over pages.
// Built by tests/test_launch_shapes.py from this file plus csrc/octopus_host.cpp.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "octopus_internal.h"

namespace octopus {
static DecodeShape g_shape;
static bool g_merged;
static int g_vq_waves;
static int show(const DecodeShape &s) {
    g_shape = s;
    g_merged = false;
    return 0;
}
int launch_rotate_queries(const octopus_plan_t &, const void *, int, const uint8_t *, const DecodeShape &, float, float *,
                          const int32_t *, int32_t *, const uint8_t *, float *, void *) { return 0; }
int launch_decode(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *, int,
                  const int32_t *, float *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_paged(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *,
                        const PageTable &, const int32_t *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_qjl(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *,
                      const float *, const void *, const int32_t *, float *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_paged_qjl(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *,
                            const float *, const void *, const PageTable &, const int32_t *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_vq(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *, int,
                     int, const int32_t *, float *, float *, float *, int32_t *, void *, PageTable) { return show(s); }
int launch_merge(const octopus_plan_t &, const DecodeShape &, const float *, const float *, const int32_t *, float *,
                 void *) { g_merged = true; return 0; }
int launch_encode(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t, int32_t, int32_t, int32_t,
                  const uint8_t *, void *, int64_t, const int32_t *, const uint8_t *, void *, void *) { return 0; }
int launch_encode_paged(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t, int32_t, int32_t,
                        int32_t, const uint8_t *, void *, const PageTable &, const int32_t *, void *, const uint8_t *, void *) { return 0; }
int launch_encode_rounding(const octopus_codebooks_t &, const void *, int, int64_t, int64_t, int64_t, int32_t, int32_t,
                           int32_t, const uint8_t *, void *, int64_t, const int32_t *, int32_t, void *) { return 0; }
int launch_encode_values(const void *, int, int64_t, int64_t, int64_t, int32_t, int32_t, int32_t, int32_t, int32_t,
                         int32_t, void *, int64_t, const int32_t *, void *, PageTable) { return 0; }
int launch_probe_read(const void *, int64_t, int, int, void *, void *) { return 0; }
int record_event(void *, void *) { return 0; }
bool plan_supported(const octopus_plan_t &) { return true; }
bool plan_sweep_only(const octopus_plan_t &) { return false; }
int qjl_rows_cap(const octopus_plan_t &) { return 8; }
int vq_mfma_available(const octopus_plan_t &, int32_t, int32_t, int32_t) { return g_vq_waves; }
}  // namespace octopus

int main(int argc, char **argv) {
    alignas(256) static unsigned char fake[4096];   // satisfies the alignment checks; the stubs never look behind it
    void *p = fake;
    const int32_t *ip = reinterpret_cast<const int32_t *>(fake);
    float *fp = reinterpret_cast<float *>(fake);
    for (int a = 1; a + 7 < argc; a += 8) {
        const int kind = std::atoi(argv[a]), d = std::atoi(argv[a + 1]);
        const int n_seq = std::atoi(argv[a + 3]), n_qh = std::atoi(argv[a + 4]), n_kv = std::atoi(argv[a + 5]), n_q = std::atoi(argv[a + 6]);
        const int64_t max_len = std::atoll(argv[a + 7]), cap = (max_len + 63) / 64 * 64;
        octopus_codebooks_t cb;
        if (octopus_build_codebooks(d, static_cast<float>(std::atof(argv[a + 2])), &cb) != OCTOPUS_OK) return 2;
        const size_t ws = octopus_attn_decode_workspace(&cb, n_seq, n_qh, n_kv, n_q, max_len);   // (only its size is looked at)
        const float scale = 0.1f;
        const int bf16 = OCTOPUS_DTYPE_BF16, n_pages = 1 << 20, pages = static_cast<int32_t>(cap / 64);
        float *out = kind == 7 ? fp + 1 : fp;
        octopus::g_vq_waves = kind % 10 == 3 ? 8 : (kind == 4 ? 4 : 0);
        int rc = -1;
        switch (kind) {
            case 0: case 7: case 2:
                rc = octopus_attn_decode(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, cap, p, kind == 2 ? OCTOPUS_DTYPE_F32 : bf16, ip,
                                         max_len, scale, out, nullptr, p, ws, nullptr);
                break;
            case 1:
                rc = octopus_attn_decode_paged(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, p, n_pages, ip, pages, ip, max_len, scale, out,
                                               p, ws, nullptr);
                break;
            case 3: case 4:
                rc = octopus_attn_decode_vq(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, cap, p, 3, 32, ip, max_len, scale, out, nullptr, p,
                                            ws, nullptr);
                break;
            case 5:
                rc = octopus_attn_decode_qjl(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, fake, p, p, cap, p, bf16, ip, max_len, scale, out,
                                             nullptr, p, ws, nullptr);
                break;
            case 6:
                rc = octopus_attn_decode_hybrid(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, cap, p, bf16, ip, max_len, p, bf16, 32, ip,
                                                scale, out, nullptr, p, ws, nullptr);
                break;
            case 13:
                rc = octopus_attn_decode_paged_vq(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, p, 3, 32, n_pages, ip, pages, ip, max_len,
                                                  scale, out, p, ws, nullptr);
                break;
            case 15:
                rc = octopus_attn_decode_paged_qjl(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, fake, p, p, p, n_pages, ip, pages, ip, max_len,
                                                   scale, out, p, ws, nullptr);
                break;
            case 16:
                rc = octopus_attn_decode_paged_hybrid(&cb, p, bf16, n_seq, n_qh, n_kv, n_q, fake, p, p, n_pages, ip, pages, ip, max_len, p,
                                                      bf16, 32, ip, scale, out, p, ws, nullptr);
                break;
        }
        if (rc != OCTOPUS_OK) { std::printf("error %d\n", rc); return 1; }
        const octopus::DecodeShape &s = octopus::g_shape;
        if ((s.out == nullptr) != octopus::g_merged) { std::printf("neither merged nor written by the kernel\n"); return 1; }
        std::printf("%d %d %d %d\n", s.rows_per_pass, s.n_row_groups, s.n_splits, octopus::g_merged ? 1 : 0);
    }
    return 0;
}
