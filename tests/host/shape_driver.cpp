// Says which kernel shape the library's host side gives a decode call, without a GPU: the launchers are stubs that print the
// shape they are handed.  Arguments, eight per call: paged (0 / 1), head_dim, bits per coordinate, n_seq, n_q_heads,
// n_kv_heads, n_q, max_len; one line per call: query rows per workgroup, row groups, splits.
// Built by tests/test_launch_shapes.py from this file plus csrc/octopus_host.cpp.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "octopus_internal.h"

namespace octopus {
static int show(const DecodeShape &s) {
    std::printf("%d %d %d\n", s.rows_per_pass, s.n_row_groups, s.n_splits);
    return 0;
}
int launch_rotate_queries(const octopus_plan_t &, const void *, int, const uint8_t *, const DecodeShape &, float, float *,
                          const int32_t *, int32_t *, const uint8_t *, float *, void *) { return 0; }
int launch_decode(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *, int,
                  const int32_t *, float *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_paged(const octopus_codebooks_t &, const DecodeShape &s, const float *, const void *, const void *,
                        const PageTable &, const int32_t *, float *, float *, int32_t *, void *) { return show(s); }
int launch_decode_qjl(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *, const void *,
                      const float *, const void *, const int32_t *, float *, float *, float *, int32_t *, void *) { return 0; }
int launch_decode_paged_qjl(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *, const void *,
                            const float *, const void *, const PageTable &, const int32_t *, float *, float *, int32_t *, void *) { return 0; }
int launch_decode_vq(const octopus_codebooks_t &, const DecodeShape &, const float *, const void *, const void *, int,
                     int, const int32_t *, float *, float *, float *, int32_t *, void *, PageTable) { return 0; }
int launch_merge(const octopus_plan_t &, const DecodeShape &, const float *, const float *, const int32_t *, float *,
                 const float *, const float *, void *) { return 0; }
int launch_window(const octopus_plan_t &, const DecodeShape &, const void *, int, const void *, int, int64_t,
                  const int32_t *, const void *, int, const int32_t *, float, float *, float *, float *, void *, PageTable) { return 0; }
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
int vq_mfma_available(const octopus_plan_t &, int32_t, int32_t, int32_t) { return 0; }
}  // namespace octopus

int main(int argc, char **argv) {
    alignas(256) static unsigned char fake[4096];   // satisfies the alignment checks; the stubs never look behind it
    void *p = fake;
    const int32_t *ip = reinterpret_cast<const int32_t *>(fake);
    float *fp = reinterpret_cast<float *>(fake);
    for (int a = 1; a + 7 < argc; a += 8) {
        const int paged = std::atoi(argv[a]), d = std::atoi(argv[a + 1]);
        const int n_seq = std::atoi(argv[a + 3]), n_qh = std::atoi(argv[a + 4]), n_kv = std::atoi(argv[a + 5]), n_q = std::atoi(argv[a + 6]);
        const int64_t max_len = std::atoll(argv[a + 7]), cap = (max_len + 63) / 64 * 64;
        octopus_codebooks_t cb;
        if (octopus_build_codebooks(d, static_cast<float>(std::atof(argv[a + 2])), &cb) != OCTOPUS_OK) return 2;
        const size_t ws = octopus_attn_decode_workspace(&cb, n_seq, n_qh, n_kv, n_q, max_len);   // (only its size is looked at)
        const int rc = paged ? octopus_attn_decode_paged(&cb, p, OCTOPUS_DTYPE_BF16, n_seq, n_qh, n_kv, n_q, fake, p, p, 1 << 20, ip,
                                                         static_cast<int32_t>(cap / 64), ip, max_len, 0.1f, fp, p, ws, nullptr)
                             : octopus_attn_decode(&cb, p, OCTOPUS_DTYPE_BF16, n_seq, n_qh, n_kv, n_q, fake, p, cap, p,
                                                   OCTOPUS_DTYPE_BF16, ip, max_len, 0.1f, fp, nullptr, p, ws, nullptr);
        if (rc != OCTOPUS_OK) { std::printf("error %d\n", rc); return 1; }
    }
    return 0;
}
