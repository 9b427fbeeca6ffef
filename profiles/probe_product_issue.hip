// What a product, a multiply-add and an exponential cost a SIMD of MI355X (gfx950): cycles of s_memtime per loop body and wavefront, the slowest
// wavefront of one workgroup of 1 to 4 wavefronts per SIMD.  A body is 8 products v_mfma_f32_32x32x16_bf16 (or 16 of 16x16x32, the same
// operations), 64 multiply-adds v_fma_f32, 64 exponentials v_exp_f32, or products with 8 (4) multiply-adds after each.
//   hipcc -O3 -std=c++17 --offload-arch=gfx950 -Xclang -target-feature -Xclang -packed-fp32-ops probe_product_issue.hip -o probe && ./probe
// Measured:
//   64 multiply-adds                                             1 per SIMD: 312.1 cycles of the counter
//   64 multiply-adds                                             2 per SIMD: 312.1 cycles of the counter
//   64 multiply-adds                                             3 per SIMD: 511.1 cycles of the counter
//   64 multiply-adds                                             4 per SIMD: 605.9 cycles of the counter
//   8 products 32x32x16                                          1 per SIMD: 264.3 cycles of the counter
//   8 products 32x32x16                                          2 per SIMD: 519.3 cycles of the counter
//   8 products 32x32x16                                          3 per SIMD: 775.5 cycles of the counter
//   8 products 32x32x16                                          4 per SIMD: 1031.4 cycles of the counter
//   8 products 32x32x16, 64 multiply-adds                        1 per SIMD: 352.5 cycles of the counter
//   8 products 32x32x16, 64 multiply-adds                        2 per SIMD: 653.7 cycles of the counter
//   8 products 32x32x16, 64 multiply-adds                        3 per SIMD: 960.1 cycles of the counter
//   8 products 32x32x16, 64 multiply-adds                        4 per SIMD: 1266.3 cycles of the counter
//   64 exponentials                                              1 per SIMD: 544.1 cycles of the counter
//   64 exponentials                                              2 per SIMD: 1054.0 cycles of the counter
//   64 exponentials                                              3 per SIMD: 1566.1 cycles of the counter
//   64 exponentials                                              4 per SIMD: 2078.2 cycles of the counter
//   16 products 16x16x32                                         1 per SIMD: 280.2 cycles of the counter
//   16 products 16x16x32                                         2 per SIMD: 533.2 cycles of the counter
//   16 products 16x16x32                                         3 per SIMD: 789.6 cycles of the counter
//   16 products 16x16x32                                         4 per SIMD: 1045.5 cycles of the counter
//   16 products 16x16x32, 64 multiply-adds                       1 per SIMD: 412.4 cycles of the counter
//   16 products 16x16x32, 64 multiply-adds                       2 per SIMD: 764.4 cycles of the counter
//   16 products 16x16x32, 64 multiply-adds                       3 per SIMD: 1121.1 cycles of the counter
//   16 products 16x16x32, 64 multiply-adds                       4 per SIMD: 1477.4 cycles of the counter
// Read: each further wavefront adds 256 for the products, 152 on average of four for the multiply-adds (one alone issues one every 4.9
// cycles), 306 for both, 512 for the exponentials: a product keeps others from issuing for about (306 - 152) / 8 = 19 of its 32 cycles.
#include <hip/hip_runtime.h>
#include <cstdio>
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
constexpr int kIter = 2000;
template <int SIZE, bool PRODUCTS, bool ADDS>
__global__ __launch_bounds__(1024) void body(float *out, unsigned long long *cycles) {
    bf16x8 a, b;
    for (int i = 0; i < 8; ++i) { a[i] = (__bf16)(0.001f * (threadIdx.x + i)); b[i] = (__bf16)(0.002f * (threadIdx.x - i)); }
    f32x16 acc[4];
    f32x4 acc4[8];
    float x[16];
    for (int i = 0; i < 4; ++i) for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    for (int i = 0; i < 8; ++i) for (int e = 0; e < 4; ++e) acc4[i][e] = 0.f;
    for (int i = 0; i < 16; ++i) x[i] = 0.01f * i;
    const float m = 0.999f, c = 0.001f * threadIdx.x;
    __syncthreads();
    const unsigned long long t0 = __builtin_readcyclecounter();
#pragma clang loop unroll(disable)
    for (int it = 0; it < kIter; ++it) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            if constexpr (PRODUCTS && SIZE == 32) acc[p % 4] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[p % 4], 0, 0, 0);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if constexpr (PRODUCTS && SIZE == 16) acc4[(2 * p + half) % 8] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc4[(2 * p + half) % 8], 0, 0, 0);
                if constexpr (SIZE == 1 && PRODUCTS)
#pragma unroll
                    for (int k = 0; k < 4; ++k) asm volatile("v_exp_f32 %0, %0" : "+v"(x[(8 * p + 4 * half + k) % 16]));
                if constexpr (ADDS)
#pragma unroll
                    for (int k = 0; k < 4; ++k) asm volatile("v_fma_f32 %0, %0, %1, %2" : "+v"(x[(8 * p + 4 * half + k) % 16]) : "v"(m), "v"(c));
            }
        }
    }
    const unsigned long long t1 = __builtin_readcyclecounter();
    float s = 0.f;
    for (int i = 0; i < 4; ++i) for (int e = 0; e < 16; ++e) s += acc[i][e];
    for (int i = 0; i < 8; ++i) for (int e = 0; e < 4; ++e) s += acc4[i][e];
    for (int i = 0; i < 16; ++i) s += x[i];
    out[threadIdx.x] = s;
    if (threadIdx.x % 64 == 0) cycles[threadIdx.x / 64] = t1 - t0;
}
template <int SIZE, bool P, bool A>
static int show(const char *what, float *out, unsigned long long *cyc) {
    for (int waves = 4; waves <= 16; waves += 4) {
        unsigned long long h[16] = {};
        for (int rep = 0; rep < 3; ++rep) {
            hipLaunchKernelGGL((body<SIZE, P, A>), dim3(1), dim3(64 * waves), 0, 0, out, cyc);
            if (hipDeviceSynchronize() != hipSuccess) return 1;
        }
        if (hipMemcpy(h, cyc, 8 * waves, hipMemcpyDeviceToHost) != hipSuccess) return 1;
        unsigned long long most = 0;
        for (int w = 0; w < waves; ++w) most = h[w] > most ? h[w] : most;
        std::printf("%-60s %d per SIMD: %.1f cycles of the counter\n", what, waves / 4, double(most) / kIter);
    }
    return 0;
}
int main() {
    float *out; unsigned long long *cyc;
    if (hipMalloc(&out, 1024 * 4) != hipSuccess || hipMalloc(&cyc, 128) != hipSuccess) return 1;
    int rc = 0;
    rc |= show<32, false, true>("64 multiply-adds", out, cyc);
    rc |= show<32, true, false>("8 products 32x32x16", out, cyc);
    rc |= show<32, true, true>("8 products 32x32x16, 64 multiply-adds", out, cyc);
    rc |= show<1, true, false>("64 exponentials", out, cyc);
    rc |= show<16, true, false>("16 products 16x16x32", out, cyc);
    rc |= show<16, true, true>("16 products 16x16x32, 64 multiply-adds", out, cyc);
    return rc;
}
