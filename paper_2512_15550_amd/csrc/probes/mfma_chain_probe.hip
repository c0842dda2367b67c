// Check of the property the exact list build rests on, not part of the library: a chain of four v_mfma_f32_32x32x2f32 from a
// zero accumulator gives, bit for bit, eight fused multiply-adds one after the other in the order of k.  2 M results on normal
// values, bf16 values, values over 2^-30 .. 2^30 and values whose products and sums are subnormal, against fmaf on the host.  Prints the
// results that differ per kind; ends with status 1 if there are any.
// Build:  hipcc --offload-arch=gfx950 -O3 -o mfma_chain_probe mfma_chain_probe.hip   (python -m paper_2512_15550_amd.build --probes)
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#define CK(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) { printf("HIP error %s at %s:%d\n", hipGetErrorString(e_), __FILE__, __LINE__); exit(1);} } while (0)

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// one tile per wave: a [tile][32 rows][8], b [tile][8][32 columns], out [tile][32][32]; grid tiles / 4, 256 threads
__global__ __launch_bounds__(256) void chain_kernel(const float *a, const float *b, float *out)
{
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), ln = threadIdx.x & 63, col = ln & 31, half = ln >> 5;
    const float *at = a + (size_t)tile * 256 + col * 8, *bt = b + (size_t)tile * 256 + col;
    f32x16_t p = f32x16_t{};
#pragma unroll
    for (int i = 0; i < 4; ++i) p = __builtin_amdgcn_mfma_f32_32x32x2f32(at[2 * i + half], bt[(2 * i + half) * 32], p, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) out[(size_t)tile * 1024 + (8 * (r >> 2) + 4 * half + (r & 3)) * 32 + col] = p[r];
}

int main()
{
    constexpr int kTiles = 512;
    const char *kind[4] = {"normal", "bf16", "wide", "subnormal"};
    std::vector<float> a(kTiles * 256), b(kTiles * 256), out(kTiles * 1024);
    float *da, *db, *dout;
    CK(hipMalloc(&da, a.size() * 4)); CK(hipMalloc(&db, b.size() * 4)); CK(hipMalloc(&dout, out.size() * 4));
    std::mt19937 rng(5);
    std::normal_distribution<float> n01;
    std::uniform_int_distribution<int> expo(-30, 30), tiny(-68, -62);
    auto draw = [&](int k) {
        float x = n01(rng);
        if (k == 1) {
            uint32_t u;
            memcpy(&u, &x, 4);
            u &= 0xffff0000u;
            memcpy(&x, &u, 4);
        }
        return k == 2 ? ldexpf(x, expo(rng)) : k == 3 ? ldexpf(x, tiny(rng)) : x;
    };
    long total = 0;
    for (int k = 0; k < 4; ++k) {
        for (float &x : a) x = draw(k);
        for (float &x : b) x = draw(k);
        CK(hipMemcpy(da, a.data(), a.size() * 4, hipMemcpyHostToDevice));
        CK(hipMemcpy(db, b.data(), b.size() * 4, hipMemcpyHostToDevice));
        chain_kernel<<<kTiles / 4, 256>>>(da, db, dout);
        CK(hipGetLastError());
        CK(hipMemcpy(out.data(), dout, out.size() * 4, hipMemcpyDeviceToHost));
        long bad = 0, sub = 0;
        for (int t = 0; t < kTiles; ++t)
            for (int m = 0; m < 32; ++m)
                for (int n = 0; n < 32; ++n) {
                    float want = 0.0f;
                    for (int i = 0; i < 8; ++i) want = fmaf(a[t * 256 + m * 8 + i], b[t * 256 + i * 32 + n], want);
                    bad += memcmp(&want, &out[t * 1024 + m * 32 + n], 4) != 0;
                    sub += want != 0.0f && fabsf(want) < 1.17549435e-38f;
                }
        printf("%s: %ld of %d results differ (%ld subnormal)\n", kind[k], bad, kTiles * 1024, sub);
        total += bad;
    }
    CK(hipFree(da)); CK(hipFree(db)); CK(hipFree(dout));
    return total != 0;
}
