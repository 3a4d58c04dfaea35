// RMSNorm in front of the block's input projection (the Mamba-130M drafter of the paper, Sec. 3.1,
// normalizes the residual stream before every mixer):  y[m, :] = x[m, :] * rsqrt(mean(x[m, :]^2) + eps) * w
// One wavefront per token row, the row and its weights kept in registers between the reduction and the scaling so that
// everything is read once and in one trip to memory.  A lane takes four adjacent features at a time: its weights are then
// 16 bytes next to its neighbour's 16.  (With eight features, 16 bytes of the row, the weights come in 16-byte pieces 32
// bytes apart, and the address path takes a cycle per lane for those, three times what the row itself takes.)  Launches one
// after the other: 8000 x 768 7.2 -> 6.2 us, 333 x 768 3.6 -> 3.4 us.  The kernel is instantiated for the row's own length:
// registers for a longer one keep wavefronts off the CU (8000 x 2560 with room for 4096 features 17.3 us, its own 15.6,
// 2000 x 2560 5.97 and 5.71; 8000 x 1280 with room for 2048 9.4 and 8.7).
#include "device_math.h"
#include "launch.h"

namespace mamba {
namespace {

constexpr int kWave = 64;
constexpr int kRowsPerBlock = 4;

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// C % 4 == 0 and C <= 64 * 4 * NV
template <int NV>
__global__ void __launch_bounds__(kWave * kRowsPerBlock)
rmsnorm_kernel(const bf16_t *__restrict__ x, const float *__restrict__ w, bf16_t *__restrict__ y, int64_t M, int C, float eps)
{
    const int lane = threadIdx.x & 63;
    const int64_t m = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    if (m >= M) return;                                  // whole wavefronts leave together
    const int vecs = C / 4;
    const uint2 *xr = reinterpret_cast<const uint2 *>(x + m * C);
    uint2 raw[NV];
    float4 wv[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = lane + i * kWave;
        raw[i] = v < vecs ? xr[v] : make_uint2(0, 0);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = lane + i * kWave;
        wv[i] = reinterpret_cast<const float4 *>(w)[v < vecs ? v : 0];
    }
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const float v0 = bf16_lo(raw[i].x), v1 = bf16_hi(raw[i].x), v2 = bf16_lo(raw[i].y), v3 = bf16_hi(raw[i].y);
        ss = fmaf(v0, v0, ss);
        ss = fmaf(v1, v1, ss);
        ss = fmaf(v2, v2, ss);
        ss = fmaf(v3, v3, ss);
    }
    ss = wave_sum(ss);
    const float scale = __builtin_amdgcn_rsqf(ss / (float)C + eps);
    uint2 *yr = reinterpret_cast<uint2 *>(y + m * C);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = lane + i * kWave;
        if (v >= vecs) continue;
        yr[v] = make_uint2(f32x2_to_bf16x2(bf16_lo(raw[i].x) * scale * wv[i].x, bf16_hi(raw[i].x) * scale * wv[i].y),
                           f32x2_to_bf16x2(bf16_lo(raw[i].y) * scale * wv[i].z, bf16_hi(raw[i].y) * scale * wv[i].w));
    }
}

// the instantiation that holds just the row: NV = ceil(C / 256), 1 to 16
template <int NV> void launch_norm(const NormArgs &a, unsigned blocks, hipStream_t stream)
{
    if constexpr (NV < 16) {
        if (a.C > 4 * kWave * NV) return launch_norm<NV + 1>(a, blocks, stream);
    }
    rmsnorm_kernel<NV><<<blocks, kWave * kRowsPerBlock, 0, stream>>>(static_cast<const bf16_t *>(a.x), a.w, static_cast<bf16_t *>(a.y),
                                                                     a.M, (int)a.C, a.eps);
}

}  // namespace

hipError_t launch_rmsnorm(const NormArgs &a, hipStream_t stream)
{
    const unsigned blocks = (unsigned)((a.M + kRowsPerBlock - 1) / kRowsPerBlock);
    launch_norm<1>(a, blocks, stream);                           // C <= 4096
    return hipGetLastError();
}

}  // namespace mamba
