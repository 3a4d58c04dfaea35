// One lane of the causal depthwise conv1d over time (conv1d.hip, and the way into a block in linear.hip): VEC adjacent channels of a
// token row, their taps, and the K - 1 rows before the next one.
#pragma once

#include "device_math.h"

namespace mamba {
namespace {

template <typename T, int VEC> struct RowVec;
template <> struct RowVec<float, 4> { typedef float4 type; };
template <> struct RowVec<float, 1> { typedef float type; };
template <> struct RowVec<bf16_t, 8> { typedef uint4 type; };
template <> struct RowVec<bf16_t, 1> { typedef uint16_t type; };

__device__ __forceinline__ void unpack_row(float4 r, float *v) { v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w; }
__device__ __forceinline__ void unpack_row(float r, float *v) { v[0] = r; }
__device__ __forceinline__ void unpack_row(uint16_t r, float *v) { v[0] = bf16_to_f32(r); }
__device__ __forceinline__ void unpack_row(uint4 r, float *v)
{
    v[0] = bf16_lo(r.x); v[1] = bf16_hi(r.x); v[2] = bf16_lo(r.y); v[3] = bf16_hi(r.y);
    v[4] = bf16_lo(r.z); v[5] = bf16_hi(r.z); v[6] = bf16_lo(r.w); v[7] = bf16_hi(r.w);
}
__device__ __forceinline__ void pack_row(const float *v, float4 &r) { r = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void pack_row(const float *v, float &r) { r = v[0]; }
__device__ __forceinline__ void pack_row(const float *v, uint16_t &r) { r = (uint16_t)f32_to_bf16(v[0]); }
__device__ __forceinline__ void pack_row(const float *v, uint4 &r)
{
    r = make_uint4(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]),
                   f32x2_to_bf16x2(v[4], v[5]), f32x2_to_bf16x2(v[6], v[7]));
}

// COUNT contiguous elements, COUNT * sizeof(T) a multiple of 16 bytes and p 16-byte aligned:
// moved as 16-byte vectors (the per-lane blocks of weights and of carried state are such blocks).
template <int COUNT> __device__ __forceinline__ void ld_block(const float *p, float *f)
{
    const float4 *q = reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int v = 0; v < COUNT / 4; ++v) unpack_row(q[v], f + 4 * v);
}
template <int COUNT> __device__ __forceinline__ void ld_block(const bf16_t *p, float *f)
{
    const uint4 *q = reinterpret_cast<const uint4 *>(p);
#pragma unroll
    for (int v = 0; v < COUNT / 8; ++v) unpack_row(q[v], f + 8 * v);
}
template <int COUNT> __device__ __forceinline__ void st_block(float *p, const float *f)
{
    float4 *q = reinterpret_cast<float4 *>(p);
#pragma unroll
    for (int v = 0; v < COUNT / 4; ++v) pack_row(f + 4 * v, q[v]);
}
template <int COUNT> __device__ __forceinline__ void st_block(bf16_t *p, const float *f)
{
    uint4 *q = reinterpret_cast<uint4 *>(p);
#pragma unroll
    for (int v = 0; v < COUNT / 8; ++v) pack_row(f + 8 * v, q[v]);
}

// What a lane keeps while it walks the tokens of its VEC adjacent channels: taps, bias and the K - 1 rows before the next one.
template <typename T, int VEC, int K, bool SILU> struct ConvLane {
    typedef typename RowVec<T, VEC>::type row_t;
    static constexpr int H = K - 1;
    float wr[VEC][K], br[VEC];
    float win[H > 0 ? H : 1][VEC];                                  // win[H - 1] is the newest
    float carried[VEC * (H > 0 ? H : 1)];

    // rows before token 0 come from the carried state, whose (VEC, H) block of this lane is one contiguous run
    __device__ __forceinline__ void load_carried(const T *state_in, const int32_t *parent, int64_t b, int64_t n_in, int64_t D, int64_t d0)
    {
        // a draft branch continues from its parent's window (the copy is fused into this load)
        const int64_t pb = parent ? (int64_t)parent[b] : b;
        const bool p_ok = !parent || (pb >= 0 && pb < n_in);
        if (!state_in) {
#pragma unroll
            for (int i = 0; i < VEC * H; ++i) carried[i] = 0.0f;
        } else if (!p_ok) {
#pragma unroll
            for (int i = 0; i < VEC * H; ++i) carried[i] = __int_as_float(0x7fc00000);
        } else if constexpr (VEC > 1) {
            ld_block<VEC * H>(state_in + (pb * D + d0) * H, carried);
        } else {
#pragma unroll
            for (int k = 0; k < H; ++k) carried[k] = ld_io(state_in, (pb * D + d0) * H + k);
        }
    }
    // window row i is token t: its row, or for a negative t the carried one
    __device__ __forceinline__ void set_window(int i, int64_t t, row_t row)
    {
        if (t >= 0) {
            unpack_row(row, win[i]);
        } else {
#pragma unroll
            for (int c = 0; c < VEC; ++c) {
                float v = 0.0f;
#pragma unroll
                for (int k = 0; k < H; ++k)
                    if (k == H + t) v = carried[c * H + k];
                win[i][c] = v;
            }
        }
    }
    __device__ __forceinline__ row_t emit(row_t raw)
    {
        float cur[VEC], o[VEC];
        unpack_row(raw, cur);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            float acc = br[c];
#pragma unroll
            for (int k = 0; k < H; ++k) acc = fmaf(wr[c][k], win[k][c], acc);
            acc = fmaf(wr[c][K - 1], cur[c], acc);
            o[c] = SILU ? silu_f32(acc) : acc;
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
#pragma unroll
            for (int k = 0; k + 1 < H; ++k) win[k][c] = win[k + 1][c];
            if (H > 0) win[H - 1][c] = cur[c];
        }
        row_t packed;
        pack_row(o, packed);
        return packed;
    }
    __device__ __forceinline__ void store_window(T *state_out, int64_t b, int64_t D, int64_t d0) const
    {
        float last[VEC * (H > 0 ? H : 1)];
#pragma unroll
        for (int c = 0; c < VEC; ++c)
#pragma unroll
            for (int k = 0; k < H; ++k) last[c * H + k] = win[k][c];
        if constexpr (VEC > 1) {
            st_block<VEC * H>(state_out + (b * D + d0) * H, last);
        } else {
#pragma unroll
            for (int k = 0; k < H; ++k) st_io(state_out, (b * D + d0) * H + k, last[k]);
        }
    }
};

}  // namespace
}  // namespace mamba
