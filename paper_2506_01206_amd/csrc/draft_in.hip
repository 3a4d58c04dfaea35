// The way into a Mamba block at a draft position (Sec. 4.1: a few rows, one per live branch): RMSNorm, in_proj, the conv step and
// the partial sums of the x projection in one launch, gfx950.
//
//   u = x * norm_w (bf16);  [xv | z] = rsqrt(mean x^2 + eps) (u w^T);  x_c = silu(conv step(xv));  part = x_c W_x^T per 16 columns
//
// Nothing is big here, w is read once, and what counts is the chain between the launch and the last store: one trip to memory,
// the instructions of a wavefront, two barriers.  One workgroup per 16 output columns (192 of them at 1536 channels) and 16 MT
// rows; its NW wavefronts share k in steps of 64, G steps of a wavefront requested at once.  A row's 128 bytes of a step lie on
// eight lanes, so that a load covers whole lines: the address path takes about 17 cycles for such a KiB, 34 with a row's 64 bytes
// on a quad (48 loads a workgroup, all through one path) and 60 where every lane is on a row of its own, as a fragment of
// v_mfma_f32_16x16x32_bf16 wants them; patches of LDS private to the wavefront turn lines into fragments.  All requests that do
// not depend on another go out first, the carried conv windows as soon as the parent index is there; only then the first
// product.  Offsets of a lane are 32 bits from scalar bases.
// Cycles from the first instruction of a workgroup, 12 rows of a 1536-channel block, this kernel (the one before it: k steps of 32,
// the windows and the parents they need waited for ahead of the first product, x projection stored one value at a time):
// requests out 2300 (4100), products done 4150 (5450), sums met 4900 (5850), columns done 5500 (6900), end 6000 (7900).
// us a launch in a replayed graph, 24 blocks in turn, 1 / 12 / 48 rows: 768 wide 3.7 / 3.9 / 7.5 (4.3 / 4.8 / 8.8), 2048 wide
// 10.0 / 11.3 / 23.9 (10.5 / 13.4 / 30.4), 4096 wide 31.9 / 34.7 / 80.9 (33.3 / 40.3 / 95.4).
#include "device_math.h"
#include "launch.h"
#include "routes.h"

namespace mamba {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short bf16x4_bits __attribute__((ext_vector_type(4)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// barrier that orders LDS traffic only: global loads in flight stay in flight
__device__ __forceinline__ void lds_barrier_d()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
template <int CTRL> __device__ __forceinline__ float add_lanes(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// EVEN: K = 64 NW G, one trip of every wavefront; otherwise any K that is a multiple of 8.  CK: taps of the conv, 2 to 4.
// grid: (2 D / 16 rounded up, ceil(M / (16 MT)))
template <int MT, int NW, int G, bool EVEN, int CK>
__global__ void __launch_bounds__(64 * NW)
draft_in_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w, const int32_t *__restrict__ parent,
                const float *__restrict__ norm_w, int M, int D, int K, int xn, const bf16_t *__restrict__ xp_w,
                const float *__restrict__ conv_w, const bf16_t *conv_src, const float *__restrict__ conv_b, bf16_t *conv_dst,
                bf16_t *__restrict__ xc_out, bf16_t *__restrict__ z_out, float *__restrict__ xp_part, int64_t n_in, float inv_k, float eps)
{
    constexpr int kThr = 64 * NW, H = CK - 1;
    static_assert(16 * G <= 64, "a lane fetches one piece of the norm weights");
    constexpr int kStep = (1 + MT) * 2048;                         // fragments of one step: w, then MT row tiles
    constexpr int PB = G * NW * kStep <= 48 * 1024 ? G : 1;     // patches in turn: several workgroups to a CU
    constexpr int OPT = (MT * 256 + kThr - 1) / kThr;              // outputs per thread
    constexpr int kXcRow = 24;                                     // elements between rows of the finished columns (48 bytes: 8-byte aligned, spread over the banks)
    constexpr int XT = MT == 1 && NW >= 5 ? 1 : 2;                 // x projection tiles of a wavefront whose weights are fetched ahead
    // a wavefront's patches, and its partial tiles once it is done with those
    constexpr int kWave = PB * kStep > MT * 1024 ? PB * kStep : MT * 1024;
    __shared__ __attribute__((aligned(16))) unsigned char patch[NW][kWave];
    __shared__ __attribute__((aligned(16))) float4 norm_lds[NW][16 * G];
    __shared__ __attribute__((aligned(16))) float ssq[MT * 16][NW];
    __shared__ __attribute__((aligned(16))) uint16_t xc[MT * 16 * kXcRow];
    const unsigned tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * (16 * MT), N = 2 * D;
    const unsigned li = lane & 15, lg = lane >> 4;                 // fragment view: row, 16-byte chunk of a k32 half
    const unsigned lrow = lane >> 3, lch = lane & 7;               // load view: row (+ 8 t), 16-byte chunk of the step
    const bool xp_on = xp_w && n0 < D;                             // uniform: D % 16 == 0 with an x projection

    __builtin_amdgcn_sched_barrier(0);
    // ---- outputs of this thread: tile o / 256, accumulator (o / 64) % 4 of lane o % 64
    const int on = n0 + (int)li;
    int om[OPT];
    int32_t par[OPT];
#pragma unroll
    for (int j = 0; j < OPT; ++j) {
        const int o6 = wave + j * NW;
        om[j] = m0 + (o6 >> 2) * 16 + (o6 & 3) + 4 * (int)lg;
        par[j] = (parent ? parent : reinterpret_cast<const int32_t *>(norm_w))[parent ? (unsigned)min(om[j], M - 1) : 0u];
    }

    __builtin_amdgcn_sched_barrier(0);                             // the parents are asked for first

    // ---- the wavefront's share of k: steps [s_first, s_end)
    const int steps = EVEN ? NW * G : (K + 63) >> 6, per = EVEN ? G : (steps + NW - 1) / NW;
    const int s_first = wave * per, s_end = EVEN || s_first + per < steps ? s_first + per : steps;
    const unsigned kchunks = (unsigned)K >> 3;                     // K % 8 == 0
    const char *wb = reinterpret_cast<const char *>(w + (int64_t)n0 * K), *xb = reinterpret_cast<const char *>(x + (int64_t)m0 * K);
    unsigned wo[2], xo[2 * MT];
#pragma unroll
    for (unsigned t = 0; t < 2; ++t) wo[t] = min(8 * t + lrow, (unsigned)(N - 1 - n0)) * (2u * (unsigned)K) + 16 * lch;
#pragma unroll
    for (unsigned t = 0; t < 2 * MT; ++t) xo[t] = min(8 * t + lrow, (unsigned)(M - 1 - m0)) * (2u * (unsigned)K) + 16 * lch;   // rows past M repeat the last one, never stored
    const unsigned put = (lrow * 8 + (lch ^ lrow)) * 16;           // + 1024 t: chunks xor-swizzled by the row, no bank conflicts either way
    const unsigned get0 = (li * 8 + (lg ^ (li & 7))) * 16, get1 = (li * 8 + ((lg + 4) ^ (li & 7))) * 16;

    f32x4v acc[MT];
    float ss[2 * MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = f32x4v(0.0f);
#pragma unroll
    for (int t = 0; t < 2 * MT; ++t) ss[t] = 0.0f;
    float cb = 0.0f, taps[CK];
    uint32_t win01[OPT];                                           // carried inputs as they come: two in one word, the last or only one
    uint16_t win2[OPT];
    uint2 xw[XT];
    const int xp_tiles = (xn + 15) >> 4;
    bool first = true;
    for (int s0 = s_first; EVEN ? first : s0 < s_end || first; s0 += G) {
        u32x4 wf[G][2], xf[G][2 * MT];
        // norm weights of the 64 G values of k: a 16-byte piece per lane, handed out by LDS
        const unsigned nf = 16u * (unsigned)s0 + lane;
        const float4 nw = reinterpret_cast<const float4 *>(norm_w)[lane < 16u * G && (EVEN || nf < 2 * kchunks) ? nf : 0u];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int s = EVEN || s0 + g < s_end ? s0 + g : 0;
            const unsigned back = EVEN || 8u * (unsigned)s + lch < kchunks ? 0u : 16 * lch;   // chunks past K re-read the step's first one
            const char *ws = wb + (int64_t)s * 128, *xs = xb + (int64_t)s * 128;
#pragma unroll
            for (int t = 0; t < 2; ++t) wf[g][t] = *reinterpret_cast<const u32x4 *>(ws + (EVEN ? wo[t] : wo[t] - back));
#pragma unroll
            for (int t = 0; t < 2 * MT; ++t) xf[g][t] = *reinterpret_cast<const u32x4 *>(xs + (EVEN ? xo[t] : xo[t] - back));
        }
        __builtin_amdgcn_sched_barrier(0);                         // (nothing waits for the parents before these are out)
        if (first) {
            // (unconditional, also in a workgroup that has no use for them: the number of requests in flight stays known) taps
            // and bias, this wavefront's fragments of the x projection, then the windows behind the parent index
            const unsigned col = (unsigned)(on < D ? on : D - 1);
            cb = (conv_b ? conv_b : conv_w)[col];
            __builtin_memcpy(taps, conv_w + col * (unsigned)CK, sizeof(taps));
#pragma unroll
            for (int r = 0; r < XT; ++r) {
                const int jt = MT == 1 ? r * NW + wave : (r * NW + wave) / MT;
                const unsigned row = min((unsigned)jt * 16u + li, (unsigned)(xn - 1));
                xw[r] = *reinterpret_cast<const uint2 *>(xp_on ? xp_w + (int64_t)row * D + n0 + 4 * lg : w);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < OPT; ++j) {
                const int32_t p = parent ? par[j] : om[j];
                const char *src = reinterpret_cast<const char *>(conv_src + ((int64_t)(p >= 0 && p < n_in ? p : 0) * D + col) * H);
                if constexpr (H >= 2) __builtin_memcpy(&win01[j], src, 4);
                if constexpr (H != 2) __builtin_memcpy(&win2[j], src + (H == 3 ? 4 : 0), 2);
            }
        }
        first = false;
        __builtin_amdgcn_sched_barrier(0);                         // all of it in flight before any of it is used
        if (lane < 16u * G) norm_lds[wave][lane] = nw;
        wave_sync();
        auto fill = [&](int g) __attribute__((always_inline)) {
            unsigned char *p = patch[wave] + g % PB * kStep;
            const bool ok = EVEN || (s0 + g < s_end && 8u * (unsigned)(s0 + g) + lch < kchunks);   // else zeros: adds nothing
#pragma unroll
            for (int t = 0; t < 2; ++t) *reinterpret_cast<u32x4 *>(p + 1024 * t + put) = ok ? wf[g][t] : u32x4(0u);
            const float4 g0 = norm_lds[wave][16 * g + 2 * lch], g1 = norm_lds[wave][16 * g + 2 * lch + 1];
#pragma unroll
            for (int t = 0; t < 2 * MT; ++t) {
                const u32x4 q = ok ? xf[g][t] : u32x4(0u);
                const float v0 = bf16_lo(q.x), v1 = bf16_hi(q.x), v2 = bf16_lo(q.y), v3 = bf16_hi(q.y);
                const float v4 = bf16_lo(q.z), v5 = bf16_hi(q.z), v6 = bf16_lo(q.w), v7 = bf16_hi(q.w);
                ss[t] += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3 + v4 * v4 + v5 * v5 + v6 * v6 + v7 * v7;
                u32x4 r;
                r.x = f32x2_to_bf16x2(v0 * g0.x, v1 * g0.y);
                r.y = f32x2_to_bf16x2(v2 * g0.z, v3 * g0.w);
                r.z = f32x2_to_bf16x2(v4 * g1.x, v5 * g1.y);
                r.w = f32x2_to_bf16x2(v6 * g1.z, v7 * g1.w);
                *reinterpret_cast<u32x4 *>(p + 2048 + 1024 * t + put) = r;
            }
        };
        auto product = [&](int g) __attribute__((always_inline)) {
            const unsigned char *p = patch[wave] + g % PB * kStep;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned get = h ? get1 : get0;
                const bf16x8 wv = *reinterpret_cast<const bf16x8 *>(p + get);
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(p + 2048 * (1 + t) + get), wv, acc[t], 0, 0, 0);
            }
        };
#pragma unroll
        for (int g = 0; g < G; ++g) {
            fill(g);
            wave_sync();
            if (PB == G) continue;
            product(g);
            wave_sync();
        }
        if constexpr (PB == G) {
#pragma unroll
            for (int g = 0; g < G; ++g) product(g);
            wave_sync();
        }
    }
    // acc[t][i] is C[m = 16 t + 4 (lane / 16) + i][n = lane % 16]
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) reinterpret_cast<float *>(patch[wave])[(4 * t + i) * 64 + lane] = acc[t][i];
#pragma unroll
    for (int t = 0; t < 2 * MT; ++t) {
        // the sum over the eight lanes of a row: quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror
        const float v = add_lanes<0x141>(add_lanes<0x4e>(add_lanes<0xb1>(ss[t])));
        if (lch == 0) ssq[8 * t + lrow][wave] = v;
    }
    lds_barrier_d();

#pragma unroll
    for (int j = 0; j < OPT; ++j) {
        const int o = tid + j * kThr, t = (o >> 8) < MT ? o >> 8 : 0, i = (o >> 6) & 3;
        float v = 0.0f, sq = 0.0f;
#pragma unroll
        for (int q = 0; q < NW; ++q) v += reinterpret_cast<const float *>(patch[q])[(4 * t + i) * 64 + lane];
#pragma unroll
        for (int q = 0; q < NW; ++q) sq += ssq[16 * t + 4 * lg + i][q];
        v *= __builtin_amdgcn_rsqf(fmaf(sq, inv_k, eps));
        if (o >= MT * 256 || om[j] >= M || on >= N) continue;
        uint32_t stored = f32_to_bf16(v);
        if (on < D) {
            // the window of this (row, channel): CK - 1 carried values, then v as stored; same order of operations as the
            // stand-alone conv kernel.  A bad parent index leaves NaN in the carried places.
            const int32_t p = parent ? par[j] : om[j];
            const bool p_ok = p >= 0 && p < n_in;
            const int64_t off = (int64_t)om[j] * D + on;
            const uint32_t nan2 = 0x7fc07fc0u, w01 = H >= 2 ? p_ok ? win01[j] : nan2 : 0, w2 = H != 2 ? p_ok ? win2[j] : nan2 & 0xffffu : 0;
            float a = conv_b ? cb : 0.0f;
            if constexpr (H == 1) a = fmaf(taps[0], bf16_to_f32(w2), a);
            if constexpr (H >= 2) a = fmaf(taps[1], bf16_hi(w01), fmaf(taps[0], bf16_lo(w01), a));
            if constexpr (H == 3) a = fmaf(taps[2], bf16_to_f32(w2), a);
            a = fmaf(taps[H], bf16_to_f32(stored), a);
            bf16_t *nwin = conv_dst + off * H;
            if constexpr (H == 3) {
                const uint32_t moved = w01 >> 16 | w2 << 16;
                __builtin_memcpy(nwin, &moved, 4);
            }
            if constexpr (H == 2) nwin[0] = (bf16_t)(w01 >> 16);
            nwin[H - 1] = (bf16_t)stored;
            stored = f32_to_bf16(silu_f32(a));
            xc_out[off] = (bf16_t)stored;
            xc[(om[j] - m0) * kXcRow + li] = (uint16_t)stored;
        } else {
            z_out[(int64_t)om[j] * D + on - D] = (bf16_t)stored;
        }
    }
    if (!xp_on) return;
    // x projection of the 16 finished columns (as stored), formed transposed: a lane's four sums are adjacent outputs of one row
    // (rows past M hold whatever was in LDS: they only reach outputs that are not stored)
    lds_barrier_d();
    const int tasks = xp_tiles * MT;
    for (int r = 0; r * NW + wave < tasks; ++r) {
        const int task = r * NW + wave, jt = MT == 1 ? task : task / MT, t = MT == 1 ? 0 : task % MT;
        uint2 a2 = xw[0];
        if (XT > 1 && r == 1) a2 = xw[XT - 1];
        if (r >= XT) a2 = *reinterpret_cast<const uint2 *>(xp_w + (int64_t)min(jt * 16 + (int)li, xn - 1) * D + n0 + 4 * lg);
        const uint2 b2 = *reinterpret_cast<const uint2 *>(&xc[(16 * t + li) * kXcRow + 4 * lg]);
        const f32x4v y = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4_bits, a2), __builtin_bit_cast(bf16x4_bits, b2),
                                                                   f32x4v(0.0f), 0, 0, 0);
        // y[i] is output 16 jt + 4 lg + i of row 16 t + li
        const int m = m0 + 16 * t + (int)li, jn = jt * 16 + 4 * (int)lg;
        if (m < M && jn < xn) *reinterpret_cast<f32x4v *>(xp_part + ((int64_t)m * (D >> 4) + blockIdx.x) * xn + jn) = y;
    }
}

template <int MT, int NW, int G, bool EVEN> hipError_t launch_k(const LinearArgs &a, hipStream_t stream)
{
    const int64_t D = a.width[0], N = 2 * D;
    const dim3 grid((unsigned)((N + 15) / 16), (unsigned)((a.M + 16 * MT - 1) / (16 * MT)));
#define MAMBA_DRAFT_IN(CK)                                                                                                        \
    draft_in_kernel<MT, NW, G, EVEN, CK><<<grid, 64 * NW, 0, stream>>>(                                                           \
        static_cast<const bf16_t *>(a.x), static_cast<const bf16_t *>(a.w), a.conv_parent, a.norm_w, (int)a.M, (int)D, (int)a.K,  \
        a.xproj_n, static_cast<const bf16_t *>(a.xproj_w), a.conv_w, static_cast<const bf16_t *>(a.conv_src), a.conv_b,           \
        static_cast<bf16_t *>(a.conv_dst), static_cast<bf16_t *>(a.out[0]), static_cast<bf16_t *>(a.out[1]), a.xproj_part,        \
        a.conv_n_in, 1.0f / (float)a.K, a.eps)
    if constexpr (EVEN) {
        MAMBA_DRAFT_IN(4);
    } else {
        switch (a.conv_k) {
        case 2: MAMBA_DRAFT_IN(2); break;
        case 3: MAMBA_DRAFT_IN(3); break;
        case 4: MAMBA_DRAFT_IN(4); break;
        default: return hipErrorInvalidValue;
        }
    }
#undef MAMBA_DRAFT_IN
    return hipGetLastError();
}

template <int MT> hipError_t launch_m(const LinearArgs &a, hipStream_t stream)
{
    // One trip of every wavefront where k allows: four wavefronts for 16 rows (their sums meet sooner), more where a wavefront
    // has more row tiles to fill.  us of a whole block (in_proj, state step, out_proj) with 12 / 24 / 48 rows on (wavefronts, steps):
    //   K =  512  (4, 2) 10.57 / 11.30 / 13.21   (8, 1) 10.93 / 11.64 / 12.89
    //   K =  768  (4, 3) 11.91 / 14.53 / 19.54   (6, 2) 12.25 / 14.22 / 19.13
    //   K = 1024  (4, 4) 15.91 / 19.43 / 26.40   (8, 2) 16.31 / 18.40 / 23.90
    if (a.conv_k == 4) {
        if (a.K == 256) return launch_k<MT, 4, 1, true>(a, stream);
        if (a.K == 512) return launch_k<MT, MT < 4 ? 4 : 8, MT < 4 ? 2 : 1, true>(a, stream);
        if (a.K == 768) return launch_k<MT, MT < 2 ? 4 : 6, MT < 2 ? 3 : 2, true>(a, stream);
        if (a.K == 1024) return launch_k<MT, MT < 2 ? 4 : 8, MT < 2 ? 4 : 2, true>(a, stream);
        if (a.K == 1536) return launch_k<MT, 8, 3, true>(a, stream);
        if constexpr (MT < 4)
            if (a.K == 2048) return launch_k<MT, 8, 4, true>(a, stream);
    }
    // any other k: as many steps at once as leave the fewest empty ones in the last trip
    const int64_t per = (a.K + 511) / 512;
    if (per <= 2 || per == 4) return launch_k<MT, 8, 2, false>(a, stream);
    return launch_k<MT, 8, 3, false>(a, stream);
}

}  // namespace

hipError_t launch_draft_in(const LinearArgs &a, hipStream_t stream)
{
    const int64_t N = a.width[0] + a.width[1];
    // norm and conv come together, the x projection only with them
    if (!linear_few_fits(N, a.K) || a.width[0] != a.width[1] || a.width[2] != 0 || a.bias || a.residual || a.M > 64 || !a.conv_w || !a.conv_src ||
        !a.conv_dst || a.conv_k < 2 || a.K % 8 || (a.xproj_w && (!a.xproj_part || a.width[0] % 16 || a.xproj_n % 4)))
        return hipErrorInvalidValue;
    switch (linear_few_row_tiles(a.M, N)) {
    case 1: return launch_m<1>(a, stream);
    case 2: return launch_m<2>(a, stream);
    default: return launch_m<4>(a, stream);
    }
}

}  // namespace mamba
