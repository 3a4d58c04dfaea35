// One selective-state update for every live branch of a draft tree (Sec. 4.1 of the paper:
// tree drafting is batch generation, and a child continues from its parent's state), gfx950.
//
//   p = parent[j];  h_out[j] = exp(delta_j A) h_in[p] + delta_j B_j x_j
//   out[j] = (C_j . h_out[j] + D x_j) silu(z_j)
//
// The step moves 2 * D * N * 4 bytes of state per branch for D * N state updates: it is bound
// by HBM.  The state row of a branch is walked as float4s, one per lane, consecutive lanes on
// consecutive float4s, so every wavefront load and store is one contiguous 1 KiB run.  A lane
// therefore owns 4 of the N states of a channel; the N/4 lanes of a channel sum their partial
// C.h with DPP lane exchanges inside a quad (and a half-row mirror for N = 32).  With a parent
// index the gather is fused into the load of h_in, which makes a separate state copy unnecessary.
#include "device_math.h"
#include "launch.h"
#include "routes.h"

namespace mamba {
namespace {

constexpr int kBlock = 256;

// barrier that orders LDS only: requests in flight stay in flight
__device__ __forceinline__ void lds_barrier_s()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false);
    return v + __int_as_float(o);
}

// sum over the Q = N/4 adjacent lanes that share a channel; every one of them gets the total
template <int Q> __device__ __forceinline__ float channel_sum(float v)
{
    if constexpr (Q >= 2) v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
    if constexpr (Q >= 4) v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    if constexpr (Q >= 8) v = dpp_add<0x141>(v);  // row_half_mirror: lane i <-> 7 - i of each 8
    return v;
}

template <int N> __device__ __forceinline__ float4 ld4_io(const float *p) { return *reinterpret_cast<const float4 *>(p); }
template <int N> __device__ __forceinline__ float4 ld4_io(const bf16_t *p)
{
    const uint2 r = *reinterpret_cast<const uint2 *>(p);
    return make_float4(bf16_lo(r.x), bf16_hi(r.x), bf16_lo(r.y), bf16_hi(r.y));
}

// The state is read once and written once per step: streaming (non-temporal) accesses keep it from displacing the
// weights and token rows in the caches (measured cold in a replayed graph: 64 branches x 4096 channels 9.9 -> 9.2 us,
// 32 x 1536 3.5 -> 2.9 us).
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_stream(const float4 *p)
{
    const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st_stream(float4 *p, float4 v)
{
    f32x4 t;
    t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
    __builtin_nontemporal_store(t, reinterpret_cast<f32x4 *>(p));
}

constexpr int kStepUnroll = 4;

// grid: (ceil(D * N / 4 / (256 * U)), n_out).  A lane owns U float4s of the branch's (D, N) state,
// 256 float4s apart, so every wavefront load or store is still one contiguous 1 KiB run; all
// loads of the U pieces are issued before the first one is used, which keeps several KiB per
// wavefront in flight (the step is a single pass over the state and lives on memory latency).
// (Arguments fetched by the kernel, not brought in registers: 1 x 768 2.03 -> 1.95 us, 4 x 1536 2.44 -> 2.39, 12 x 1536 2.60 -> 2.55; the
// kernel below is faster the other way, 64 x 4096 8.02 -> 7.90, 128 x 4096 15.49 -> 15.27.)
template <typename T, int N, int U, bool HAS_Z, bool SOFTPLUS>
__global__ void __launch_bounds__(kBlock)
state_step_kernel(StepStates states, const int32_t *__restrict__ parent,
                  const T *__restrict__ x, const T *__restrict__ dt, const float *__restrict__ A,
                  const T *__restrict__ Bm, const T *__restrict__ Cm,
                  const float *__restrict__ Dskip, const T *__restrict__ z,
                  const float *__restrict__ dt_bias, T *__restrict__ out, int64_t n_in, int64_t D,
                  const bf16_t *__restrict__ dt_w, int64_t dt_rank)
{
    constexpr int Q = N / 4;
    const int64_t j = blockIdx.y;
    const int64_t row4 = D * Q;  // float4s per branch
    const float4 *a4 = reinterpret_cast<const float4 *>(A);

    int64_t f[U], d[U];
    bool live[U];
    float4 h[U], a[U], bv[U], cv[U];
    float xv[U], dv[U], zv[U], bias[U], dsk[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int64_t f_raw = ((int64_t)blockIdx.x * U + i) * kBlock + threadIdx.x;
        live[i] = f_raw < row4;
        f[i] = live[i] ? f_raw : row4 - 1;
        d[i] = f[i] / Q;
        const int q = (int)(f[i] - d[i] * Q);
        a[i] = a4[f[i]];
        bv[i] = ld4_io<N>(Bm + j * N + 4 * q);
        cv[i] = ld4_io<N>(Cm + j * N + 4 * q);
        xv[i] = ld_io(x, j * D + d[i]);
        if (sizeof(T) == 2 && dt_w) {
            // dt projection fused in: the Q lanes of a channel share the dt_rank products (4 at a time)
            const uint2 *wrow = reinterpret_cast<const uint2 *>(dt_w + d[i] * dt_rank);
            const uint2 *lrow = reinterpret_cast<const uint2 *>(reinterpret_cast<const bf16_t *>(dt) + j * dt_rank);
            float acc = 0.0f;
#pragma unroll 4
            for (int64_t c = q; c < dt_rank / 4; c += Q) {
                const uint2 a2 = wrow[c], b2 = lrow[c];
                acc = fmaf(bf16_lo(a2.x), bf16_lo(b2.x), acc);
                acc = fmaf(bf16_hi(a2.x), bf16_hi(b2.x), acc);
                acc = fmaf(bf16_lo(a2.y), bf16_lo(b2.y), acc);
                acc = fmaf(bf16_hi(a2.y), bf16_hi(b2.y), acc);
            }
            dv[i] = bf16_to_f32(f32_to_bf16(channel_sum<Q>(acc)));     // rounded like the stored tensor it replaces
        } else {
            dv[i] = ld_io(dt, j * D + d[i]);
        }
        zv[i] = HAS_Z ? ld_io(z, j * D + d[i]) : 0.0f;
        bias[i] = dt_bias ? dt_bias[d[i]] : 0.0f;
        dsk[i] = Dskip ? Dskip[d[i]] : 0.0f;
    }
    // the state row is the only load that has to wait for the parent index
    const int64_t p = parent ? (int64_t)parent[j] : j;
    const bool p_ok = p >= 0 && p < n_in;
    const float4 *hin4 = reinterpret_cast<const float4 *>(states.in) + (p_ok ? p : 0) * row4;
#pragma unroll
    for (int i = 0; i < U; ++i) h[i] = ld_stream(hin4 + f[i]);
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const float v = dv[i] + bias[i];
        const float delta = SOFTPLUS ? softplus_f32(v) : v;
        const float u = delta * xv[i];
        const float dl = delta * kLog2e;
        float4 hh = h[i];
        hh.x = fmaf(exp2_hw(dl * a[i].x), hh.x, u * bv[i].x);
        hh.y = fmaf(exp2_hw(dl * a[i].y), hh.y, u * bv[i].y);
        hh.z = fmaf(exp2_hw(dl * a[i].z), hh.z, u * bv[i].z);
        hh.w = fmaf(exp2_hw(dl * a[i].w), hh.w, u * bv[i].w);
        float y = hh.x * cv[i].x;
        y = fmaf(hh.y, cv[i].y, y);
        y = fmaf(hh.z, cv[i].z, y);
        y = fmaf(hh.w, cv[i].w, y);
        y = channel_sum<Q>(y);
        if (!p_ok) {
            const float nan = __int_as_float(0x7fc00000);
            hh = make_float4(nan, nan, nan, nan);
            y = nan;
        }
        if (live[i]) {
            st_stream(reinterpret_cast<float4 *>(states.out) + j * row4 + f[i], hh);
            if (f[i] - d[i] * Q == 0) {
                y = fmaf(dsk[i], xv[i], y);
                if constexpr (HAS_Z) y *= silu_f32(zv[i]);
                st_io(out, j * D + d[i], y);
            }
        }
    }
}

// The same step with what a channel's lanes have in common formed once per channel: with several float4s per lane
// (many branches: the launch moves tens of MB and lives on bandwidth) a workgroup covers 64 U channels, one per
// thread, and every lane of the plain kernel above would fetch x, dt, z, dt_bias and D of each of its U channels for
// itself: five small loads per piece, each a full trip through the address unit for 2 or 4 bytes a lane, and softplus
// and SiLU four times per channel.  Here the state rows are requested first, each thread then does one channel's
// token-side work (same operations in the same order, so the results are bit for bit the plain kernel's) and leaves
// delta * log2(e), delta * x, x, D and silu(z) in LDS for the lanes that own the channel's states.
// grid: (ceil(D * N / 4 / (256 * U)), n_out)
template <typename T, int N, int U, bool HAS_Z, bool SOFTPLUS>
__global__ void __launch_bounds__(kBlock)
state_step_shared_kernel(float *h_out, const float *h_in, const int32_t *__restrict__ parent,
                         const T *__restrict__ x, const T *__restrict__ dt, const float *__restrict__ A,
                         const T *__restrict__ Bm, const T *__restrict__ Cm,
                         const float *__restrict__ Dskip, const T *__restrict__ z,
                         const float *__restrict__ dt_bias, T *__restrict__ out, int64_t n_in, int64_t D)
{
    constexpr int Q = N / 4;
    constexpr int kChannels = kBlock * U / Q;                     // channels whose states this workgroup owns
    __shared__ __attribute__((aligned(16))) float4 ch4[kChannels];   // delta * log2(e), delta * x, x, D
    __shared__ float chg[kChannels];                                  // silu(z)
    const int64_t j = blockIdx.y;
    const int64_t row4 = D * Q;  // float4s per branch
    const int64_t d_lo = (int64_t)blockIdx.x * kChannels;
    const float4 *a4 = reinterpret_cast<const float4 *>(A);

    // the state rows are the bytes that count: the parent index and their requests go out first
    const int64_t p = parent ? (int64_t)parent[j] : j;
    const bool p_ok = p >= 0 && p < n_in;
    const float4 *hin4 = reinterpret_cast<const float4 *>(h_in) + (p_ok ? p : 0) * row4;
    int64_t f[U];
    bool live[U];
    float4 h[U], a[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int64_t f_raw = ((int64_t)blockIdx.x * U + i) * kBlock + threadIdx.x;
        live[i] = f_raw < row4;
        f[i] = live[i] ? f_raw : row4 - 1;
        h[i] = ld_stream(hin4 + f[i]);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) a[i] = a4[f[i]];
    const int q = (int)(threadIdx.x % Q);                         // 256 i is a multiple of Q: the same for all pieces
    const float4 bv = ld4_io<N>(Bm + j * N + 4 * q), cv = ld4_io<N>(Cm + j * N + 4 * q);

    for (int c = threadIdx.x; c < kChannels; c += kBlock) {
        const int64_t dc = d_lo + c;
        if (dc >= D) break;
        const float xv = ld_io(x, j * D + dc);
        const float v = ld_io(dt, j * D + dc) + (dt_bias ? dt_bias[dc] : 0.0f);
        const float zv = HAS_Z ? ld_io(z, j * D + dc) : 0.0f;
        const float delta = SOFTPLUS ? softplus_f32(v) : v;
        ch4[c] = make_float4(delta * kLog2e, delta * xv, xv, Dskip ? Dskip[dc] : 0.0f);
        if constexpr (HAS_Z) chg[c] = silu_f32(zv);
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int64_t d = f[i] / Q;
        const int ci = (int)(d - d_lo);
        const float4 t = ch4[ci];
        const float dl = t.x, u = t.y;
        float4 hh = h[i];
        hh.x = fmaf(exp2_hw(dl * a[i].x), hh.x, u * bv.x);
        hh.y = fmaf(exp2_hw(dl * a[i].y), hh.y, u * bv.y);
        hh.z = fmaf(exp2_hw(dl * a[i].z), hh.z, u * bv.z);
        hh.w = fmaf(exp2_hw(dl * a[i].w), hh.w, u * bv.w);
        float y = hh.x * cv.x;
        y = fmaf(hh.y, cv.y, y);
        y = fmaf(hh.z, cv.z, y);
        y = fmaf(hh.w, cv.w, y);
        y = channel_sum<Q>(y);
        if (!p_ok) {
            const float nan = __int_as_float(0x7fc00000);
            hh = make_float4(nan, nan, nan, nan);
            y = nan;
        }
        if (live[i]) {
            st_stream(reinterpret_cast<float4 *>(h_out) + j * row4 + f[i], hh);
            if (f[i] - d * Q == 0) {
                y = fmaf(t.w, t.z, y);
                if constexpr (HAS_Z) y *= chg[ci];
                st_io(out, j * D + d, y);
            }
        }
    }
}

// H carried inputs of a channel (or K taps), one run of memory: moved as widely as its alignment allows.
template <typename T, int COUNT> struct Run { T v[COUNT]; };
template <typename T, int COUNT> __device__ __forceinline__ Run<T, COUNT> ld_run(const T *p)
{
    Run<T, COUNT> r;
    __builtin_memcpy(&r, p, sizeof(r));
    return r;
}
__device__ __forceinline__ float as_f32(float v) { return v; }
__device__ __forceinline__ float as_f32(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ float from_lane(float v, unsigned byte_of_lane) { return __int_as_float(__builtin_amdgcn_ds_bpermute((int)byte_of_lane, __float_as_int(v))); }

// Fork, conv step and state update of one layer in a single launch (Sec. 4.1: a child continues from its parent's
// states; the draft loop of a tree is this, once per layer and position).  x is the input *before* the conv:
//   win = conv_src[p, d, :];  a = conv_bias[d] + sum_k w[d,k] win[k] + w[d,K-1] x[j,d];  x_c = silu(a)
//   conv_dst[j, d, :] = (win[1..], x[j,d]);  then the step above on x_c rounded to the I/O type
// in the arithmetic order of the conv kernel and of the step kernel, so that the result is bit for bit what
// mamba_conv1d_fwd (L = 1, on the window gathered by parent) followed by mamba_state_step gives.
// A wavefront owns 64 P / Q adjacent channels of a branch (Q = N / 4) in two layouts.  Channel layout (a lane per channel):
// everything that there is once per channel, i.e. window, taps, input, dt, z and the parameters, the conv, softplus, the gate
// and the stores of window and output.  State layout: piece i of P is the float4s 64 i .. 64 i + 63 of the channels' states,
// one contiguous KiB; lane l of it works on channel (64 i + l) / Q.  delta * log2(e) and delta * x go from the first to the
// second by one lane permutation each per piece, the sums come back by one: no LDS memory, no barrier.
// What bounds a launch of a few branches is a wavefront's own chain, parent index -> state row -> arithmetic -> store, and the
// instructions in it: with every lane of a channel doing the channel's work (five small loads, softplus and gate four
// times) and the conv in one wavefront of a workgroup behind a barrier 32 x 1536 took 3.71 us in a replayed graph and 64 x
// 4096 9.39; now 3.33 and 8.74, where a bare copy of the same state rows takes 2.4 and 7.6 and an empty launch 1.6.
// grid: (ceil(D / (64 P / Q)), n_out)
template <typename T, int N, int K, int P, bool HAS_Z, bool SOFTPLUS>
__global__ void __launch_bounds__(64)
state_step_conv_kernel(const int32_t *__restrict__ parent, const float *h_in, const T *conv_src, const T *__restrict__ x,
                       const float *__restrict__ A, const T *__restrict__ dt, const T *__restrict__ z,
                       const T *__restrict__ Bm, const T *__restrict__ Cm, const float *__restrict__ conv_w,
                       const float *__restrict__ conv_bias, const float *__restrict__ dt_bias, const float *__restrict__ Dskip,
                       float *h_out, T *conv_dst, T *__restrict__ out, T *__restrict__ xc_out, int64_t n_in, uint32_t D, int conv_silu)
{
    constexpr int Q = N / 4, H = K - 1;
    constexpr unsigned kPer = 64 / Q, kCh = kPer * P;             // channels of a piece and of the wavefront
    const unsigned lane = threadIdx.x, j = blockIdx.y, d0 = blockIdx.x * kCh;
    const int32_t parent_in = (parent ? parent : reinterpret_cast<const int32_t *>(A))[parent ? j : 0];
    const unsigned nd = min(D - d0, kCh);
    const unsigned c = min(lane % kCh, nd - 1);                   // (offsets of a lane are 32 bits from a scalar base)
    const bool live = lane < nd;
    const int64_t row = (int64_t)((uint64_t)j * D + d0);

    // what does not depend on the parent index
    const T xr = (x + row)[c], dtr = (dt + row)[c];
    T zr{};
    if constexpr (HAS_Z) zr = (z + row)[c];
    const Run<float, K> taps = ld_run<float, K>(conv_w + (uint64_t)d0 * K + c * K);
    const float cb_in = ((conv_bias ? conv_bias : A) + d0)[c], bias_in = ((dt_bias ? dt_bias : A) + d0)[c], dsk_in = ((Dskip ? Dskip : A) + d0)[c];
    const unsigned q = lane % Q;                                  // 64 i is a multiple of Q: the same for all pieces
    const Run<T, 4> br = ld_run<T, 4>(static_cast<const T *>(__builtin_assume_aligned(Bm + j * N + 4 * q, 4 * sizeof(T))));
    const Run<T, 4> cr = ld_run<T, 4>(static_cast<const T *>(__builtin_assume_aligned(Cm + j * N + 4 * q, 4 * sizeof(T))));
    unsigned f[P];
    float4 h[P], a[P];
    const float4 *a4 = reinterpret_cast<const float4 *>(A) + (uint64_t)d0 * Q;
#pragma unroll
    for (unsigned i = 0; i < P; ++i) {
        f[i] = min(64 * i + lane, nd * Q - 1);
        a[i] = a4[f[i]];
    }
    // the window and the state rows
    const int64_t p = parent ? (int64_t)parent_in : (int64_t)j;
    const bool p_ok = p >= 0 && p < n_in;
    const uint64_t pd = (uint64_t)(p_ok ? (uint32_t)p : 0u) * D + d0;
    const Run<T, H> win = ld_run<T, H>(conv_src + pd * H + c * H);
    const float4 *hin4 = reinterpret_cast<const float4 *>(h_in) + pd * Q;
#pragma unroll
    for (int i = 0; i < P; ++i) h[i] = ld_stream(hin4 + f[i]);
    __builtin_amdgcn_sched_barrier(0);                            // all of it in flight before any of it is used

    // conv step, same order of operations as the conv kernel: bias, taps oldest to newest, the new input last
    const float nan = __int_as_float(0x7fc00000);
    const float xpre = as_f32(xr);
    float acc = conv_bias ? cb_in : 0.0f;
#pragma unroll
    for (int k = 0; k < H; ++k) acc = fmaf(taps.v[k], as_f32(win.v[k]), acc);
    acc = fmaf(taps.v[H], xpre, acc);
    const float xc = conv_silu ? silu_f32(acc) : acc;
    const float xv = sizeof(T) == 2 ? bf16_to_f32(f32_to_bf16(xc)) : xc;    // the stored tensor the step would read
    if (live) {
        // new window: the carried inputs move up, the new input comes last (NaN in front where the parent was bad)
        Run<T, H> nwin;
#pragma unroll
        for (int k = 0; k + 1 < H; ++k) {
            nwin.v[k] = win.v[k + 1];
            if (!p_ok) st_io(nwin.v, k, nan);
        }
        nwin.v[H - 1] = xr;
        __builtin_memcpy(conv_dst + row * H + c * H, &nwin, sizeof(nwin));
        if (xc_out) st_io(xc_out + row, c, p_ok ? xc : nan);
    }

    const float v = as_f32(dtr) + (dt_bias ? bias_in : 0.0f);
    const float delta = SOFTPLUS ? softplus_f32(v) : v;
    // (a bad parent's states and output become NaN through the input term; x + -0 is x, its sign included)
    const float u = delta * xv + (p_ok ? -0.0f : nan);
    const float dl = delta * kLog2e;
    float bv[4], cv[4], y = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bv[k] = as_f32(br.v[k]);
        cv[k] = as_f32(cr.v[k]);
    }
    float4 *hout4 = reinterpret_cast<float4 *>(h_out) + row * Q;
#pragma unroll
    for (unsigned i = 0; i < P; ++i) {
        const unsigned from = (lane / Q + i * kPer) * 4;
        const float dli = Q == 1 ? dl : from_lane(dl, from), ui = Q == 1 ? u : from_lane(u, from);
        float4 hh = h[i];
        hh.x = fmaf(exp2_hw(dli * a[i].x), hh.x, ui * bv[0]);
        hh.y = fmaf(exp2_hw(dli * a[i].y), hh.y, ui * bv[1]);
        hh.z = fmaf(exp2_hw(dli * a[i].z), hh.z, ui * bv[2]);
        hh.w = fmaf(exp2_hw(dli * a[i].w), hh.w, ui * bv[3]);
        float yi = hh.x * cv[0];
        yi = fmaf(hh.y, cv[1], yi);
        yi = fmaf(hh.z, cv[2], yi);
        yi = fmaf(hh.w, cv[3], yi);
        yi = channel_sum<Q>(yi);
        y = q == i ? yi : y;                                      // all Q lanes of a channel have it: lane q keeps piece q's
        if (64 * i + lane < nd * Q) st_stream(hout4 + f[i], hh);
    }
    y = Q == 1 ? y : from_lane(y, (lane % kPer * Q + lane / kPer) * 4);
    y = fmaf(Dskip ? dsk_in : 0.0f, xv, y);
    if constexpr (HAS_Z) y *= silu_f32(as_f32(zr));
    if (live) st_io(out + row, c, y);
}

// The same step for a draft position of the whole block (bf16, softplus, gate), where the x projection arrives as partial sums (see
// StepArgs::xpart).  The branch's row of it (dt low rank | B | C) is n_parts runs of xn = dt_rank + 2 N floats: they are added up
// in order and rounded to bf16, as the stored tensors they replace would have been.  The workgroup reads `sides` contiguous ranges
// of `per` parts side by side, as many as it has threads for, 16 bytes each, and adds those few sums up from LDS; then dt (through
// the fused dt projection), B and C come out of LDS.  The parts are what the step waits for first, so the first eight of a range are
// requested ahead of everything else; the state row, behind the parent index, last.  Longer ranges (MORE: wide models) go on by eight.
// Nothing but the parts' trip to memory is long here: what counts is the instructions between the launch and the last store.
// Offsets of a lane are 32 bits from scalar bases (step_xproj_fits), the split of the parts is worked out on the host, and the shapes that occur have
// no conditions left (EXACT: eight parts to every range; NC: pieces of four dt weights per lane, 0: any number).  us a launch in a
// replayed graph, 1 / 12 / 48 rows (before: divisions by the run's length, 64-bit offsets, loops of unknown length): 1024 channels 2.70 /
// 2.82 / 4.17 (3.24 / 3.37 / 4.52), 1536 2.39 / 3.00 / 5.52 (3.28 / 3.84 / 6.12), 4096 5.4 / 9.2 / 18.7 (7.1 / 9.6 / 19.5), 5120 7.0 / 13.4 /
// 35.4 (9.0 / 13.5 / 37.7).
// grid: (ceil(D * N / 4 / (256 * U)), n_out)
constexpr int kParts = 8;
template <typename V> __device__ __forceinline__ V ld_at(const void *base, unsigned byte) { return *reinterpret_cast<const V *>(static_cast<const char *>(base) + byte); }
struct XprojSplit {
    int sides, per, magic;                                        // thread t reads range t * magic >> 16
};
__host__ __device__ inline XprojSplit xproj_split(int xn, int n_parts)
{
    const int xn4 = xn / 4, sides = kBlock / xn4 < n_parts ? kBlock / xn4 : n_parts;
    return {sides, (n_parts + sides - 1) / sides, (65536 + xn4 - 1) / xn4};   // t < 256 and xn4 <= 64: t / xn4 exactly
}

template <int N, int U, int NC, bool EXACT, bool MORE>
__global__ void __launch_bounds__(kBlock)
state_step_xproj_kernel(const float *__restrict__ xpart, int n_parts, int sides_in, int per, int magic, int D, int dt_rank_in, const int32_t *__restrict__ parent,
                        const float *h_in, const bf16_t *__restrict__ dt_w, const bf16_t *__restrict__ x, const bf16_t *__restrict__ z,
                        const float *__restrict__ A, const float *__restrict__ dt_bias, const float *__restrict__ Dskip, float *h_out,
                        bf16_t *__restrict__ out, int64_t n_in)
{
    constexpr int Q = N / 4, CW = NC ? NC : 4;                    // CW: dt_w pieces a lane can hold ahead of the x projection sums
    __shared__ __attribute__((aligned(16))) float xs[256], xs_side[kBlock * 4 + 4];   // + 4: where threads past the last range write
    const unsigned tid = threadIdx.x, j = blockIdx.y;
    const int dt_rank = NC ? 4 * NC * Q : dt_rank_in, xn = dt_rank + 2 * N;
    const int sides = NC && EXACT ? kBlock / (xn >> 2) : sides_in;   // (eight parts to a range: there are more parts than ranges)
    const unsigned xn4 = (unsigned)xn >> 2, row4 = (unsigned)D * Q;

    // ---- the partial sums
    const unsigned side = NC ? tid / xn4 : tid * (unsigned)magic >> 16, k4 = tid - side * xn4;
    const unsigned sd = min(side, (unsigned)sides - 1), first = sd * (unsigned)per;
    const unsigned count = EXACT ? kParts : first < (unsigned)n_parts ? min((unsigned)per, (unsigned)n_parts - first) : 0u;   // parts of this range
    const float4 *pr = reinterpret_cast<const float4 *>(xpart) + (uint64_t)j * (unsigned)n_parts * xn4;
    const unsigned at = ((EXACT || first < (unsigned)n_parts ? first : 0u) * xn4 + k4) * 16, part_bytes = xn4 * 16;
    float4 pv[kParts];
#pragma unroll
    for (unsigned u = 0; u < kParts; ++u) pv[u] = ld_at<float4>(pr, at + (EXACT ? u : min(u, count ? count - 1 : 0u)) * part_bytes);
    __builtin_amdgcn_sched_barrier(0);

    // ---- everything else that does not depend on the x projection
    const int32_t parent_in = (parent ? parent : reinterpret_cast<const int32_t *>(dt_w))[parent ? j : 0];
    unsigned f[U], d[U];
    const unsigned q = tid % Q;                                   // 256 i is a multiple of Q: the same for all pieces
    float4 h[U], a[U];
    bf16_t xr[U], zr[U];
    float bias_in[U], dsk_in[U];
    uint2 wq[U][CW];
    const unsigned pieces = NC ? NC * Q : (unsigned)dt_rank >> 2;
    const bool hold_w = NC || pieces <= CW * Q;
#pragma unroll
    for (unsigned i = 0; i < U; ++i) {
        f[i] = min((blockIdx.x * U + i) * kBlock + tid, row4 - 1);
        d[i] = f[i] / Q;
#pragma unroll
        for (unsigned c = 0; c < CW; ++c) {
            const unsigned cc = q + c * Q;
            wq[i][c] = make_uint2(0, 0);
            if constexpr (NC) wq[i][c] = ld_at<uint2>(dt_w, (d[i] * (NC * Q) + q) * 8 + c * Q * 8);
            else if (hold_w && cc < pieces) wq[i][c] = reinterpret_cast<const uint2 *>(dt_w)[(uint64_t)d[i] * pieces + cc];
        }
        a[i] = ld_at<float4>(A, 16 * f[i]);
        xr[i] = ld_at<bf16_t>(x + (uint64_t)j * (unsigned)D, 2 * d[i]);
        zr[i] = ld_at<bf16_t>(z + (uint64_t)j * (unsigned)D, 2 * d[i]);
        bias_in[i] = ld_at<float>(dt_bias ? dt_bias : A, 4 * d[i]);
        dsk_in[i] = ld_at<float>(Dskip ? Dskip : A, 4 * d[i]);
    }
    const int64_t p = parent ? (int64_t)parent_in : (int64_t)j;
    const bool p_ok = p >= 0 && p < n_in;
    const float4 *hin4 = reinterpret_cast<const float4 *>(h_in) + (uint64_t)(p_ok ? (uint32_t)p : 0u) * row4;
#pragma unroll
    for (int i = 0; i < U; ++i) h[i] = ld_stream(reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(hin4) + 16 * f[i]));
    __builtin_amdgcn_sched_barrier(0);                            // all of it in flight before any of it is used
    args_here(h_out, out);

    {
        float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto add = [&](float4 v, bool use) __attribute__((always_inline)) {
            sum.x += use ? v.x : 0.0f; sum.y += use ? v.y : 0.0f; sum.z += use ? v.z : 0.0f; sum.w += use ? v.w : 0.0f;
        };
#pragma unroll
        for (unsigned u = 0; u < kParts; ++u) add(pv[u], EXACT || u < count);
        if constexpr (MORE) {
            for (unsigned c = kParts; c < count; c += kParts) {   // as many in flight again
#pragma unroll
                for (unsigned u = 0; u < kParts; ++u) pv[u] = ld_at<float4>(pr, at + min(c + u, count - 1) * part_bytes);
#pragma unroll
                for (unsigned u = 0; u < kParts; ++u) add(pv[u], c + u < count);
            }
        }
        // (unconditional: under a condition the compiler would move the requests in there too)
        *reinterpret_cast<float4 *>(&xs_side[side < (unsigned)sides ? side * xn + 4 * k4 : kBlock * 4]) = sum;
    }
    lds_barrier_s();
    if (tid < (unsigned)xn) {
        float sum = 0.0f;
        constexpr int kTurn = NC && EXACT ? kBlock / (NC * Q + N / 2) : 12;
        for (int u0 = 0; u0 < sides; u0 += kTurn) {
            float v[kTurn];
#pragma unroll
            for (int u = 0; u < kTurn; ++u) v[u] = xs_side[(NC && EXACT ? u : min(u0 + u, sides - 1)) * xn + tid];
#pragma unroll
            for (int u = 0; u < kTurn; ++u) sum += (NC && EXACT) || u0 + u < sides ? v[u] : 0.0f;
        }
        xs[tid] = bf16_to_f32(f32_to_bf16(sum));
    }
    lds_barrier_s();

    const float4 bv = *reinterpret_cast<const float4 *>(&xs[dt_rank + 4 * q]), cv = *reinterpret_cast<const float4 *>(&xs[dt_rank + N + 4 * q]);
#pragma unroll
    for (int i = 0; i < U; ++i) {
        float acc = 0.0f;
        auto dot = [&](uint2 w, unsigned cc) __attribute__((always_inline)) {
            const float4 b4 = *reinterpret_cast<const float4 *>(&xs[4 * cc]);
            acc = fmaf(bf16_lo(w.x), b4.x, acc);
            acc = fmaf(bf16_hi(w.x), b4.y, acc);
            acc = fmaf(bf16_lo(w.y), b4.z, acc);
            acc = fmaf(bf16_hi(w.y), b4.w, acc);
        };
        if (hold_w) {
#pragma unroll
            for (unsigned c = 0; c < CW; ++c) dot(wq[i][c], NC || q + c * Q < pieces ? q + c * Q : 0u);
        } else {
            const uint2 *wrow = reinterpret_cast<const uint2 *>(dt_w) + (uint64_t)d[i] * pieces;
            for (unsigned c = q; c < pieces; c += Q) dot(wrow[c], c);
        }
        const float xv = bf16_to_f32(xr[i]);
        const float delta = softplus_f32(bf16_to_f32(f32_to_bf16(channel_sum<Q>(acc))) + (dt_bias ? bias_in[i] : 0.0f));
        const float u = delta * xv + (p_ok ? -0.0f : __int_as_float(0x7fc00000));   // (x + -0 is x; a bad parent poisons states and output)
        const float dl = delta * kLog2e;
        float4 hh = h[i];
        hh.x = fmaf(exp2_hw(dl * a[i].x), hh.x, u * bv.x);
        hh.y = fmaf(exp2_hw(dl * a[i].y), hh.y, u * bv.y);
        hh.z = fmaf(exp2_hw(dl * a[i].z), hh.z, u * bv.z);
        hh.w = fmaf(exp2_hw(dl * a[i].w), hh.w, u * bv.w);
        float y = hh.x * cv.x;
        y = fmaf(hh.y, cv.y, y);
        y = fmaf(hh.z, cv.z, y);
        y = fmaf(hh.w, cv.w, y);
        y = channel_sum<Q>(y);
        if ((blockIdx.x * U + i) * kBlock + tid < row4) {
            st_stream(reinterpret_cast<float4 *>(h_out) + (uint64_t)j * row4 + f[i], hh);
            if (q == 0) st_io(out + (uint64_t)j * (unsigned)D, d[i], fmaf(Dskip ? dsk_in[i] : 0.0f, xv, y) * silu_f32(bf16_to_f32(zr[i])));
        }
    }
}

template <typename T, int N, int U> hipError_t launch_step_u(const StepArgs &a, hipStream_t stream)
{
    const int64_t row4 = a.D * (N / 4);
    const int64_t per_block = (int64_t)kBlock * U;
    dim3 grid((unsigned)((row4 + per_block - 1) / per_block), (unsigned)a.n_out);
    if (U > 1 && !a.dt_w) {
#define MAMBA_STEP_S(HZ, SP)                                                                      \
    state_step_shared_kernel<T, N, U, HZ, SP><<<grid, kBlock, 0, stream>>>(                       \
        a.h_out, a.h_in, a.parent, static_cast<const T *>(a.x), static_cast<const T *>(a.dt), a.A, \
        static_cast<const T *>(a.Bm), static_cast<const T *>(a.Cm), a.Dskip,                      \
        static_cast<const T *>(a.z), a.dt_bias, static_cast<T *>(a.out), a.n_in, a.D)
        if (a.z) {
            if (a.dt_softplus) MAMBA_STEP_S(true, true);
            else MAMBA_STEP_S(true, false);
        } else {
            if (a.dt_softplus) MAMBA_STEP_S(false, true);
            else MAMBA_STEP_S(false, false);
        }
#undef MAMBA_STEP_S
        return hipGetLastError();
    }
    if constexpr (U <= kStepUnroll) {
#define MAMBA_STEP(HZ, SP)                                                                        \
    state_step_kernel<T, N, U, HZ, SP><<<grid, kBlock, 0, stream>>>(                              \
        StepStates{a.h_out, a.h_in}, a.parent, static_cast<const T *>(a.x), static_cast<const T *>(a.dt), a.A, \
        static_cast<const T *>(a.Bm), static_cast<const T *>(a.Cm), a.Dskip,                      \
        static_cast<const T *>(a.z), a.dt_bias, static_cast<T *>(a.out), a.n_in, a.D,                \
        static_cast<const bf16_t *>(a.dt_w), a.dt_rank)
    if (a.z) {
        if (a.dt_softplus) MAMBA_STEP(true, true);
        else MAMBA_STEP(true, false);
    } else {
        if (a.dt_softplus) MAMBA_STEP(false, true);
        else MAMBA_STEP(false, false);
    }
#undef MAMBA_STEP
    return hipGetLastError();
    } else {
        return hipErrorInvalidValue;   // eight float4s per lane exist for the plain step only
    }
}

template <typename T, int N, int K, int P> hipError_t launch_step_conv(const StepArgs &a, hipStream_t stream)
{
    constexpr int kCh = 64 / (N / 4) * P;
    const dim3 grid((unsigned)((a.D + kCh - 1) / kCh), (unsigned)a.n_out);
#define MAMBA_STEP_C(HZ, SP)                                                                      \
    state_step_conv_kernel<T, N, K, P, HZ, SP><<<grid, 64, 0, stream>>>(                             \
        a.parent, a.h_in, static_cast<const T *>(a.conv_src), static_cast<const T *>(a.x), a.A,   \
        static_cast<const T *>(a.dt), static_cast<const T *>(a.z), static_cast<const T *>(a.Bm),  \
        static_cast<const T *>(a.Cm), a.conv_w, a.conv_bias, a.dt_bias, a.Dskip, a.h_out,         \
        static_cast<T *>(a.conv_dst), static_cast<T *>(a.out), static_cast<T *>(a.xc_out), a.n_in, (uint32_t)a.D, a.conv_silu)
    if (a.z) {
        if (a.dt_softplus) MAMBA_STEP_C(true, true);
        else MAMBA_STEP_C(true, false);
    } else {
        if (a.dt_softplus) MAMBA_STEP_C(false, true);
        else MAMBA_STEP_C(false, false);
    }
#undef MAMBA_STEP_C
    return hipGetLastError();
}

template <int N, int U> hipError_t launch_step_xproj(const StepArgs &a, hipStream_t stream)
{
    const int64_t per_block = (int64_t)kBlock * U, row4 = a.D * (N / 4);
    const dim3 grid((unsigned)((row4 + per_block - 1) / per_block), (unsigned)a.n_out);
    const XprojSplit sp = xproj_split((int)a.dt_rank + 2 * N, a.n_parts);
    const bool exact = sp.per == kParts && sp.sides * kParts == a.n_parts, more = sp.per > kParts;
#define MAMBA_STEP_X(NC, EX, MR)                                                                  \
    state_step_xproj_kernel<N, U, NC, EX, MR><<<grid, kBlock, 0, stream>>>(                       \
        a.xpart, a.n_parts, sp.sides, sp.per, sp.magic, (int)a.D, (int)a.dt_rank, a.parent, a.h_in,                       \
        static_cast<const bf16_t *>(a.dt_w), static_cast<const bf16_t *>(a.x), static_cast<const bf16_t *>(a.z), a.A, \
        a.dt_bias, a.Dskip, a.h_out, static_cast<bf16_t *>(a.out), a.n_in)
#define MAMBA_STEP_XC(NC) do { if (exact) MAMBA_STEP_X(NC, true, false); else if (more) MAMBA_STEP_X(NC, false, true); else MAMBA_STEP_X(NC, false, false); } while (0)
    if constexpr (N == 16) {
        switch (a.dt_rank) {
        case 32: MAMBA_STEP_XC(2); return hipGetLastError();
        case 48: MAMBA_STEP_XC(3); return hipGetLastError();
        case 64: MAMBA_STEP_XC(4); return hipGetLastError();
        default: break;
        }
    }
    MAMBA_STEP_XC(0);
#undef MAMBA_STEP_XC
#undef MAMBA_STEP_X
    return hipGetLastError();
}

template <typename T, int N> hipError_t launch_step_n(const StepArgs &a, hipStream_t stream)
{
    if (a.conv_w) {
        // Four pieces per wavefront, two while those come to no more than one wavefront per SIMD.  us a launch in a
        // replayed graph on 4 / 2 pieces: 4 x 768 2.43 / 2.23, 32 x 768 3.16 / 2.99, 32 x 1536 3.33 / 3.38, 64 x 1536 4.73 /
        // 5.00, 64 x 4096 8.74 / 9.18, 128 x 4096 14.90 / 16.18
        constexpr int Q = N / 4, kFew = Q < 2 ? Q : 2, kMany = Q < 4 ? Q : 4;
        if (!conv_step_fits(a.D, N)) return hipErrorInvalidValue;
        const bool few = a.n_out * ((a.D + 64 / Q * kFew - 1) / (64 / Q * kFew)) <= 1024;
        switch (a.conv_k) {
        case 2: return few ? launch_step_conv<T, N, 2, kFew>(a, stream) : launch_step_conv<T, N, 2, kMany>(a, stream);
        case 3: return few ? launch_step_conv<T, N, 3, kFew>(a, stream) : launch_step_conv<T, N, 3, kMany>(a, stream);
        case 4: return few ? launch_step_conv<T, N, 4, kFew>(a, stream) : launch_step_conv<T, N, 4, kMany>(a, stream);
        default: return hipErrorInvalidValue;
        }
    }
    // several float4s per lane as long as that still leaves about three workgroups per CU
    const int64_t row4 = a.D * (N / 4);
    auto blocks = [&](int u) { return a.n_out * ((row4 + kBlock * u - 1) / (kBlock * u)); };
    // the plain step with eight per lane while that gives between 1.5 and 4 workgroups per CU: 64 branches x 4096
    // channels 8.7 -> 7.6 us, the time of a bare copy of the same state rows; 128 branches are better off with four
    if (!a.dt_w && blocks(8) >= 384 && blocks(8) < 1024) return launch_step_u<T, N, 8>(a, stream);
    if constexpr (sizeof(T) == 2) {
        if (a.xpart) {
            if (!a.dt_w || !a.z || !a.dt_softplus || a.dt_rank + 2 * N > kBlock || a.dt_rank % 4 || a.n_parts < 1 || !step_xproj_fits(a.D, N, a.dt_rank)) return hipErrorInvalidValue;
            if (blocks(4) >= 768) return launch_step_xproj<N, 4>(a, stream);
            return blocks(2) >= 768 ? launch_step_xproj<N, 2>(a, stream) : launch_step_xproj<N, 1>(a, stream);
        }
    }
    if (blocks(kStepUnroll) >= 768) return launch_step_u<T, N, kStepUnroll>(a, stream);
    if (kStepUnroll > 2 && blocks(2) >= 768) return launch_step_u<T, N, 2>(a, stream);
    return launch_step_u<T, N, 1>(a, stream);
}

template <typename T> hipError_t launch_step_io(const StepArgs &a, hipStream_t stream)
{
    switch (a.N) {
    case 4: return launch_step_n<T, 4>(a, stream);
    case 8: return launch_step_n<T, 8>(a, stream);
    case 16: return launch_step_n<T, 16>(a, stream);
    case 32: return launch_step_n<T, 32>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_step(const StepArgs &a, hipStream_t stream)
{
    if (a.io == kIoBf16) return launch_step_io<bf16_t>(a, stream);
    return launch_step_io<float>(a, stream);
}

}  // namespace mamba
