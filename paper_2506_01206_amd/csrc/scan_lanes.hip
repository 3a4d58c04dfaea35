// Selective scan in a single pass for shapes with few independent channels (one sequence, or a few, of a
// Mamba-130M-sized layer: the contexts of a few thousand tokens the paper's drafter encodes, Sec. 3.1 and the
// long-context experiments), gfx950, N = 16.  Same arithmetic as scan.hip:
//
//   delta = softplus(dt + dt_bias);  h_t = exp(delta_t A) h_{t-1} + delta_t B_t x_t
//   y_t = C_t . h_t + D x_t;  out_t = y_t silu(z_t)
//
// With 1536 channels there is not enough channel parallelism for 1024 SIMDs, so time has to run in
// parallel somewhere.  Here it runs across the lanes of a wavefront instead of across workgroups: no chunk
// states in memory, no carry kernel, every token read once, exp evaluated once per state update.
//
// (Every workgroup then reads its own 12 bytes of every token row, a 64-byte request each: at a few thousand
// tokens this beats the two-pass kernels' launches and hand-overs, on long sequences their full-line accesses
// win; scan_lanes_applies draws the line.)
//
// A workgroup owns 6 adjacent channels (256 workgroups for 1536 channels; 4 or 2 of a narrower layer, so that it still has as
// many: 1 x 1000 x 768 15.2 -> 12.4 us, 1 x 1000 x 512 15.7 -> 10.4) and walks the sequence in
// super-steps of 512 (384, 256) tokens.  Its 12 (8, 4) wavefronts are (channel pair, group of 4 states); the 64 lanes of a
// wavefront are 64 consecutive blocks of 8 tokens (or 6 or 4, lanes_tau).  Per super-step a lane
//   1. integrates its 8 tokens from a zero state (lane 0 from the true state that enters the super-step),
//      keeping the 8 x 8 decay factors a = exp(delta A) in registers: mul, exp2, mul, fma per update;
//   2. forms the decay over its whole block, P = exp(A * sum of its deltas);
//   3. takes part in an inclusive scan over the 64 lanes of the pairs (P, H) under
//      (P1, H1) o (P2, H2) = (P1 P2, P2 H1 + H2): four row_shr steps inside each row of 16 lanes, then
//      row_bcast:15 and row_bcast:31 across the rows (DPP, no LDS): afterwards H is the true state at the
//      end of the lane's block, and a one-lane rotation hands every lane the state its block starts from
//      (lane 0 thereby receives the state that enters the next super-step);
//   4. walks its 8 tokens again from that state with the stored decays (mul, fma) and accumulates
//      C . h (fma); the four state groups of a channel leave their parts in LDS.
// Loads, per-token arithmetic (softplus, delta * x, skip term, gate) and stores happen in a token layout:
// thread (j, i) of the first 8 wavefronts owns token 8 i + j of the super-step, all 6 channels (B_t and C_t are
// fetched by all threads in consecutive 16-byte pieces);
// operands go to LDS as float32 in layouts in which consecutive lanes touch consecutive 16-byte slots.
// The next super-step's rows are requested at the start of the current one, its B_t and C_t before the second walk (float32: where
// they are used); both are used after that.
#include "device_math.h"
#include "launch.h"
#include "routes.h"

namespace mamba {
namespace {

constexpr int kN = kLanesStates;         // states per channel
constexpr int kParts = 4;                // groups of 4 states
constexpr int kBcPart = 66, kBcTau = kParts * kBcPart + 1;   // slots per state group and per token j of lds_B / lds_C

__device__ __forceinline__ void lds_barrier_l()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One level of the scan for the 8 (P, H) pairs of a lane.  Lanes whose DPP source is valid combine with it,
//   H <- P * H_src + H,  P <- P * P_src,
// the others are left alone (a DPP instruction does not write lanes without a source, and row_mask picks the
// receiving rows of a broadcast).  Written as DPP forms of v_fmac / v_mul, one instruction per update; the
// compiler, given the builtin, moves the source lane into a register first and doubles the count.  Within a
// block every instruction reads registers written at least eight instructions earlier; the s_nop covers the two
// wait states a DPP read needs after a VALU write by whatever precedes the block.
#define MAMBA_SCAN_H(CTRL)                                                   \
    "v_fmac_f32_dpp %0, %0, %8 " CTRL " bank_mask:0xf\n"                     \
    "v_fmac_f32_dpp %1, %1, %9 " CTRL " bank_mask:0xf\n"                     \
    "v_fmac_f32_dpp %2, %2, %10 " CTRL " bank_mask:0xf\n"                    \
    "v_fmac_f32_dpp %3, %3, %11 " CTRL " bank_mask:0xf\n"                    \
    "v_fmac_f32_dpp %4, %4, %12 " CTRL " bank_mask:0xf\n"                    \
    "v_fmac_f32_dpp %5, %5, %13 " CTRL " bank_mask:0xf\n"                    \
    "v_fmac_f32_dpp %6, %6, %14 " CTRL " bank_mask:0xf\n"                    \
    "v_fmac_f32_dpp %7, %7, %15 " CTRL " bank_mask:0xf\n"
#define MAMBA_SCAN_P(CTRL)                                                   \
    "v_mul_f32_dpp %8, %8, %8 " CTRL " bank_mask:0xf\n"                      \
    "v_mul_f32_dpp %9, %9, %9 " CTRL " bank_mask:0xf\n"                      \
    "v_mul_f32_dpp %10, %10, %10 " CTRL " bank_mask:0xf\n"                   \
    "v_mul_f32_dpp %11, %11, %11 " CTRL " bank_mask:0xf\n"                   \
    "v_mul_f32_dpp %12, %12, %12 " CTRL " bank_mask:0xf\n"                   \
    "v_mul_f32_dpp %13, %13, %13 " CTRL " bank_mask:0xf\n"                   \
    "v_mul_f32_dpp %14, %14, %14 " CTRL " bank_mask:0xf\n"                   \
    "v_mul_f32_dpp %15, %15, %15 " CTRL " bank_mask:0xf\n"
#define MAMBA_SCAN_OPERANDS(H, P)                                                                              \
    "+v"(H[0]), "+v"(H[1]), "+v"(H[2]), "+v"(H[3]), "+v"(H[4]), "+v"(H[5]), "+v"(H[6]), "+v"(H[7]),            \
    "+v"(P[0]), "+v"(P[1]), "+v"(P[2]), "+v"(P[3]), "+v"(P[4]), "+v"(P[5]), "+v"(P[6]), "+v"(P[7])

// inclusive scan over the 64 lanes; afterwards H is the state at the end of the lane's block (P is used up)
__device__ __forceinline__ void lane_scan(float (&H)[8], float (&P)[8])
{
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_shr:1 row_mask:0xf") MAMBA_SCAN_P("row_shr:1 row_mask:0xf") : MAMBA_SCAN_OPERANDS(H, P));
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_shr:2 row_mask:0xf") MAMBA_SCAN_P("row_shr:2 row_mask:0xf") : MAMBA_SCAN_OPERANDS(H, P));
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_shr:4 row_mask:0xf") MAMBA_SCAN_P("row_shr:4 row_mask:0xf") : MAMBA_SCAN_OPERANDS(H, P));
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_shr:8 row_mask:0xf") MAMBA_SCAN_P("row_shr:8 row_mask:0xf") : MAMBA_SCAN_OPERANDS(H, P));
    // lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows 2 and 3
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_bcast:15 row_mask:0xa") MAMBA_SCAN_P("row_bcast:15 row_mask:0xa") : MAMBA_SCAN_OPERANDS(H, P));
    asm volatile("s_nop 1\n" MAMBA_SCAN_H("row_bcast:31 row_mask:0xc") : MAMBA_SCAN_OPERANDS(H, P));
}

// lane i <- lane i - 1, lane 0 <- lane 63
__device__ __forceinline__ float wave_rotate1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x13C, 0xf, 0xf, false));
}

// G adjacent channels of one token row, as they lie in memory
template <typename T, int G> struct RowG;
template <int G> struct RowG<bf16_t, G> {
    uint32_t v[G / 2];
    __device__ __forceinline__ void load(const bf16_t *p)
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) v[c] = reinterpret_cast<const uint32_t *>(p)[c];
    }
    __device__ __forceinline__ void unpack(float *f) const
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) f[2 * c] = bf16_lo(v[c]), f[2 * c + 1] = bf16_hi(v[c]);
    }
};
template <int G> struct RowG<float, G> {
    float2 v[G / 2];
    __device__ __forceinline__ void load(const float *p)
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) v[c] = reinterpret_cast<const float2 *>(p)[c];
    }
    __device__ __forceinline__ void unpack(float *f) const
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) f[2 * c] = v[c].x, f[2 * c + 1] = v[c].y;
    }
};
// G adjacent channels of one output row, rounded to the type they are stored as
template <typename T, int G> struct OutG;
template <int G> struct OutG<bf16_t, G> {
    typedef uint32_t words __attribute__((ext_vector_type(G / 2)));
    typedef words words_at4 __attribute__((aligned(4)));
    uint32_t v[G / 2];
    __device__ __forceinline__ void pack(const float *f)
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) v[c] = f32x2_to_bf16x2(f[2 * c], f[2 * c + 1]);
    }
    __device__ __forceinline__ void store(bf16_t *p) const
    {
        if constexpr (G == 6) *reinterpret_cast<words_at4 *>(p) = words{v[0], v[1], v[2]};
        else if constexpr (G == 4) *reinterpret_cast<words_at4 *>(p) = words{v[0], v[1]};
        else *reinterpret_cast<uint32_t *>(p) = v[0];
    }
    __device__ __forceinline__ void store_pair(bf16_t *p, int c) const { reinterpret_cast<uint32_t *>(p)[c] = v[c]; }
};
template <int G> struct OutG<float, G> {
    float2 v[G / 2];
    __device__ __forceinline__ void pack(const float *f)
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) v[c] = make_float2(f[2 * c], f[2 * c + 1]);
    }
    __device__ __forceinline__ void store(float *p) const
    {
#pragma unroll
        for (int c = 0; c < G / 2; ++c) reinterpret_cast<float2 *>(p)[c] = v[c];
    }
    __device__ __forceinline__ void store_pair(float *p, int c) const { reinterpret_cast<float2 *>(p)[c] = v[c]; }
};

// B_t and C_t of a super-step are fetched by all threads in 16-byte chunks, consecutive threads on consecutive
// chunks (fully coalesced), and land in LDS as float32 groups of 4 states.
template <typename T> struct BcChunk;
template <> struct BcChunk<bf16_t> {     // 8 values: two groups of 4 states
    static constexpr int kGroups = 2;
    uint4 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint4 *>(p); }
    __device__ __forceinline__ float4 group(int g) const
    {
        const uint32_t a = g ? v.z : v.x, b = g ? v.w : v.y;
        return make_float4(bf16_lo(a), bf16_hi(a), bf16_lo(b), bf16_hi(b));
    }
};
template <> struct BcChunk<float> {      // 4 values: one group
    static constexpr int kGroups = 1;
    float4 v;
    __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
    __device__ __forceinline__ float4 group(int) const { return v; }
};

// A context of one super-step in a whole block (LOW): the dt projection in here, from its low-rank input.  A workgroup's six channels of
// 512 tokens are 16 small products of a wavefront each on the idle matrix cores, and what it fetches for them is contiguous where
// dt is 12 bytes of every row; as a launch of its own the projection is a trip to memory and back and little else.  us of the scan, and
// of both: 100 x 1536 7.1 -> 7.7, 10.2 -> 7.7; 333 x 1536 10.9 -> 11.4, 14.6 -> 11.4; 24-block prefill of 333 tokens 874 -> 808.  Longer contexts, whose
// next rows are on their way while one super-step is walked, have no registers for it, and their two narrow products share a kernel
// (xdt.hip).
struct LowDt {
    const bf16_t *w;                 // (D, rank)
    bf16_t *out;                     // (batch, L, D): what the projection as a launch of its own would have stored
    int rank;                        // a multiple of 8, at most kLanesLowRank
};

// kG: channels per workgroup (2, 4 or 6); kTau: tokens per lane and super-step (4, 6 or 8), 64 kTau tokens no more than threads.
// grid: (ceil(D / kG) rounded up to a multiple of 8, batch); block: 128 kG.  N = 16, D even and >= kG.
template <typename T, bool HAS_Z, bool SOFTPLUS, int kG, int kTau, bool LOW = false>
__global__ void __launch_bounds__(64 * kParts * (kG / 2))
scan_lanes_kernel(const T *x, const T *dt, const float *__restrict__ A, const T *Bm, const T *Cm,
                  const float *__restrict__ Dskip, const T *z, const float *__restrict__ dt_bias,
                  const float *h0 /* may alias h_final */, T *out, float *h_final, int64_t L, int64_t D, LowDt low)
{
    constexpr int kThreadsL = 64 * kParts * (kG / 2);
    constexpr int kT = 64 * kTau;            // tokens per super-step
    // Exponentials in runs of eight (a token's), logarithms with them.  Runs of 16 spill, and runs of the gate's do in float32.  The
    // one wavefront to a SIMD that two channels make has no others to keep out, only the order to lose: 256 x 256 float32 4.42 us,
    // 4.58 in runs.  With more, us: 2048 x 1536 bf16 28.2 -> 26.8, float32 32.4 -> 31.5; 333 x 1536 9.6 -> 9.3; 8000 x 1536
    // 99.1 -> 97.7; 2000 x 1000 21.2 -> 20.4; 4 x 3000 x 768 74.6 -> 72.0.
    constexpr bool kRuns = kG > 2;
    constexpr int kTokenThreads = kT;        // one token row per thread of the first wavefronts
    static_assert(kTokenThreads <= kThreadsL, "a token row per thread");
    // [token j of the lane's block][state group][lane][4 states]: the lanes of a wavefront read consecutive slots.
    // The threads that fill them write, eight lanes at a time, four consecutive tokens (j) x two state groups two
    // apart: with rows of 66 slots and 265 slots per j those eight 16-byte slots fall on eight different quarters
    // of the banks (j * 265 + 2 * 66 * pos = j + 4 * pos mod 8).
    __shared__ __attribute__((aligned(16))) float4 lds_B[kTau * kBcTau];
    __shared__ __attribute__((aligned(16))) float4 lds_C[kTau * kBcTau];
    // [channel][part of the block][lane][kQ tokens]; rows of two tokens are padded so that the three parts a token row of threads
    // writes fall on different banks
    constexpr int kQ = kTau % 4 == 0 ? 4 : 2, kRow = kQ == 4 ? 64 : 64 + 11;
    typedef float quad __attribute__((ext_vector_type(kQ)));
    __shared__ __attribute__((aligned(16))) quad lds_d[kG][kTau / kQ][kRow];   // delta
    __shared__ __attribute__((aligned(16))) quad lds_u[kG][kTau / kQ][kRow];   // delta * x
    __shared__ __attribute__((aligned(16))) quad lds_y[kParts][kG][kTau / kQ][kRow];   // C . h per token, same layout: one part per state group
    __shared__ float lds_par[2][kG];                                           // dt_bias, D of the workgroup's channels

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t b = blockIdx.y;
    // the last workgroup of a row may have fewer than 6 channels of its own (2 or 4, D being even): it then loads
    // the last 6 of the row, works on all of them, and keeps results only for its own (the leading `dead` ones
    // belong to its neighbour and are neither stored nor taken as a state)
    // Workgroups are dealt to the 8 XCDs in turn (workgroup i runs on XCD i % 8, each with an L2 of its own) and
    // neighbouring channel groups share every 128-byte line of a token row, so the groups are numbered to put
    // neighbours on the same XCD: XCD x takes groups x * per_xcd .. (x + 1) * per_xcd - 1.  The grid is padded to a
    // multiple of 8; a workgroup without a group leaves at once.
    const int64_t n_groups = (D + kG - 1) / kG;
    const int64_t per_xcd = (n_groups + 7) / 8;
    const int64_t group = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || group >= n_groups) return;
    int64_t c0 = group * kG;
    int dead = 0;
    if (c0 + kG > D) {
        dead = (int)(c0 + kG - D);
        c0 = D - kG;
    }
    const int64_t row0 = b * L;

    // ---- token layout (threads of the first 8 wavefronts): thread t has token t of the super-step, which is token
    // tj of the block of lane ti.  (A wavefront's 4-byte accesses to the [..][lane][4 tokens] arrays then cover all
    // banks: 8 lanes x 4 positions.)
    const bool token_thread = tid < kTokenThreads;
    const int tj = tid % kTau, ti = (tid / kTau) & 63;
    // dt_bias and D of the workgroup's channels: one load per thread, requested here and put into LDS only after the
    // first rows have been requested as well (written where it is fetched, wavefront 0 would sit through two
    // memory round trips before it asks for anything else, and the whole workgroup waits for it at the barrier)
    float par = 0.0f;
    if (tid < 2 * kG) {
        const float *src = tid < kG ? dt_bias : Dskip;
        if (src) par = src[c0 + (tid < kG ? tid : tid - kG)];
    }

    // ---- state layout: channels ca, ca + 1 of the workgroup, states 4 * part .. 4 * part + 3, tokens 8 * lane ..
    const int pair = wave / kParts, part = wave % kParts;
    const int ca = 2 * pair;
    float a2[2][4];              // A * log2(e)
    float hp[2][4];              // the state that enters the next super-step: one value per wavefront (scalar registers)
#pragma unroll
    for (int ch = 0; ch < 2; ++ch)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int64_t idx = (c0 + ca + ch) * kN + 4 * part + n;
            a2[ch][n] = A[idx] * kLog2e;
            hp[ch][n] = (h0 && ca >= dead) ? h0[b * D * kN + idx] : 0.0f;   // wave-uniform address
        }

    // With 2-byte elements everything a super-step needs is requested during the one before; with float32 (twice
    // the registers) only x and dt are, and z, B_t, C_t are fetched where they are used.
    constexpr bool kAhead = sizeof(T) == 2;
    RowG<T, kG> x_cur, z_cur;                                            // the super-step's own: kept for the gate
    constexpr int kChunkGroups = BcChunk<T>::kGroups;
    constexpr int kChunksPerRow = kParts / kChunkGroups;             // 2 (bf16) or 4 (float32)
    constexpr int kChunks = 2 * kT * kChunksPerRow;                  // B and C of a super-step
    constexpr int kBcIters = (kChunks + kThreadsL - 1) / kThreadsL;  // 2 to 8
    constexpr int kBcHeld = kAhead ? kBcIters : (kBcIters + 1) / 2;  // chunks a thread holds at a time
    BcChunk<T> bc_nxt[kBcHeld];

    // Addresses are a base of the super-step, which is uniform (scalar registers), and 32 bits of the thread's own (512 rows
    // of the widest layer that takes this kernel, 4608 channels, are far below that): with 64 bits of its own for
    // every tensor the walk had to spill, and a kernel with scratch memory takes 0.4 us longer to start.
    // The last token of a super-step, counted from its start; tokens past it re-read its row and are zeroed at use.
    auto last_of = [&](int64_t t_base) { return (int)(L - 1 - t_base < kT - 1 ? L - 1 - t_base : kT - 1); };
    // chunk q of a super-step: (array, token, position in the row); `first`: 0, or kBcHeld for the second half of float32
    auto fetch_bc = [&](int64_t t_base, int first) {
#pragma unroll
        for (int it = 0; it < kBcHeld; ++it) {
            const int q = tid + (first + it) * kThreadsL;
            if (kChunks % kThreadsL == 0 || q < kChunks) {
                const int arr = q / (kT * kChunksPerRow), r = q % (kT * kChunksPerRow);
                bc_nxt[it].load((arr ? Cm : Bm) + (row0 + t_base) * kN + (uint32_t)(min(r / kChunksPerRow, last_of(t_base)) * kN + (r % kChunksPerRow) * (kN / kChunksPerRow)));
            }
        }
    };
    auto publish_bc = [&](int first) {
#pragma unroll
        for (int it = 0; it < kBcHeld; ++it) {
            const int q = tid + (first + it) * kThreadsL;
            if (kChunks % kThreadsL == 0 || q < kChunks) {
                const int arr = q / (kT * kChunksPerRow), r = q % (kT * kChunksPerRow);
                const int tok = r / kChunksPerRow, pos = r % kChunksPerRow;
                // (a token past the end re-reads the last row: its delta is zero, which alone keeps the state as it is)
                float4 *dst = arr ? lds_C : lds_B;
#pragma unroll
                for (int g = 0; g < kChunkGroups; ++g)
                    dst[(tok % kTau) * kBcTau + (pos * kChunkGroups + g) * kBcPart + tok / kTau] = bc_nxt[it].group(g);
            }
        }
    };
    auto fetch = [&](int64_t t_base, RowG<T, kG> &xr, RowG<T, kG> &dtr, RowG<T, kG> &zr) {
        const int64_t base = (row0 + t_base) * D + c0;
        const uint32_t o = (uint32_t)min(kTau * ti + tj, last_of(t_base)) * (uint32_t)D;
        xr.load(x + base + o);
        if constexpr (!LOW) dtr.load(dt + base + o);
        if constexpr (kAhead && HAS_Z) zr.load(z + base + o);
    };
    auto publish = [&](int64_t t_base, const RowG<T, kG> &xr, const RowG<T, kG> &dtr) {
        const bool valid = kTau * ti + tj <= last_of(t_base);
        float xv[kG], dv[kG];
        xr.unpack(xv);
        dtr.unpack(dv);
#pragma unroll
        for (int c = 0; c < kG; ++c) dv[c] += lds_par[0][c];
        if constexpr (SOFTPLUS) {
            if constexpr (kRuns) softplus_run(dv);
            else
#pragma unroll
                for (int c = 0; c < kG; ++c) dv[c] = softplus_f32(dv[c]);
        }
#pragma unroll
        for (int c = 0; c < kG; ++c) {
            const float d = valid ? dv[c] : 0.0f;    // a token past the end leaves the state as it is
            reinterpret_cast<float *>(&lds_d[c][tj / kQ][ti])[tj % kQ] = d;
            reinterpret_cast<float *>(&lds_u[c][tj / kQ][ti])[tj % kQ] = d * xv[c];
        }
    };
    auto gate = [&](int64_t t_base, OutG<T, kG> &o6) {   // the outputs of the super-step
        float xv[kG], zv[kG], ov[kG];
        x_cur.unpack(xv);
        if constexpr (HAS_Z && !kAhead) {
            z_cur.load(z + (row0 + t_base) * D + c0 + (uint32_t)min(kTau * ti + tj, last_of(t_base)) * (uint32_t)D);
        }
        if constexpr (HAS_Z) z_cur.unpack(zv);
#pragma unroll
        for (int c = 0; c < kG; ++c) {
            // the four state groups in a fixed order: the result does not depend on which wavefront was first
            auto part_y = [&](int p) { return reinterpret_cast<const float *>(&lds_y[p][c][tj / kQ][ti])[tj % kQ]; };
            const float ch = (part_y(0) + part_y(1)) + (part_y(2) + part_y(3));
            const float y = fmaf(lds_par[1][c], xv[c], ch);
            ov[c] = HAS_Z ? y * silu_f32(zv[c]) : y;
        }
        o6.pack(ov);
    };
    auto store = [&](T *rows, int64_t t_base, const OutG<T, kG> &o6) {
        if (kTau * ti + tj > last_of(t_base)) return;
        T *p = rows + (row0 + t_base) * D + c0 + (uint32_t)(kTau * ti + tj) * (uint32_t)D;
        if (dead == 0) {
            o6.store(p);
        } else {
#pragma unroll
            for (int c = 0; c < kG; c += 2)
                if (c >= dead) o6.store_pair(p, c / 2);
        }
    };

    const int64_t n_super = LOW ? 1 : (L + kT - 1) / kT;
    // (the first rows land where they stay: passed on through the registers of the next ones, the copy would wait for them here,
    // before B and C are requested)
    RowG<T, kG> dt_first;
    if (token_thread) fetch(0, x_cur, dt_first, z_cur);
    if constexpr (LOW) {
        // dt = dt_low W_dt^T on the matrix cores: a wavefront's 64 tokens as two blocks of 32 columns, the workgroup's channels as the
        // first rows, 16 k at a time; rounded as the stored tensor is.  y[q][j] is token 32 q + lane % 32, channel 4 (lane / 32) + j.
        typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
        typedef float f32x16 __attribute__((ext_vector_type(16)));
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        if (token_thread) {
            u32x4 wf[kLanesLowRank / 16], xf[2][kLanesLowRank / 16];
            const int up = lane >> 5, ch = (lane & 31) < kG ? lane & 31 : kG - 1;
#pragma unroll
            for (int ks = 0; ks < kLanesLowRank / 16; ++ks) {
                const int k = min(16 * ks + 8 * up, low.rank - 8);
                wf[ks] = *reinterpret_cast<const u32x4 *>(low.w + (c0 + ch) * low.rank + k);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    xf[q][ks] = *reinterpret_cast<const u32x4 *>(dt + (row0 + min((tid & ~63) + 32 * q + (lane & 31), last_of(0))) * low.rank + k);
            }
            fetch_bc(0, 0);
            f32x16 y[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int i = 0; i < 16; ++i) y[q][i] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < kLanesLowRank / 16; ++ks) {
                    const bool in = 16 * ks + 8 * up < low.rank;   // (both operands: what stands in for the missing k may be infinite)
                    const u32x4 wv = in ? wf[ks] : u32x4(0u), xv = in ? xf[q][ks] : u32x4(0u);
                    y[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wv), __builtin_bit_cast(bf16x8, xv), y[q], 0, 0, 0);
                }
            }
            // a lane has the first four channels of one token and the others of another: what is not its own goes to the lane 32 away
            float dv[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float other = __shfl_xor(up ? y[0][j] : y[1][j], 32);
                dv[j] = up ? other : y[0][j];
                dv[4 + j] = up ? y[1][j] : other;
            }
            OutG<T, kG> stored;
            stored.pack(dv);
#pragma unroll
            for (int c = 0; c < kG / 2; ++c) dt_first.v[c] = stored.v[c];
            store(low.out, 0, stored);
        } else {
            fetch_bc(0, 0);
        }
    } else {
        fetch_bc(0, 0);
    }
    if (tid < 2 * kG) (&lds_par[0][0])[tid] = par;
    lds_barrier_l();   // the channel parameters are in LDS
    if (token_thread) publish(0, x_cur, dt_first);
    publish_bc(0);
    if constexpr (kBcIters > kBcHeld) {
        fetch_bc(0, kBcHeld);
        publish_bc(kBcHeld);
    }
    lds_barrier_l();

    for (int64_t k = 0; k < n_super; ++k) {                       // L >= 1: at least one
        const int64_t t_base = k * kT;
        const bool more = !LOW && k + 1 < n_super;
        RowG<T, kG> x_nxt, dt_nxt, z_nxt;
        if (token_thread && more) fetch(t_base + kT, x_nxt, dt_nxt, z_nxt);

        // ---- 1. the lane's 8 tokens from zero (lane 0: from the state entering the super-step), decays kept
        // (delta and delta * x are taken from LDS four tokens at a time: fewer registers held at once)
        float a[kTau][2][4], h[2][4], P[2][4], dsum[2] = {0.0f, 0.0f};
#pragma unroll
        for (int ch = 0; ch < 2; ++ch)
#pragma unroll
            for (int n = 0; n < 4; ++n) h[ch][n] = lane == 0 ? hp[ch][n] : 0.0f;
#pragma unroll
        for (int jh = 0; jh < kTau / kQ; ++jh) {
            quad d4[2], u4[2];
#pragma unroll
            for (int ch = 0; ch < 2; ++ch) {
                d4[ch] = lds_d[ca + ch][jh][lane];
                u4[ch] = lds_u[ca + ch][jh][lane];
            }
#pragma unroll
            for (int jj = 0; jj < kQ; ++jj) {
                const int j = kQ * jh + jj;
                const float4 b4 = lds_B[j * kBcTau + part * kBcPart + lane];
                const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
                float e[8];
#pragma unroll
                for (int ch = 0; ch < 2; ++ch)
#pragma unroll
                    for (int n = 0; n < 4; ++n) e[4 * ch + n] = d4[ch][jj] * a2[ch][n];
                if constexpr (kRuns) exp2_run(e);
                else
#pragma unroll
                    for (int i = 0; i < 8; ++i) e[i] = exp2_hw(e[i]);
#pragma unroll
                for (int ch = 0; ch < 2; ++ch) {
                    const float d = d4[ch][jj];
                    const float u = u4[ch][jj];
                    dsum[ch] += d;
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        a[j][ch][n] = e[4 * ch + n];
                        h[ch][n] = fmaf(a[j][ch][n], h[ch][n], u * bv[n]);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- 2. decay over the whole block
#pragma unroll
        for (int ch = 0; ch < 2; ++ch)
#pragma unroll
            for (int n = 0; n < 4; ++n) P[ch][n] = exp2_hw(dsum[ch] * a2[ch][n]);
        // ---- 3. inclusive scan over the 64 lanes, then every lane takes the state at the end of the block before it
        float hin[2][4];
        {
            float Hs[8], Ps[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                Hs[r] = h[r >> 2][r & 3];
                Ps[r] = P[r >> 2][r & 3];
            }
            lane_scan(Hs, Ps);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float rot = wave_rotate1(Hs[r]);
                hin[r >> 2][r & 3] = lane == 0 ? hp[r >> 2][r & 3] : rot;
                // lane 63's end state enters the next super-step
                hp[r >> 2][r & 3] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Hs[r]), 63));
            }
        }
        // the final state leaves as soon as it is known, not behind the last outputs (a wavefront's own, as its part of h0 was)
        if (!more && h_final && lane == 0 && ca >= dead) {
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    h_final[b * D * kN + (c0 + ca + ch) * kN + 4 * part + n] = hp[ch][n];
        }
        // The next super-step's B and C are requested here rather than with its rows at the top: their registers would
        // otherwise be held through the first walk, where the decays pile up; the second walk, the barrier and the gating
        // of this super-step's outputs are what their latency hides behind.
        if (more) {
            if constexpr (kAhead) fetch_bc(t_base + kT, 0);
        }
        // ---- 4. the 8 tokens again from the true state, with outputs (delta * x is read again rather than kept)
#pragma unroll
        for (int jh = 0; jh < kTau / kQ; ++jh) {
            __builtin_amdgcn_sched_barrier(0);
            quad u4[2];
            quad yq[2];
#pragma unroll
            for (int ch = 0; ch < 2; ++ch) u4[ch] = lds_u[ca + ch][jh][lane];
#pragma unroll
            for (int jj = 0; jj < kQ; ++jj) {
                const int j = kQ * jh + jj;
                const float4 b4 = lds_B[j * kBcTau + part * kBcPart + lane], c4 = lds_C[j * kBcTau + part * kBcPart + lane];
                const float bv[4] = {b4.x, b4.y, b4.z, b4.w}, cv[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int ch = 0; ch < 2; ++ch) {
                    const float u = u4[ch][jj];
                    float yp = 0.0f;
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        hin[ch][n] = fmaf(a[j][ch][n], hin[ch][n], u * bv[n]);
                        yp = fmaf(hin[ch][n], cv[n], yp);
                    }
                    yq[ch][jj] = yp;
                }
            }
#pragma unroll
            for (int ch = 0; ch < 2; ++ch) lds_y[part][ca + ch][jh][lane] = yq[ch];
        }
        lds_barrier_l();   // y of the super-step is complete; its operands are used up

        if constexpr (!kAhead) {
            if (more) fetch_bc(t_base + kT, 0);
        }
        OutG<T, kG> o6;
        // The outputs are stored last: loads and stores are waited for by one counter, so a wait for the next rows that came
        // after the stores would also wait for the stores, with everyone else at the barrier.
        if (token_thread) {
            gate(t_base, o6);
            if constexpr (!kAhead) store(out, t_base, o6);   // (float32 has no registers to hold them in)
            if (more) {
                publish(t_base + kT, x_nxt, dt_nxt);
                x_cur = x_nxt;
                if constexpr (HAS_Z && kAhead) z_cur = z_nxt;
            }
        }
        if (more) {
            publish_bc(0);
            if constexpr (kBcIters > kBcHeld) {
                fetch_bc(t_base + kT, kBcHeld);
                publish_bc(kBcHeld);
            }
        }
        if constexpr (kAhead) {
            if (token_thread) store(out, t_base, o6);
        }
        lds_barrier_l();   // the next super-step is in LDS
    }
}

}  // namespace

namespace {

template <typename T, int G, int TAU> hipError_t launch_lanes(const ScanArgs &a, hipStream_t stream)
{
    const int64_t n_groups = (a.D + G - 1) / G;
    const dim3 grid((unsigned)(8 * ((n_groups + 7) / 8)), (unsigned)a.batch);   // padded for the XCD-aware numbering
#define MAMBA_LAUNCH_LANES(HZ, SP, LOW, LOWDT)                                                              \
    scan_lanes_kernel<T, HZ, SP, G, TAU, LOW><<<grid, 64 * kParts * (G / 2), 0, stream>>>(                  \
        static_cast<const T *>(a.x), static_cast<const T *>(a.dt), a.A, static_cast<const T *>(a.Bm),       \
        static_cast<const T *>(a.Cm), a.Dskip, static_cast<const T *>(a.z), a.dt_bias, a.h0,                \
        static_cast<T *>(a.out), a.h_final, a.L, a.D, LOWDT)
    if constexpr (sizeof(T) == 2) {
        if (a.dt_w) {
            const LowDt low{static_cast<const bf16_t *>(a.dt_w), static_cast<bf16_t *>(a.dt_out), (int)a.dt_rank};
            MAMBA_LAUNCH_LANES(true, true, true, low);
            return hipGetLastError();
        }
    }
    if (a.z) {
        if (a.dt_softplus) MAMBA_LAUNCH_LANES(true, true, false, LowDt{});
        else MAMBA_LAUNCH_LANES(true, false, false, LowDt{});
    } else {
        if (a.dt_softplus) MAMBA_LAUNCH_LANES(false, true, false, LowDt{});
        else MAMBA_LAUNCH_LANES(false, false, false, LowDt{});
    }
#undef MAMBA_LAUNCH_LANES
    return hipGetLastError();
}

template <typename T> hipError_t launch_lanes_io(const ScanArgs &a, hipStream_t stream)
{
    switch (10 * lanes_channels(a.batch, a.L, a.D) + lanes_tau(a.batch, a.L, a.D, a.io == kIoBf16)) {
    case 24: return launch_lanes<T, 2, 4>(a, stream);
    case 44: return launch_lanes<T, 4, 4>(a, stream);
    case 46: return launch_lanes<T, 4, 6>(a, stream);
    case 48: return launch_lanes<T, 4, 8>(a, stream);
    case 64: return launch_lanes<T, 6, 4>(a, stream);
    case 66: return launch_lanes<T, 6, 6>(a, stream);
    default: return launch_lanes<T, 6, 8>(a, stream);
    }
}

}  // namespace

hipError_t launch_scan_lanes(const ScanArgs &a, hipStream_t stream)
{
    return a.io == kIoBf16 ? launch_lanes_io<bf16_t>(a, stream) : launch_lanes_io<float>(a, stream);
}

}  // namespace mamba
