// Causal depthwise conv1d over time with optional SiLU (first stage of the selective-SSM layer,
// run over the context when the drafter encodes it and over one token per branch while it
// drafts), gfx950.
//
//   y[b,t,d] = act(bias[d] + sum_k w[d,k] xpad[b,t+k,d]),  xpad = [carried K-1 rows or zeros ; x]
//   conv_state_out[b,d,:] = last K-1 rows of xpad
//
// HBM-bound: 2 elements moved per output.  A lane owns VEC adjacent channels (16 bytes of a token
// row), walks a tile of consecutive tokens and keeps the K-1 previous rows in registers, so every
// input element is read once (plus K-1 halo rows per tile) and every wavefront access is a
// contiguous run.  Loads of the next group of rows are issued before the current group is used.  Groups are short:
// what is in flight is bounded by wavefronts, and those by registers.  Against tiles of 8 to 32 rows per single wavefront
// with taps of its own (bf16, operands from memory): 64 x 1536 4.3 -> 3.4 us, 2048 x 1536 6.7 -> 5.8, 8000 x 1536 14.9 -> 12.0,
// 32768 x 1536 46.7 -> 42 us (201 MB, 4.8 TB/s), 15 x 5525 x 544 60 -> 50 us.  What gains nothing from it keeps the single
// wavefronts (launch_conv_k).
// In tree drafting (Sec. 4.1) a branch starts from the window of its parent: the carried rows can be
// read through a parent index, which replaces a separate copy of the window.
#include "conv_lane.h"
#include "device_math.h"
#include "launch.h"

namespace mamba {
namespace {

constexpr int kWave = 64;
constexpr int kTilesPerBlock = 4;   // wavefronts of a workgroup: consecutive time tiles of the same channels
constexpr int kBlock = kWave * kTilesPerBlock;
constexpr int kRows = 2;       // rows loaded together, one group ahead
constexpr int kRowsWave = 8;   // the same of a wavefront on its own

// orders LDS only: the rows requested ahead of it stay in flight
__device__ __forceinline__ void lds_barrier_c()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// grid: (channel-vector groups, groups of four time tiles, batch), blocks of 64 x 4 threads (a grid has fewer than 2^32 threads
// along x, so the wavefronts of a workgroup count along y)
template <typename T, int VEC, int K, bool SILU>
__global__ void __launch_bounds__(kBlock)
conv1d_kernel(const T *__restrict__ x, const float *__restrict__ w, const float *__restrict__ bias,
              const T *state_in, T *__restrict__ y, T *state_out, int64_t L, int64_t D,
              int64_t tile_len, int lanes, const int32_t *__restrict__ parent, int64_t n_in)
{
    typedef typename RowVec<T, VEC>::type row_t;
    constexpr int H = K - 1;
    const int64_t b = blockIdx.z;
    const int lane = threadIdx.x, wave = threadIdx.y, tid = wave * kWave + lane;
    const int64_t d_block = (int64_t)blockIdx.x * (lanes * VEC);    // first channel of the workgroup
    const int64_t d0 = d_block + lane * VEC;
    const bool live = lane < lanes && d0 < D;
    const int64_t t0 = ((int64_t)blockIdx.y * kTilesPerBlock + wave) * tile_len;
    const int64_t t1 = (t0 + tile_len < L) ? t0 + tile_len : L;

    // Taps and bias of the 64 VEC channels, fetched once for the workgroup with adjacent lanes on adjacent 16 bytes.  (A
    // lane's own VEC K taps are one run of memory, but read by that lane every 16-byte piece lies 128 bytes from its
    // neighbour's, and the address path takes a cycle per lane: three times what the token rows themselves take.)
    constexpr int kSlots = VEC * K / 4;                             // float4 of taps per lane
    constexpr int kTapIters = (kWave * kSlots + kBlock - 1) / kBlock, kBiasIters = (kWave * VEC + kBlock - 1) / kBlock;
    __shared__ __attribute__((aligned(16))) float4 lds_w[kSlots][kWave + 1];   // + 1: eight slots of a lane fall on eight bank groups
    __shared__ __attribute__((aligned(16))) float lds_b[kWave * VEC];
    float4 tap[kTapIters];
    float bias_in[kBiasIters];
    const int64_t n_taps = (D - d_block) * K / 4;                   // D % VEC == 0: whole float4
#pragma unroll
    for (int i = 0; i < kTapIters; ++i) {
        const int q = tid + i * kBlock;
        tap[i] = reinterpret_cast<const float4 *>(w + d_block * K)[q < n_taps ? q : 0];
    }
#pragma unroll
    for (int i = 0; i < kBiasIters; ++i) {
        const int64_t d = d_block + tid + i * kBlock;
        bias_in[i] = bias ? bias[d < D ? d : D - 1] : 0.0f;
    }

    const T *xb = x + b * L * D + d0;
    T *yb = y + b * L * D + d0;
    auto ld_row = [&](int64_t t) { return *reinterpret_cast<const row_t *>(xb + t * D); };
    ConvLane<T, VEC, K, SILU> c;
    if (live && t0 < H && t0 < t1 + (L == 0)) c.load_carried(state_in, parent, b, n_in, D, d0);
    // (the rows before the tile and its first group of rows are on their way before anything is waited for)
    row_t before[H > 0 ? H : 1];
    row_t cur[kRows];
    // rows t .. t + kRows - 1, those past the tile's end replaced by its last one (never used)
    auto ld_group = [&](row_t (&r)[kRows], int64_t t) {
#pragma unroll
        for (int i = 0; i < kRows; ++i) r[i] = ld_row(t + i < t1 ? t + i : t1 - 1);
    };
    if (live && t0 < t1) {
#pragma unroll
        for (int i = 0; i < H; ++i) before[i] = ld_row(t0 - H + i < 0 ? 0 : t0 - H + i);
        ld_group(cur, t0);
    }
#pragma unroll
    for (int i = 0; i < kTapIters; ++i) {
        const int q = tid + i * kBlock;
        if (q < kWave * kSlots) lds_w[q % kSlots][q / kSlots] = tap[i];
    }
#pragma unroll
    for (int i = 0; i < kBiasIters; ++i)
        if (tid + i * kBlock < kWave * VEC) lds_b[tid + i * kBlock] = bias_in[i];
    lds_barrier_c();
#pragma unroll
    for (int i = 0; i < kSlots; ++i) unpack_row(lds_w[i][lane], &c.wr[0][0] + 4 * i);
#pragma unroll
    for (int i = 0; i < VEC / 4; ++i) unpack_row(*reinterpret_cast<const float4 *>(&lds_b[lane * VEC + 4 * i]), c.br + 4 * i);
    if (!live || t0 >= t1 + (t0 == 0 && L == 0)) return;        // (no token at all: one tile passes the carried state on)
#pragma unroll
    for (int i = 0; i < H; ++i) c.set_window(i, t0 - H + i, before[i]);

    auto emit = [&](int64_t t, row_t raw) { *reinterpret_cast<row_t *>(yb + t * D) = c.emit(raw); };
    for (int64_t t = t0; t < t1; t += kRows) {
        row_t nxt[kRows];
        const bool more = t + kRows < t1;
        if (more) ld_group(nxt, t + kRows);
        if (t + kRows <= t1) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) emit(t + i, cur[i]);
        } else {
#pragma unroll
            for (int i = 0; i < kRows - 1; ++i)
                if (t + i < t1) emit(t + i, cur[i]);
        }
        if (more) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) cur[i] = nxt[i];
        }
    }
    if (state_out && t1 == L) c.store_window(state_out, b, D, d0);
}

// The same with one wavefront to a workgroup, taps of its own and longer groups of rows: for what the kernel above has no use of
// its four wavefronts for, or of 16-byte pieces (launch_conv_k).
// grid: (channel-vector groups, time tiles, batch)
template <typename T, int VEC, int K, bool SILU>
__global__ void __launch_bounds__(kWave)
conv1d_wave_kernel(const T *__restrict__ x, const float *__restrict__ w, const float *__restrict__ bias,
                   const T *state_in, T *__restrict__ y, T *state_out, int64_t L, int64_t D,
                   int64_t tile_len, const int32_t *__restrict__ parent, int64_t n_in)
{
    typedef typename RowVec<T, VEC>::type row_t;
    constexpr int H = K - 1;
    const int64_t b = blockIdx.z;
    const int64_t d0 = ((int64_t)blockIdx.x * kWave + threadIdx.x) * VEC;
    if (d0 >= D) return;                                            // no cross-lane work below
    const int64_t t0 = (int64_t)blockIdx.y * tile_len;
    const int64_t t1 = (t0 + tile_len < L) ? t0 + tile_len : L;
    ConvLane<T, VEC, K, SILU> c;
    if constexpr (VEC > 1) {
        ld_block<VEC * K>(w + d0 * K, &c.wr[0][0]);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) c.wr[0][k] = w[d0 * K + k];
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) c.br[i] = bias ? bias[d0 + i] : 0.0f;

    const T *xb = x + b * L * D + d0;
    T *yb = y + b * L * D + d0;
    auto ld_row = [&](int64_t t) { return *reinterpret_cast<const row_t *>(xb + t * D); };
    if (t0 < H) c.load_carried(state_in, parent, b, n_in, D, d0);
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const int64_t t = t0 - H + i;
        row_t row{};
        if (t >= 0) row = ld_row(t);
        c.set_window(i, t, row);
    }
    auto emit = [&](int64_t t, row_t raw) { *reinterpret_cast<row_t *>(yb + t * D) = c.emit(raw); };
    int64_t t = t0;
    row_t cur[kRowsWave];
    if (t + kRowsWave <= t1) {
#pragma unroll
        for (int i = 0; i < kRowsWave; ++i) cur[i] = ld_row(t + i);
    }
    for (; t + kRowsWave <= t1; t += kRowsWave) {
        row_t nxt[kRowsWave];
        const bool more = t + 2 * kRowsWave <= t1;
        if (more) {
#pragma unroll
            for (int i = 0; i < kRowsWave; ++i) nxt[i] = ld_row(t + kRowsWave + i);
        }
#pragma unroll
        for (int i = 0; i < kRowsWave; ++i) emit(t + i, cur[i]);
        if (more) {
#pragma unroll
            for (int i = 0; i < kRowsWave; ++i) cur[i] = nxt[i];
        }
    }
    for (; t < t1; ++t) emit(t, ld_row(t));
    if (state_out && t1 == L) c.store_window(state_out, b, D, d0);
}

template <typename T, int VEC, int K> hipError_t launch_conv_k(const ConvArgs &a, hipStream_t stream)
{
    const int64_t vecs = (a.D + VEC - 1) / VEC;
    const unsigned gx = (unsigned)((vecs + kWave - 1) / kWave);
    // Whose kernel: time tiles side by side in a workgroup, or single wavefronts.  The first needs several tiles and 16-byte
    // pieces; us on tiles / single wavefronts:
    //   a state updated in place, which is one tile: 2048 x 1536 bf16 622 / 437, f32 378 / 260; 64 x 8 x 1536 5.8 / 4.7
    //   one or two tokens: 64 x 1 x 1536 bf16 4.0 / 3.4, f32 3.8 / 3.4, 128 x 2 x 768 4.2 / 3.8 (64 x 4 x 1536 4.2 / 4.4)
    //   one channel to a lane: 4000 x 777 bf16 8.0 / 6.8, f32 8.1 / 7.3; 32768 x 777 34.9 / 32.8, 50.0 / 46.9
    //   few float32 lanes on many rows: 16384 x 64 5.4 / 5.1, 32768 x 64 7.7 / 7.2 (12000 x 64 4.6 / 5.1, 16384 x 256 6.7 / 7.5)
    // Everywhere else the tiles are as fast or faster (8000 x 1536 bf16 11.4 / 14.7, f32 16.8 / 17.6).
    const bool in_place = a.state_out && a.state_in == a.state_out;
    const bool waves = VEC == 1 || in_place || a.L <= 2 || (sizeof(T) == 4 && vecs <= 32 && a.batch * a.L >= 16384);
    const int rows = waves ? kRowsWave : kRows;
    // Time tiles: enough workgroups to fill the chip, long enough to amortize the K-1 halo rows.
    // An in-place state update keeps one tile so that a thread reads the state before it writes it.
    // Short inputs get shorter tiles (down to one group of rows) until there are about two wavefronts per SIMD: a row
    // takes a wavefront some 500 cycles of arithmetic, so on a short input the rows in turn are most of the time.
    // Rows of 2 or 4 KB take tiles of 18 rows: with 16 all tiles of a round start on the same memory channels (f32, 8192 x
    // 1024 14.1 -> 12.5 us, 16384 x 512 13.2 -> 12.3; bf16, 8192 x 2048 15.5 -> 14.5; rows of 3, 6 and 8 KB are faster with 16).
    const int64_t row_bytes = a.D * (int64_t)sizeof(T);
    int64_t tile_len = waves ? 32 : row_bytes == 2048 || row_bytes == 4096 ? 18 : 16;
    while (tile_len > rows && (int64_t)gx * ((a.L + tile_len - 1) / tile_len) * a.batch < 2048) tile_len /= 2;
    if (in_place) tile_len = a.L;
    if ((a.L + tile_len - 1) / tile_len > 65535) tile_len = (a.L + 65534) / 65535;
    if (tile_len < 1) tile_len = 1;
    int64_t tiles = (a.L + tile_len - 1) / tile_len;
    if (tiles < 1) tiles = 1;  // L == 0: one tile that only passes the carried state on
    const T *x = static_cast<const T *>(a.x);
    const T *si = static_cast<const T *>(a.state_in);
    T *y = static_cast<T *>(a.y);
    T *so = static_cast<T *>(a.state_out);
    if (waves) {
        const dim3 grid(gx, (unsigned)tiles, (unsigned)a.batch);
        if (a.apply_silu)
            conv1d_wave_kernel<T, VEC, K, true><<<grid, kWave, 0, stream>>>(x, a.w, a.bias, si, y, so, a.L, a.D, tile_len, a.parent, a.n_in);
        else
            conv1d_wave_kernel<T, VEC, K, false><<<grid, kWave, 0, stream>>>(x, a.w, a.bias, si, y, so, a.L, a.D, tile_len, a.parent, a.n_in);
        return hipGetLastError();
    }
    if constexpr (VEC > 1) {
        // channel vectors per wavefront: an even split, not a remainder for the last one, in whole 128-byte lines
        const int lanes = (int)((vecs + gx - 1) / gx + 7) / 8 * 8;
        const dim3 grid(gx, (unsigned)((tiles + kTilesPerBlock - 1) / kTilesPerBlock), (unsigned)a.batch), block(kWave, kTilesPerBlock);
        if (a.apply_silu)
            conv1d_kernel<T, VEC, K, true><<<grid, block, 0, stream>>>(x, a.w, a.bias, si, y, so, a.L, a.D, tile_len, lanes, a.parent, a.n_in);
        else
            conv1d_kernel<T, VEC, K, false><<<grid, block, 0, stream>>>(x, a.w, a.bias, si, y, so, a.L, a.D, tile_len, lanes, a.parent, a.n_in);
    }
    return hipGetLastError();
}

template <typename T, int VEC> hipError_t launch_conv_v(const ConvArgs &a, hipStream_t stream)
{
    switch (a.K) {
    case 2: return launch_conv_k<T, VEC, 2>(a, stream);
    case 3: return launch_conv_k<T, VEC, 3>(a, stream);
    case 4: return launch_conv_k<T, VEC, 4>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_conv1d(const ConvArgs &a, hipStream_t stream)
{
    // 16-byte channel vectors need every token row to start on a 16-byte boundary
    if (a.io == kIoBf16) {
        if (a.D % 8 == 0) return launch_conv_v<bf16_t, 8>(a, stream);
        return launch_conv_v<bf16_t, 1>(a, stream);
    }
    if (a.D % 4 == 0) return launch_conv_v<float, 4>(a, stream);
    return launch_conv_v<float, 1>(a, stream);
}

}  // namespace mamba
