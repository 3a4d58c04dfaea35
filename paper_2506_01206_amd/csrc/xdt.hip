// x projection and dt projection of a context in one pass (the two narrow products between the conv and the scan of a
// Mamba block), gfx950 matrix cores:
//
//   [dt_low | B | C][m, :] = x_c[m, :] W_x^T,   dt[m, :] = dt_low[m, :] W_dt^T      (bf16, float32 sums)
//
// The first product reads all of x_c for 80 columns, the second writes a tensor as large from 48 of them: as two launches each
// has a load (or store) phase of its own and the narrow result goes through memory in between.  Here a workgroup keeps 16 MT
// token rows: its eight wavefronts share the k range of the first product in contiguous pieces, every row of x_c and of W_x
// fetched in whole 128-byte lines and turned into fragments in a wavefront's own LDS patch; the partial tiles
// meet in LDS, the sums are rounded to bf16 (what the stored tensor holds is what the second product reads), and the
// wavefronts share the columns of dt, 64 at a time, W_dt fetched as the contiguous run of memory that 64 of its rows are.
// Every workgroup reads all the weights from L2 (392 KB at 1536 channels); the first W_dt rows are on their way while the
// partial sums meet.  What a workgroup takes is that: 10 to 12 us with 16 rows, 12 to 15 with 32, 16 to 19 with 64 (1536
// channels, 48 dt columns; rows in 64-byte pieces, twice as many pieces for the address path, cost 1.5 us more).
// Against the two launches: 8000 rows 27 -> 15.4 us, 32768 rows 76 -> 46.7 us; 24-block prefill of 1024 tokens 1494 -> 1466
// us, of 2000 2037 -> 2001, of 4096 3218 -> 3165, of 8000 5376 -> 5130, of 12000 7860 -> 7585.
#include "device_math.h"
#include "launch.h"
#include "routes.h"

namespace mamba {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kNW = 8, kThr = 64 * kNW;
constexpr int kStates = kXdtStates;

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void lds_barrier_x()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// KS: dt_rank / 16; 16 states.  K (= d_inner) a multiple of 64.  grid: (ceil(M / (16 MT)), column groups): every column
// group forms the first product again and takes the 64-column blocks kNW * y + piece, + kNW * gridDim.y, ... of dt.
template <int KS, int MT>
__global__ void __launch_bounds__(kThr)
xdt_kernel(const bf16_t *__restrict__ xc, const bf16_t *__restrict__ wx, const bf16_t *__restrict__ wdt, bf16_t *__restrict__ dtl,
           bf16_t *__restrict__ bm, bf16_t *__restrict__ cm, bf16_t *__restrict__ dt, int64_t M, int K)
{
    constexpr int R = 16 * KS, NT = KS + 2 * kStates / 16;         // 16-column tiles of the first product
    constexpr int G = MT > 2 ? 2 : 3;                              // k64 steps in flight per wavefront
    constexpr int kWave = (MT + NT) * 2048;                        // fragments of one k64 step: a wavefront's patch of LDS
    constexpr int kWRow = 2 * R + 16, kORow = 64 * 2 + 16;         // LDS rows of a W_dt block and of a dt block
    constexpr int MH = MT > 2 ? 2 : MT;                            // row tiles whose partial sums meet at a time
    constexpr int kPart = MH * NT * 1024;                          // a wavefront's partial tiles
    constexpr int kLds = kNW * (kWave > kPart ? kWave : kPart);
    constexpr int kLRow = 2 * R + 16, kLRows = MT > 2 ? 16 * MT : 32;
    constexpr int NL = 2 * KS;                                     // 1 KiB loads per W_dt block (64 rows)
    static_assert(64 * kWRow + 32 * kORow <= kWave, "a wavefront's second-phase patches fit its first-phase ones");
    static_assert(kLds + kLRows * kLRow <= 160 * 1024, "LDS of a CU");
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
    __shared__ __attribute__((aligned(16))) unsigned char low[kLRows * kLRow];   // dt_low of the rows (MT == 1: the upper half is never stored)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;                      // fragment view: row, 16-byte chunk of a k32 half
    const int lrow = lane >> 3, lch = lane & 7;                    // load view: row (+ 8 i), 16-byte slot
    const int put = (lrow * 8 + (lch ^ lrow)) * 16;                // + 1024 i: slots xor-swizzled by the row, no bank conflicts either way
    const int get0 = (li * 8 + (lg ^ (li & 7))) * 16, get1 = (li * 8 + ((lg + 4) ^ (li & 7))) * 16;
    const int64_t m0 = (int64_t)blockIdx.x * (16 * MT);
    unsigned char *patch = lds + wave * kWave;

    // ---- first product
    const int steps = K >> 6, per = (steps + kNW - 1) / kNW;
    // (the workgroups of an XCD start at different pieces of k, so that they do not all ask its L2 for the same lines at once)
    const int piece = (wave + (int)(blockIdx.x >> 3)) & (kNW - 1);
    const int s_first = piece * per, s_end = s_first + per < steps ? s_first + per : steps;
    const u32x4 *wrow = reinterpret_cast<const u32x4 *>(wx + (int64_t)lrow * K);   // 8 rows further: + K pieces
    const u32x4 *xrow[2 * MT];
#pragma unroll
    for (int t = 0; t < 2 * MT; ++t) {
        const int64_t m = m0 + 8 * t + lrow;
        xrow[t] = reinterpret_cast<const u32x4 *>(xc + (m < M ? m : M - 1) * K);   // rows past M repeat the last one, never stored
    }
    f32x4v acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] = f32x4v(0.0f);
    for (int s0 = s_first; s0 < s_end; s0 += G) {
        u32x4 xf[G][2 * MT], wf[G][2 * NT];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int c = 8 * (s0 + g < s_end ? s0 + g : s_first) + lch;
#pragma unroll
            for (int t = 0; t < 2 * MT; ++t) xf[g][t] = xrow[t][c];
#pragma unroll
            for (int n = 0; n < 2 * NT; ++n) wf[g][n] = wrow[(int64_t)n * K + c];
        }
        __builtin_amdgcn_sched_barrier(0);                         // all of it in flight before any of it is used
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (s0 + g < s_end) {                                  // uniform
#pragma unroll
                for (int t = 0; t < 2 * MT; ++t) *reinterpret_cast<u32x4 *>(patch + t * 1024 + put) = xf[g][t];
#pragma unroll
                for (int n = 0; n < 2 * NT; ++n) *reinterpret_cast<u32x4 *>(patch + (2 * MT + n) * 1024 + put) = wf[g][n];
                wave_sync();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int get = h ? get1 : get0;
                    bf16x8 xv[MT];
#pragma unroll
                    for (int t = 0; t < MT; ++t) xv[t] = *reinterpret_cast<const bf16x8 *>(patch + t * 2048 + get);
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const bf16x8 wv = *reinterpret_cast<const bf16x8 *>(patch + (MT + n) * 2048 + get);
#pragma unroll
                        for (int t = 0; t < MT; ++t) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[t], wv, acc[t][n], 0, 0, 0);
                    }
                }
                wave_sync();
            }
        }
    }

    // ---- the first W_dt block of this wavefront is requested before the sums meet
    const int blocks = K >> 6, stride = kNW * (int)gridDim.y;
    int blk = (int)blockIdx.y * kNW + piece;
    u32x4 wq[NL];
    auto fetch_w = [&](int b) {
        const u32x4 *p = reinterpret_cast<const u32x4 *>(wdt + (int64_t)(b < blocks ? b : 0) * 64 * R) + lane;
#pragma unroll
        for (int q = 0; q < NL; ++q) wq[q] = p[q * 64];
    };
    fetch_w(blk);

    // acc[t][n][i] is C[m = 16 t + 4 (lane / 16) + i][16 n + lane % 16]
    float (*part)[MH * NT][4][64] = reinterpret_cast<float (*)[MH * NT][4][64]>(lds);
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += MH) {
        lds_barrier_x();                                           // the patches (or the last sums) are done with: their memory is reused
#pragma unroll
        for (int t = 0; t < MH; ++t)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) part[piece][t * NT + n][i][lane] = acc[t0 + t][n][i];
        lds_barrier_x();
#pragma unroll
        for (int o = tid; o < MH * NT * 256; o += kThr) {
            const int tile = o >> 8, i = (o >> 6) & 3;             // of lane `lane`
            float v = 0.0f;
#pragma unroll
            for (int q = 0; q < kNW; ++q) v += part[q][tile][i][lane];
            const int t = tile / NT, n = tile - t * NT;            // uniform over a wavefront
            const int ml = 16 * (t0 + t) + 4 * lg + i;
            const int64_t m = m0 + ml;
            const uint16_t s = (uint16_t)f32_to_bf16(v);
            const bool keep = blockIdx.y == 0 && m < M;
            if (n < KS) {
                *reinterpret_cast<uint16_t *>(low + ml * kLRow + (16 * n + li) * 2) = s;
                if (keep) dtl[m * R + 16 * n + li] = s;
            } else if (keep) {
                (n == KS ? bm : cm)[m * kStates + li] = s;
            }
        }
    }
    lds_barrier_x();

    // ---- dt: 64 columns at a time, formed transposed so that a lane's four accumulators are adjacent columns of one row
    const int r = lane & 31, up = lane >> 5;
    constexpr int MB = kLRows / 32;
    bf16x8 lowf[MB][KS];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) lowf[mb][ks] = *reinterpret_cast<const bf16x8 *>(low + (32 * mb + r) * kLRow + ks * 32 + up * 16);
    unsigned char *wpatch = patch, *opatch = patch + 64 * kWRow;
    for (; blk < blocks; blk += stride) {
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int e = q * 64 + lane;                           // 16-byte piece of the block: row e / NL, piece e % NL
            *reinterpret_cast<u32x4 *>(wpatch + (e / NL) * kWRow + (e % NL) * 16) = wq[q];
        }
        fetch_w(blk + stride);
        wave_sync();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                f32x16 y;
#pragma unroll
                for (int i = 0; i < 16; ++i) y[i] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(wpatch + (32 * b + r) * kWRow + ks * 32 + up * 16),
                                                                lowf[mb][ks], y, 0, 0, 0);
                // y[4 g + j] is dt[m = 32 mb + lane % 32][64 blk + 32 b + 8 g + 4 (lane / 32) + j]
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<uint2 *>(opatch + r * kORow + (32 * b + 8 * g + 4 * up) * 2) =
                        make_uint2(f32x2_to_bf16x2(y[4 * g], y[4 * g + 1]), f32x2_to_bf16x2(y[4 * g + 2], y[4 * g + 3]));
            }
            wave_sync();
#pragma unroll
            for (int i = 0; i < (MT == 1 ? 2 : 4); ++i) {
                const int row = 8 * i + (lane >> 3);
                const int64_t m = m0 + 32 * mb + row;
                const u32x4 v = *reinterpret_cast<const u32x4 *>(opatch + row * kORow + (lane & 7) * 16);
                if (m < M) *reinterpret_cast<u32x4 *>(dt + m * K + blk * 64 + (lane & 7) * 8) = v;
            }
            wave_sync();
        }
    }
}

}  // namespace

hipError_t launch_xdt(const XdtArgs &a, hipStream_t stream)
{
    unsigned groups;
    const int rows = xdt_plan(a.M, a.d_inner, a.dt_rank, kStates, &groups);
    const unsigned blocks = rows ? (unsigned)((a.M + rows - 1) / rows) : 0u;
#define MAMBA_XDT(KS, MT)                                                                                                          \
    xdt_kernel<KS, MT><<<dim3(blocks, groups), kThr, 0, stream>>>(                                                                \
        static_cast<const bf16_t *>(a.xc), static_cast<const bf16_t *>(a.wx), static_cast<const bf16_t *>(a.wdt),                 \
        static_cast<bf16_t *>(a.dtl), static_cast<bf16_t *>(a.bm), static_cast<bf16_t *>(a.cm), static_cast<bf16_t *>(a.dt), a.M, \
        (int)a.d_inner)
    switch (a.dt_rank * 128 + rows) {
    case 32 * 128 + 16: MAMBA_XDT(2, 1); break;
    case 32 * 128 + 32: MAMBA_XDT(2, 2); break;
    case 32 * 128 + 64: MAMBA_XDT(2, 4); break;
    case 48 * 128 + 16: MAMBA_XDT(3, 1); break;
    case 48 * 128 + 32: MAMBA_XDT(3, 2); break;
    case 48 * 128 + 64: MAMBA_XDT(3, 4); break;
    case 64 * 128 + 16: MAMBA_XDT(4, 1); break;
    case 64 * 128 + 32: MAMBA_XDT(4, 2); break;
    default: return hipErrorInvalidValue;
    }
#undef MAMBA_XDT
    return hipGetLastError();
}

}  // namespace mamba
