// Dense projections of the Mamba block (in_proj, x_proj, dt_proj, out_proj of the Mamba-130M
// drafter the paper uses, Sec. 3.1) on the gfx950 matrix cores.
//
//   out[m, n] = sum_k x[m, k] * w[n, k]  (+ bias[n]) (+ residual[m, n])
//
// x: (M, K) bf16, w: (N, K) bf16 (one row per output feature, K contiguous in both operands, which
// is the order MFMA operands want), fp32 accumulation, bf16 output.  The N output columns may be
// split over up to three contiguous output tensors (in_proj -> x | z; x_proj -> dt_low | B | C), so
// that the consumers get the dense (tokens, features) tensors they expect without a copy.
//
// Tiling: a workgroup of 4 wavefronts (2 x 2) owns a BM x BN output tile (128 x 128, or 64 x 128 or
// 64 x 64 when that is needed to give every CU a few workgroups); each wavefront a (BM/2) x (BN/2) part as
// MFMA tiles of v_mfma_f32_32x32x16_bf16.  K is walked in slabs of BK = 64: the x and w slabs are
// fetched with 16-byte loads one slab ahead into registers, parked in LDS (rows padded by 16 B)
// and read back as MFMA fragments with 16-byte LDS reads: lane l holds row l % 32,
// k = 8 * (l / 32) .. + 7 of each k16 step.  Three resident workgroups per CU hide the latencies.  (Larger
// tiles on this scheme, with its register staging and full barriers, measured slower; long contexts
// take the 256-row tiles of linear_wide_kernel below, which is built differently.)
// Rows past M or N re-read the last valid row and are never stored; a K tail is zero-filled.
// Epilogue: the accumulators (+ bias) are rounded to bf16 into LDS, then leave as 16-byte row
// chunks (+ residual), so that stores are coalesced; output splits that are not multiples of 8
// columns take an element-wise path.
#include <algorithm>
#include <type_traits>

#include "conv_lane.h"
#include "device_math.h"
#include "launch.h"
#include "routes.h"

namespace mamba {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

// barrier that orders LDS traffic only: global loads in flight stay in flight
__device__ __forceinline__ void lds_barrier_linear()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct OutSplit {
    bf16_t *ptr[3];
    int64_t width[3];
};

// column n of the virtual (M, N) output -> tensor and column inside it
__device__ __forceinline__ int locate(const OutSplit &o, int64_t n, int64_t *col)
{
    int64_t c = n;
    int s = 0;
    if (c >= o.width[0]) { c -= o.width[0]; s = 1; if (c >= o.width[1]) { c -= o.width[1]; s = 2; } }
    *col = c;
    return s;
}

// grid: (ceil(N / BN), ceil(M / BM)).  WSTREAM: w is read once and is large (the LM head on a draft position): its
// loads are streaming, so that they do not push the blocks' weights, which the next position reads again, out of
// the last-level cache.
template <int BM, int BN, int BK, bool WSTREAM = false>
__global__ void __launch_bounds__(kThreads)
linear_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w, const float *__restrict__ bias,
              const bf16_t *residual, OutSplit out, int64_t M, int64_t N, int64_t K, int vector_out)
{
    constexpr int MT = BM / 64, NT = BN / 64;                 // 32 x 32 MFMA tiles per wavefront along m, n
    constexpr int kBN = BN, kBK = BK;
    constexpr int kStageCols = BN < 128 ? BN : 128;           // the output tile is staged at most 128 columns at a time
    constexpr int kOutRowBytes = kStageCols * 2 + 16;
    constexpr int kRowBytes = BK * 2 + 16;                    // data + 16 B pad against bank conflicts
    constexpr int kOperandBytes = (BM + kBN) * kRowBytes;
    constexpr int kStageBytes = BM * kOutRowBytes;
    constexpr int kLdsBytes = kOperandBytes > kStageBytes ? kOperandBytes : kStageBytes;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLdsBytes];
    unsigned char *lds_x = lds, *lds_w = lds + BM * kRowBytes;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * kBN;

    // global -> LDS staging: (BM + BN) rows x BK/8 chunks of 16 B, NCH chunks per thread
    constexpr int kCpr = BK / 8;                              // chunks per row
    constexpr int NCH = (BM + kBN) * kCpr / kThreads;
    const uint4 *src[NCH];
    int dst_off[NCH], chunk[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tid + i * kThreads;
        const int row = c / kCpr;                             // 0 .. BM + BN - 1: x rows first, then w rows
        chunk[i] = c % kCpr;
        if (row < BM) {
            int64_t r = m0 + row;
            r = r < M ? r : M - 1;
            src[i] = reinterpret_cast<const uint4 *>(x + r * K);
        } else {
            int64_t r = n0 + (row - BM);
            r = r < N ? r : N - 1;
            src[i] = reinterpret_cast<const uint4 *>(w + r * K);
        }
        dst_off[i] = row * kRowBytes + chunk[i] * 16;
    }
    const int64_t kchunks = K / 8;                            // K is a multiple of 8 (checked on the host)
    uint4 regs[NCH];
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int64_t ch = k0 / 8 + chunk[i];
            if (WSTREAM && i * kThreads >= BM * kCpr) {         // chunks of w rows (whole multiples of the block: BM * kCpr % kThreads == 0)
                const u32x4 t = ch < kchunks ? __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src[i] + ch)) : u32x4(0u);
                regs[i] = make_uint4(t.x, t.y, t.z, t.w);
            } else {
                regs[i] = ch < kchunks ? src[i][ch] : make_uint4(0, 0, 0, 0);
            }
        }
    };
    auto park = [&]() {
#pragma unroll
        for (int i = 0; i < NCH; ++i) *reinterpret_cast<uint4 *>(lds + dst_off[i]) = regs[i];
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    const int frag_row = lane & 31, frag_k = (lane >> 5) * 16;    // byte offset of the lane's 8 k values
    fetch(0);
    for (int64_t k0 = 0; k0 < K; k0 += kBK) {
        __syncthreads();                                          // everyone is done reading the last slab
        park();
        __syncthreads();
        if (k0 + kBK < K) fetch(k0 + kBK);                        // in flight while this slab is multiplied
#pragma unroll
        for (int ks = 0; ks < kBK / 16; ++ks) {
            bf16x8 af[MT], bfr[NT];
#pragma unroll
            for (int t = 0; t < MT; ++t)
                af[t] = *reinterpret_cast<const bf16x8 *>(lds_x + (wm * (BM / 2) + t * 32 + frag_row) * kRowBytes + ks * 32 + frag_k);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                bfr[t] = *reinterpret_cast<const bf16x8 *>(lds_w + (wn * (BN / 2) + t * 32 + frag_row) * kRowBytes + ks * 32 + frag_k);
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
        }
    }

    // epilogue.  acc[a][b][i] is C[8 * (i / 4) + 4 * (lane / 32) + i % 4][lane % 32] of its 32 x 32 tile.
    // The tile leaves through LDS 128 columns at a time.
#pragma unroll
    for (int half = 0; half < BN / kStageCols; ++half) {
        __syncthreads();                                          // LDS (operands or the last half) is free
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int tile_col = wn * (BN / 2) + b * 32;      // column of this MFMA tile in the BN-wide tile
                if (tile_col / kStageCols != half) continue;      // compile-time per (wn is uniform per wavefront)
                const int col = tile_col - half * kStageCols + (lane & 31);
                const int64_t n = n0 + half * kStageCols + col;
                const float bv = (bias && n < N) ? bias[n] : 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = wm * (BM / 2) + a * 32 + 8 * (i / 4) + 4 * (lane >> 5) + (i & 3);
                    *reinterpret_cast<uint16_t *>(lds + row * kOutRowBytes + col * 2) = (uint16_t)f32_to_bf16(acc[a][b][i] + bv);
                }
            }
        __syncthreads();
        const int64_t nh = n0 + half * kStageCols;
        if (vector_out) {
            // every output width is a multiple of 8 columns: 16-byte chunks never straddle two tensors
            constexpr int kChunks = BM * (kStageCols / 8);
#pragma unroll
            for (int c = tid; c < kChunks; c += kThreads) {
                const int row = c / (kStageCols / 8), cc = c % (kStageCols / 8);
                const int64_t m = m0 + row, n = nh + cc * 8;
                if (m >= M || n >= N) continue;
                uint4 v = *reinterpret_cast<const uint4 *>(lds + row * kOutRowBytes + cc * 16);
                int64_t col;
                const int s = locate(out, n, &col);
                const int64_t off = m * out.width[s] + col;
                if (residual) {
                    const uint4 r = *reinterpret_cast<const uint4 *>(residual + off);   // single output: same offset
                    v.x = f32x2_to_bf16x2(bf16_lo(v.x) + bf16_lo(r.x), bf16_hi(v.x) + bf16_hi(r.x));
                    v.y = f32x2_to_bf16x2(bf16_lo(v.y) + bf16_lo(r.y), bf16_hi(v.y) + bf16_hi(r.y));
                    v.z = f32x2_to_bf16x2(bf16_lo(v.z) + bf16_lo(r.z), bf16_hi(v.z) + bf16_hi(r.z));
                    v.w = f32x2_to_bf16x2(bf16_lo(v.w) + bf16_lo(r.w), bf16_hi(v.w) + bf16_hi(r.w));
                }
                *reinterpret_cast<uint4 *>(out.ptr[s] + off) = v;
            }
        } else {
            for (int e = tid; e < BM * kStageCols; e += kThreads) {
                const int row = e / kStageCols, cl = e % kStageCols;
                const int64_t m = m0 + row, n = nh + cl;
                if (m >= M || n >= N) continue;
                float v = bf16_to_f32(*reinterpret_cast<const uint16_t *>(lds + row * kOutRowBytes + cl * 2));
                int64_t col;
                const int s = locate(out, n, &col);
                const int64_t off = m * out.width[s] + col;
                if (residual) v += bf16_to_f32(residual[off]);
                out.ptr[s][off] = (bf16_t)f32_to_bf16(v);
            }
        }
    }
}


// ---------------------------------------------------------------------------------------------------
// The way into a block on a context: [x | z] = u W_in^T, x_c = silu(conv1d(x)).  The tile kernels below (CONV) have a finished tile of x
// in LDS, rounded as the stored tensor would be, and form x_c from it where they would store x, which never goes to memory.  What that
// takes is vector work of the epilogue (45 cycles an output of a lane), under another workgroup's products where two share a CU, and
// three rows more in a tile; what it saves is a launch that reads and writes all of x.  us, in_proj and conv / one launch, 24 blocks in
// turn: 333 x 1536 11.6 / 8.7, 2048 20.5 / 18.5, 8000 53.9 / 47.3, 32768 216 / 187 (linear_conv_tiles has the tiles).  Formed on the way into
// the x projection instead (xdt.hip), with no other workgroup to hide it: 8000 rows 28.3 -> 23.0, 32768 101 -> 92, but 333 11.1 -> 14.2.
struct ConvTail {
    const float *w, *bias;           // (width[0], kConvTaps), (width[0]) or null
    const bf16_t *state_in;          // (sequences, width[0], kConvTaps - 1) or null: zeros
    bf16_t *state_out;               // the same or null
    uint32_t L;                      // rows of a sequence
    int z_blocks;                    // row blocks of z (linear_wide_kernel)
};
constexpr int kConvHalo = kConvTaps - 1;

// Rows of row block r: m0 + dead .. m0 + BM - 1, of BM that are multiplied.  The last block moves back to end at M; with the conv the
// first rows of every block but the first are there for the windows of the others.
template <int BM, bool CONV> __device__ __forceinline__ void rows_of_block(int r, int64_t M, int64_t *m0, int *dead)
{
    const int64_t first = !CONV ? (int64_t)r * BM : r == 0 ? 0 : BM + (int64_t)(r - 1) * (BM - kConvHalo);
    const int64_t from = CONV && r > 0 ? first - kConvHalo : first;
    *m0 = from + BM <= M ? from : M - BM;
    *dead = (int)(first - *m0);
}

// x_c of a tile of x: rows kRow bytes apart in LDS, channels n0 .. n0 + BN - 1.  A thread takes eight adjacent channels of consecutive rows.
template <int BM, int BN, int THREADS, int kRow>
__device__ __forceinline__ void conv_rows(const unsigned char *tile, int64_t m0, int dead, int64_t n0, bf16_t *xc, int64_t D, const ConvTail &conv)
{
    constexpr int kCpr = BN / 8, kPer = BM * kCpr / THREADS, H = kConvHalo;
    static_assert(BM * kCpr % THREADS == 0 && THREADS % kCpr == 0, "whole runs of rows");
    const int cc = (int)threadIdx.x % kCpr, row0 = (int)threadIdx.x / kCpr * kPer;
    const int64_t d0 = n0 + cc * 8;
    ConvLane<bf16_t, 8, kConvTaps, true> c;
    ld_block<8 * kConvTaps>(conv.w + d0 * kConvTaps, &c.wr[0][0]);
    if (conv.bias) ld_block<8>(conv.bias + d0, c.br);
    else
#pragma unroll
        for (int i = 0; i < 8; ++i) c.br[i] = 0.0f;
    auto raw = [&](int row) __attribute__((always_inline)) { return *reinterpret_cast<const uint4 *>(tile + row * kRow + cc * 16); };
    bf16_t *o = xc + (m0 + row0) * D + d0;
    // A tile that lies inside a sequence needs no looking at t: none of its rows has a window that reaches back before one, none is the last.
    const uint32_t t_first = (uint32_t)(m0 + dead) % conv.L;
    if (t_first >= (uint32_t)H && (uint64_t)t_first + (uint32_t)(BM - dead) < conv.L) {
#pragma unroll
        for (int i = 0; i < H; ++i) c.set_window(i, 0, raw(row0 - H + i < 0 ? 0 : row0 - H + i));   // (rows before the tile: for dead ones)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint4 y = c.emit(raw(row0 + i));
            if (row0 + i >= dead) *reinterpret_cast<uint4 *>(o + i * D) = y;
        }
    } else {
        const uint32_t m = (uint32_t)(m0 + row0);
        uint32_t q = m / conv.L, t = m - q * conv.L;
        if (t < (uint32_t)H) c.load_carried(conv.state_in, nullptr, q, 0, D, d0);
#pragma unroll
        for (int i = 0; i < H; ++i) c.set_window(i, (int64_t)t - H + i, raw(row0 - H + i < 0 ? 0 : row0 - H + i));
#pragma unroll 1
        for (int i = 0; i < kPer; ++i) {
            if (i > 0 && t == 0) {
                c.load_carried(conv.state_in, nullptr, q, 0, D, d0);
#pragma unroll
                for (int k = 0; k < H; ++k) c.set_window(k, k - H, uint4{});
            }
            const uint4 y = c.emit(raw(row0 + i));
            if (row0 + i >= dead) {
                *reinterpret_cast<uint4 *>(o + i * D) = y;
                if (conv.state_out && t == conv.L - 1) c.store_window(conv.state_out, q, D, d0);
            }
            if (++t == conv.L) t = 0, ++q;
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Many rows (the projections of a long context).  A 128 x 128 tile asks the L1 for 512 bytes per k and
// multiplies 8 cycles per k on every SIMD, so the cache, which delivers 64 bytes a cycle, can feed the
// matrix cores half the time at best.  This kernel takes 256 x 256 tiles, one workgroup per CU and two
// wavefronts per SIMD, each with a 128 x 64 part in 128 accumulator registers: per k the same
// 8 cycles of cache traffic now feed 32 cycles of MFMA.  (As four wavefronts of 128 x 128, which read a third less LDS, a SIMD has nothing
// to multiply while its one wavefront waits at the slab's barrier or for fragments: us of four / eight wavefronts, 24 weights in turn, 4096 x
// 3072, K = 768 24.9 / 21.9, 16384 x 3072 83.8 / 77.4, 32768 x 3072 179 / 170, 8000 x 768, K = 1536 39.8 / 33.4, 8000 x 4096, K = 1024 68.3 / 64.9.)
// (With four wavefronts it also runs 128 x 128 and 192 x 128 tiles, two workgroups to a CU, for products too small to give every CU
// a 256-row tile, or that leave CUs without one: the feeding scheme below, not the tile size, is what those gain from.)
// (And 256 x 192 tiles, eight wavefronts of 64 x 96, where those leave fewer CUs idle in the last round: 32768 x 768, K = 1536 is two whole rounds
// instead of one and a half of 256 x 256, 79.6 -> 75.1 us; a round of them takes six sevenths of one of 256 x 256 for three quarters of the
// products.  With the conv, whose epilogue leaves a quarter of the threads idle there, they are slower than the others throughout: one block of
// 8000 x 1536 188 -> 200 us, of 32768 645 -> 674 with both products on them.)
//
// Operands go from memory straight into LDS (global_load_lds_dwordx4: lane l of a wavefront lands at
// M0 + 16 l, so one instruction fills eight 128-byte rows): no staging registers, and none of the LDS
// write instructions whose data path the counters showed full when the slabs were parked from registers.
// Rows lie 128 bytes apart without padding; the 16-byte slot c of row r sits at slot c ^ ((r >> 1) & 7), chosen
// on the memory side of the load, which makes the fragment reads (32 rows, one slot each) conflict-free.
// The instruction is issued from inline assembly so that the compiler's wait-count pass does not see an LDS
// write it cannot place (it would wait for every load in flight before each LDS read); the waits are explicit:
// vmcnt(0) and lgkmcnt(0) before the one barrier per slab.  Slabs of 64 k alternate between two stages.  The barrier of
// slab s comes when its last fragments have been read, a quarter before its end; slab s + 2 is requested
// right after it into the stage just freed and has a whole slab of multiplications to arrive.
// The product is formed transposed (w fragments as the row operand), so that a lane's four accumulators
// of a group are four adjacent output columns of one row and leave as one 8-byte write.
// Requires M >= BM, N % BN == 0, K % 128 == 0 and output widths that are multiples of 8.  The last row block of an M
// that is not a multiple of BM is moved back to end at M: it works on a full tile of rows that exist and stores only
// the rows the block before it does not have.
// grid: 8 * ceil(tiles / 8) workgroups; consecutive workgroups go to different XCDs, so tile numbers are
// dealt such that each XCD (each L2) works on a contiguous range of tiles, column tiles of one row block
// adjacent.
constexpr int kWideBK = 64, kWideRow = kWideBK * 2;

// 16 bytes per lane from base + lane_off into LDS at lds_addr + 16 * lane (lds_addr wave-uniform)
__device__ __forceinline__ void load_to_lds16(const char *base, uint32_t lane_off, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(lane_off), "s"(base) : "memory");
}

template <int BM, int BN, bool CONV = false, int WM = 2, int WN = 2>
__global__ void __launch_bounds__(64 * WM * WN)
linear_wide_kernel(const bf16_t *x, const bf16_t *w, const float *__restrict__ bias, const bf16_t *residual,
                   OutSplit out, int64_t M, int64_t N, int64_t K, int tiles_n, int n_tiles, ConvTail conv)
{
    constexpr int NW = WM * WN, kThr = 64 * NW;
    constexpr int MT = BM / WM / 32, NT = BN / WN / 32;           // 32 x 32 MFMA tiles per wavefront along m and n
    constexpr int kRows = BM + BN;
    constexpr int kStage = kRows * kWideRow;
    constexpr int kOutRow = BN * 2 + 16;
    constexpr int kLds = 2 * kStage > BM * kOutRow ? 2 * kStage : BM * kOutRow;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int per_xcd = (n_tiles + 7) / 8;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    int row_block = tile / tiles_n, column = tile % tiles_n;
    if constexpr (CONV) {                                         // the row blocks that only x has, whose own overlap, come last
        const int both = conv.z_blocks * tiles_n, x_columns = (int)(out.width[0] / BN);
        if (tile >= both) row_block = conv.z_blocks + (tile - both) / x_columns, column = (tile - both) % x_columns;
    }
    const int64_t n0 = (int64_t)column * BN;
    int64_t m0;
    int dead;                                                     // leading rows that belong to the row block before
    if (CONV && n0 < out.width[0]) rows_of_block<BM, true>(row_block, M, &m0, &dead);
    else rows_of_block<BM, false>(row_block, M, &m0, &dead);

    // Loads: wavefront v takes the row groups g = NW j + v (rows 8 g .. 8 g + 7 of the stage; x rows first, then w);
    // lane l lands in row 8 g + l / 8, slot l % 8, and therefore fetches slot (l % 8) ^ ((4 (g & 1) + l / 16) & 7)
    // of that row (g & 1 == v & 1).
    constexpr int NLX = BM / 8 / NW, NLW = BN / 8 / NW;      // loads per wavefront and slab
    const uint32_t lane_off = (uint32_t)((lane >> 3) * K * 2 + (((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) << 4));
    const char *xrow = reinterpret_cast<const char *>(x + (m0 + 8 * wave) * K);
    const char *wrow = reinterpret_cast<const char *>(w + (n0 + 8 * wave) * K);
    const int64_t rows_nw = 16 * NW * K;                           // bytes between a wavefront's groups of 8 rows
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;
    // loads [first, last) of the slab at k0 into the stage at byte `stage`
    auto request = [&](int64_t k0, int stage, auto first, auto last) __attribute__((always_inline)) {
#pragma unroll
        for (int i = decltype(first)::value; i < decltype(last)::value; ++i) {
            const char *base = i < NLX ? xrow + (i * rows_nw + 2 * k0) : wrow + ((i - NLX) * rows_nw + 2 * k0);
            load_to_lds16(base, lane_off, lds0 + stage + (i < NLX ? 0 : BM * kWideRow) + wave * 1024 + (i < NLX ? i : i - NLX) * (1024 * NW));
        }
    };
    typedef std::integral_constant<int, 0> L0;
    typedef std::integral_constant<int, (NLX + NLW) / 4> L1;
    typedef std::integral_constant<int, (NLX + NLW) / 2> L2;
    typedef std::integral_constant<int, 3 * (NLX + NLW) / 4> L3;
    typedef std::integral_constant<int, NLX + NLW> L4;

    f32x16 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    // fragment of k16 step ks: row lane % 32 of a 32-row block, slot (2 ks + lane / 32) ^ ((lane >> 1) & 7)
    int frag_x[4], frag_w[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int slot = ((2 * ks + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4;
        frag_x[ks] = (wm * (BM / WM) + (lane & 31)) * kWideRow + slot;
        frag_w[ks] = (BM + wn * (BN / WN) + (lane & 31)) * kWideRow + slot;
    }
    struct Frags { bf16x8 xf[MT], wf[NT]; };
    auto load_x = [&](const unsigned char *stage, int ks, Frags &f, int t) __attribute__((always_inline)) {
        f.xf[t] = *reinterpret_cast<const bf16x8 *>(stage + frag_x[ks] + t * 32 * kWideRow);
    };
    auto load_w = [&](const unsigned char *stage, int ks, Frags &f, int t) __attribute__((always_inline)) {
        f.wf[t] = *reinterpret_cast<const bf16x8 *>(stage + frag_w[ks] + t * 32 * kWideRow);
    };
    auto load_frags = [&](const unsigned char *stage, int ks, Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < MT; ++t) load_x(stage, ks, f, t);
#pragma unroll
        for (int t = 0; t < NT; ++t) load_w(stage, ks, f, t);
    };
    auto multiply_row = [&](const Frags &f, int a) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NT; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.wf[b], f.xf[a], acc[a][b], 0, 0, 0);
    };
    auto multiply = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < MT; ++a) multiply_row(f, a);
    };
    // Slab s, read from stage s % 2, whose first fragments are already in f0.  Four quarters of MT NT MFMAs; the
    // fragments of a quarter are read during the one before it (the instruction groups keep the scheduler from
    // moving the reads next to their use).  After the third quarter every read of this stage has been issued, and is waited
    // for: behind the barrier other wavefronts' loads overwrite the stage, which keep no order with a read that is still
    // under way.  The slab s + 1 must have landed by then (requested a slab ago), the barrier publishes it, the stage of slab s is
    // free, and the last quarter requests slab s + 2 into it (REQUEST) and reads the first fragments of slab s + 1
    // (NEXT) between its multiplications.
    Frags f0, f1;
    auto slab = [&](auto parity, int64_t k_next, auto do_request, auto do_next) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        constexpr bool REQUEST = decltype(do_request)::value, NEXT = decltype(do_next)::value;
        const unsigned char *cur = lds + P * kStage;
        const unsigned char *nxt = lds + (1 - P) * kStage;
/* one fragment read per two MFMAs */
#define MAMBA_WIDE_SPREAD __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); __builtin_amdgcn_sched_group_barrier(0x008, NT / 2, 0);
#define MAMBA_WIDE_QUARTER(KS, FA, FB)                                                                                \
        load_frags(cur, KS, FB);                                                                                      \
        multiply(FA);                                                                                                 \
        MAMBA_WIDE_SPREAD MAMBA_WIDE_SPREAD                                                                           \
        if constexpr (MT == 4) { MAMBA_WIDE_SPREAD MAMBA_WIDE_SPREAD }                                                \
        __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);                                                           \
        __builtin_amdgcn_sched_group_barrier(0x008, MT * NT / 2, 0);                                                  \
        __builtin_amdgcn_sched_barrier(0);
        MAMBA_WIDE_QUARTER(1, f0, f1)
        MAMBA_WIDE_QUARTER(2, f1, f0)
        MAMBA_WIDE_QUARTER(3, f0, f1)
#undef MAMBA_WIDE_QUARTER
#undef MAMBA_WIDE_SPREAD
        // vmcnt(0) lgkmcnt(0): this wavefront's part of slab s + 1 is in LDS, its fragments of slab s are in registers
        __builtin_amdgcn_s_waitcnt(0x0070);
        lds_barrier_linear();
#define MAMBA_WIDE_LAST(A, FROM, TO)                                                                                  \
        if constexpr (REQUEST) request(k_next, P * kStage, FROM(), TO());                                             \
        if constexpr (NEXT) {                                                                                         \
            if constexpr (A < MT) load_x(nxt, 0, f0, A);                                                              \
            if constexpr (A < NT) load_w(nxt, 0, f0, A);                                                              \
        }                                                                                                             \
        if constexpr (A < MT) multiply_row(f1, A);                                                                    \
        __builtin_amdgcn_sched_barrier(0);
        MAMBA_WIDE_LAST(0, L0, L1)
        MAMBA_WIDE_LAST(1, L1, L2)
        MAMBA_WIDE_LAST(2, L2, L3)
        MAMBA_WIDE_LAST(3, L3, L4)
#undef MAMBA_WIDE_LAST
    };
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    const int S = (int)(K / kWideBK);
    request(0, 0, L0(), L4());
    request(kWideBK, kStage, L0(), L4());
    // vmcnt(loads of one slab): slab 0 is in, slab 1 may be under way (vmcnt is split over bits 3:0 and 15:14)
    __builtin_amdgcn_s_waitcnt(0x0F70 | ((NLX + NLW) & 15) | (((NLX + NLW) >> 4) << 14));
    lds_barrier_linear();
    load_frags(lds, 0, f0);
    int s = 0;
    for (; s + 2 < S; s += 2) {
        slab(Even(), (int64_t)(s + 2) * kWideBK, std::true_type(), std::true_type());
        slab(Odd(), (int64_t)(s + 3) * kWideBK, std::true_type(), std::true_type());
    }
    slab(Even(), 0, std::false_type(), std::true_type());         // S is even: two slabs left, nothing more to request
    slab(Odd(), 0, std::false_type(), std::false_type());
    // Epilogue.  The residual chunks this thread will add are requested first, all at once: with one workgroup per
    // CU nothing else would hide their latency, and fetched four at a time inside the store loop they cost a third
    // of the tile's time.
    constexpr int kCpr = BN / 8, kChunks = BM * kCpr / kThr;
    u32x4 res[kChunks];
    if (residual) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const int c = tid + i * kThr, row = c / kCpr, cc = c % kCpr;
            int64_t col;
            const int sp = locate(out, n0 + cc * 8, &col);
            // (a dead row is not read: where the residual is the output itself its owner may be writing it)
            res[i] = *reinterpret_cast<const u32x4 *>(residual + (m0 + (row < dead ? dead : row)) * out.width[sp] + col);
        }
    }
    lds_barrier_linear();                                         // the stages are free for the output tile (the requests stay in flight)

    // acc[a][b][4 g + j] is C[m = 32 a + lane % 32][n = 32 b + 8 g + 4 (lane / 32) + j] of the wavefront's part
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int nl = wn * (BN / WN) + b * 32 + 8 * g + 4 * (lane >> 5);
            float4 bv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (bias) bv = *reinterpret_cast<const float4 *>(bias + n0 + nl);
#pragma unroll
            for (int a = 0; a < MT; ++a) {
                const int ml = wm * (BM / WM) + a * 32 + (lane & 31);
                uint2 v;
                v.x = f32x2_to_bf16x2(acc[a][b][4 * g + 0] + bv.x, acc[a][b][4 * g + 1] + bv.y);
                v.y = f32x2_to_bf16x2(acc[a][b][4 * g + 2] + bv.z, acc[a][b][4 * g + 3] + bv.w);
                *reinterpret_cast<uint2 *>(lds + ml * kOutRow + nl * 2) = v;
            }
            __builtin_amdgcn_sched_barrier(0);                    // one group at a time: the accumulators stay where they are until used
        }
    lds_barrier_linear();
    if constexpr (CONV) {
        if (n0 < out.width[0]) {                                  // width[0] is a multiple of BN
            conv_rows<BM, BN, kThr, kOutRow>(lds, m0, dead, n0, out.ptr[0], out.width[0], conv);
            return;
        }
    }
    auto store_chunk = [&](int i, int row, int cc) __attribute__((always_inline)) {
        uint4 v = *reinterpret_cast<const uint4 *>(lds + row * kOutRow + cc * 16);
        int64_t col;
        const int sp = locate(out, n0 + cc * 8, &col);
        const int64_t off = (m0 + row) * out.width[sp] + col;
        if (residual) {
            const u32x4 r = res[i];
            v.x = f32x2_to_bf16x2(bf16_lo(v.x) + bf16_lo(r.x), bf16_hi(v.x) + bf16_hi(r.x));
            v.y = f32x2_to_bf16x2(bf16_lo(v.y) + bf16_lo(r.y), bf16_hi(v.y) + bf16_hi(r.y));
            v.z = f32x2_to_bf16x2(bf16_lo(v.z) + bf16_lo(r.z), bf16_hi(v.z) + bf16_hi(r.z));
            v.w = f32x2_to_bf16x2(bf16_lo(v.w) + bf16_lo(r.w), bf16_hi(v.w) + bf16_hi(r.w));
        }
        *reinterpret_cast<uint4 *>(out.ptr[sp] + off) = v;
    };
    if (dead == 0) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) store_chunk(i, (tid + i * kThr) / kCpr, (tid + i * kThr) % kCpr);
    } else {
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
            if ((tid + i * kThr) / kCpr >= dead) store_chunk(i, (tid + i * kThr) / kCpr, (tid + i * kThr) % kCpr);
    }
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------------------------------
// One round of tiles (the projections of a context of some hundred to a few thousand tokens): no CU has a second tile to work
// on while it waits, so what counts is how many slabs are under way.  A slab of 64 k takes about 1 us to come from the last-level
// cache and 0.1 to 0.4 to be multiplied, so a ring of LDS stages holds as many slabs as fit (64 x 128 tiles: six of 24 KB, 128 x
// 128: four of 32 KB, both eight wavefronts and one workgroup to a CU; 64 x 64: four of 16 KB, four wavefronts and two), all but
// one of them requested.  Loads, swizzle and fragments are those of linear_wide_kernel, and so are the sums, to the bit.  Before the
// last quarter of slab s a wavefront waits for its part of slab s + 1 (loads arrive in order, so it leaves as many under way as
// the younger slabs have), the barrier publishes that and frees the stage of slab s, and slab s + STAGES is requested into it, a
// quarter of its loads under every quarter of products.  The epilogue goes through 2 KB of LDS private to a wavefront, a 32 x 32
// block at a time, without a barrier; the residual is requested three slabs before the end.
// Of the 12.0 us of 2048 x 768, K = 1536 (64 x 128 tiles), the loads alone take 8.2 and the fragment reads with the products 8.4 (LDS: a
// slab is written once and read 2.7 times, 700 cycles against 256 of matrix work), the outputs 2 (each alone; busy over all CUs the address
// units 4.2, LDS 2.0, matrix cores 1.9).  us in chains of 24 weights,
// replayed, before (register-staged tiles, memory-to-LDS tiles of two stages) / now: 512 x 3072, K = 768 8.9 / 8.1; 1000 x 3072
// 12.3 / 10.1; 2048 x 768, K = 1536 17.1 / 12.0; 4000 x 768 19.3 / 16.1; 1500 x 1024, K = 2048 20.7 / 14.6; 2048 x 1536, K = 3072
// 41.7 / 30.8.  As one persistent workgroup per CU on 256 x 128 tiles the same scheme does not beat the tiles above on long contexts
// (32768 x 3072 175 to 182 us against 165 to 175): matrix cores on random data are held back by power there (the MFMAs alone take
// 75 us on constant operands and 97 to 106 on random ones).
// Requires M >= BM, N % BN == 0, K % 64 == 0 and output widths that are multiples of 8; the last row block moves back as above.
// grid: 8 * ceil(tiles / 8) workgroups, each XCD a contiguous range of tiles in groups of group_n columns: a walk over all
// columns would bring all of w into every XCD's L2.
template <int BM, int BN, int WM, int WN, int STAGES, int PER_CU, bool CONV = false>
__global__ void __launch_bounds__(64 * WM * WN, WM * WN * PER_CU / 4)
linear_ring_kernel(const bf16_t *x, const bf16_t *w, const float *__restrict__ bias, const bf16_t *residual,
                   int64_t M, int64_t K, int tiles_m, int tiles_n, int group_n, OutSplit out, ConvTail conv)
{
    constexpr int NW = WM * WN;
    constexpr int MT = BM / WM / 32, NT = BN / WN / 32;           // 32 x 32 MFMA tiles per wavefront along m and n
    constexpr int kStage = (BM + BN) * kWideRow;
    constexpr int NLX = BM / 8 / NW, NLW = BN / 8 / NW, NL = NLX + NLW;   // loads per wavefront and slab
    static_assert(NLX * 8 * NW == BM && NLW * 8 * NW == BN && MT * WM * 32 == BM && NT * WN * 32 == BN, "whole loads and tiles");
    constexpr int kPatch = 32 * 64;                               // a 32 x 32 block of outputs
    __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES * kStage + NW * kPatch];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || tile >= n_tiles) return;
    const int group = tile / (group_n * tiles_m), in_group = tile - group * group_n * tiles_m;
    const int width = min(group_n, tiles_n - group * group_n), row_block = in_group / width;
    const int64_t n0 = (int64_t)(group * group_n + in_group - row_block * width) * BN;
    int64_t m0;
    int dead;                                                     // leading rows that belong to the row block before
    rows_of_block<BM, CONV>(row_block, M, &m0, &dead);

    const uint32_t lane_off = (uint32_t)((lane >> 3) * K * 2 + (((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) << 4));
    const char *xrow = reinterpret_cast<const char *>(x + (m0 + 8 * wave) * K);   // of the next slab to be requested
    const char *wrow = reinterpret_cast<const char *>(w + (n0 + 8 * wave) * K);
    const int64_t rows_nw = 16 * NW * K;                          // bytes between a wavefront's groups of 8 rows
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const int S = (int)(K / kWideBK);
    int to_request = S, stage_at = 0;
    auto request = [&](auto first, auto last) __attribute__((always_inline)) {   // loads [first, last) of that slab
        if (to_request <= 0) return;
#pragma unroll
        for (int i = decltype(first)::value; i < decltype(last)::value; ++i)
            load_to_lds16(i < NLX ? xrow + i * rows_nw : wrow + (i - NLX) * rows_nw, lane_off,
                          lds0 + stage_at + (i < NLX ? 0 : BM * kWideRow) + wave * 1024 + (i < NLX ? i : i - NLX) * (1024 * NW));
    };
    auto requested = [&]() __attribute__((always_inline)) {
        stage_at = stage_at + kStage == STAGES * kStage ? 0 : stage_at + kStage;
        xrow += kWideRow;
        wrow += kWideRow;
        --to_request;
    };
    typedef std::integral_constant<int, 0> L0;
    typedef std::integral_constant<int, (NL + 3) / 4> L1;
    typedef std::integral_constant<int, (2 * NL + 3) / 4> L2;
    typedef std::integral_constant<int, (3 * NL + 3) / 4> L3;
    typedef std::integral_constant<int, NL> L4;
    // waits until no more than the loads of min(younger, STAGES - 2) slabs are under way (vmcnt is split over bits 3:0 and 15:14)
    auto wait_for = [&](int younger) __attribute__((always_inline)) {
#define MAMBA_RING_WAIT(SLABS) __builtin_amdgcn_s_waitcnt(0x0F70 | (((SLABS) * NL) & 15) | ((((SLABS) * NL) >> 4) << 14))
        static_assert(STAGES >= 3 && STAGES <= 6 && (STAGES - 2) * NL < 64, "a case for every number of slabs under way");
        if (younger >= STAGES - 2) MAMBA_RING_WAIT(STAGES - 2);
        else if (STAGES > 5 && younger == 3) MAMBA_RING_WAIT(3);
        else if (STAGES > 4 && younger == 2) MAMBA_RING_WAIT(2);
        else if (STAGES > 3 && younger == 1) MAMBA_RING_WAIT(1);
        else MAMBA_RING_WAIT(0);
#undef MAMBA_RING_WAIT
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;
    int frag_x[4], frag_w[4];                                     // as in linear_wide_kernel
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int slot = ((2 * ks + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4;
        frag_x[ks] = (wm * (BM / WM) + (lane & 31)) * kWideRow + slot;
        frag_w[ks] = (BM + wn * (BN / WN) + (lane & 31)) * kWideRow + slot;
    }
    struct Frags { bf16x8 xf[MT], wf[NT]; };
    auto load_frags = [&](const unsigned char *stage, int ks, Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < MT; ++t) f.xf[t] = *reinterpret_cast<const bf16x8 *>(stage + frag_x[ks] + t * 32 * kWideRow);
#pragma unroll
        for (int t = 0; t < NT; ++t) f.wf[t] = *reinterpret_cast<const bf16x8 *>(stage + frag_w[ks] + t * 32 * kWideRow);
    };
    auto multiply = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.wf[b], f.xf[a], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // the 16-byte chunks of the outputs that this thread stores: row 16 i + lane / 4 of block (a, b), chunk lane % 4 of its row
    auto out_row = [&](int a, int i) __attribute__((always_inline)) { return wm * (BM / WM) + a * 32 + 16 * i + (lane >> 2); };
    auto out_at = [&](int row, int b, int *sp) __attribute__((always_inline)) {
        int64_t col;
        *sp = locate(out, n0 + wn * (BN / WN) + b * 32 + (lane & 3) * 8, &col);
        return (m0 + row) * out.width[*sp] + col;
    };
    u32x4 res[MT][NT][2];

#pragma unroll
    for (int i = 0; i < STAGES - 1; ++i) {
        request(L0(), L4());
        requested();
    }
    int younger = S - 1;                                          // slabs behind the one that is waited for
    wait_for(younger);
    lds_barrier_linear();
    Frags f0, f1;
    const unsigned char *cur = lds;
    load_frags(cur, 0, f0);
    request(L0(), L1());
    const int fetch_res = residual ? (S > 3 ? S - 3 : 0) : -1;
#pragma unroll 1
    for (int s = 0; s < S; ++s) {
        if (s == fetch_res) {
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        int sp;                                   // (a dead row is not read: its owner may be writing it)
                        const int64_t at = out_at(max(out_row(a, i), dead), b, &sp);
                        res[a][b][i] = *reinterpret_cast<const u32x4 *>(residual + at);
                    }
        }
        load_frags(cur, 1, f1);
        request(L1(), L2());
        multiply(f0);
        load_frags(cur, 2, f0);
        request(L2(), L3());
        multiply(f1);
        load_frags(cur, 3, f1);
        request(L3(), L4());
        requested();
        multiply(f0);
        // every read of this stage has been issued, and the last ones are waited for (the products below want them): the stage is
        // free behind the barrier
        __builtin_amdgcn_s_waitcnt(0xC07F);                       // lgkmcnt(0)
        wait_for(--younger);
        lds_barrier_linear();
        cur = cur + kStage == lds + STAGES * kStage ? lds : cur + kStage;
        if (s + 1 < S) load_frags(cur, 0, f0);
        request(L0(), L1());
        multiply(f1);
    }

    if constexpr (CONV) {
        // the whole tile, since windows reach into the rows of other wavefronts; every read of the stages is behind the last barrier
        constexpr int kOutRow = BN * 2 + 16, kCpr = BN / 8;
        static_assert(BM * kOutRow <= STAGES * kStage, "the stages hold the output tile");
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<uint2 *>(lds + (wm * (BM / WM) + a * 32 + (lane & 31)) * kOutRow + (wn * (BN / WN) + b * 32 + 8 * g + 4 * (lane >> 5)) * 2) =
                        make_uint2(f32x2_to_bf16x2(acc[a][b][4 * g + 0], acc[a][b][4 * g + 1]), f32x2_to_bf16x2(acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]));
        lds_barrier_linear();
        if (n0 < out.width[0]) {                                  // width[0] is a multiple of BN
            conv_rows<BM, BN, 64 * NW, kOutRow>(lds, m0, dead, n0, out.ptr[0], out.width[0], conv);
        } else {
#pragma unroll
            for (int i = 0; i < BM * kCpr / (64 * NW); ++i) {
                const int row = (tid + i * 64 * NW) / kCpr, cc = (tid + i * 64 * NW) % kCpr;
                int64_t col;
                const int sp = locate(out, n0 + cc * 8, &col);
                if (row >= dead)
                    *reinterpret_cast<uint4 *>(out.ptr[sp] + (m0 + row) * out.width[sp] + col) = *reinterpret_cast<const uint4 *>(lds + row * kOutRow + cc * 16);
            }
        }
        return;
    }
    // acc[a][b][4 g + j] is C[m = 32 a + lane % 32][n = 32 b + 8 g + 4 (lane / 32) + j] of the wavefront's part.  Rows of a block lie
    // 64 bytes apart, their four 16-byte slots swizzled by the row pair.
    unsigned char *patch = lds + STAGES * kStage + wave * kPatch;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int r = lane & 31;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float4 bv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (bias) bv = *reinterpret_cast<const float4 *>(bias + n0 + wn * (BN / WN) + b * 32 + 8 * g + 4 * (lane >> 5));
                uint2 v;
                v.x = f32x2_to_bf16x2(acc[a][b][4 * g + 0] + bv.x, acc[a][b][4 * g + 1] + bv.y);
                v.y = f32x2_to_bf16x2(acc[a][b][4 * g + 2] + bv.z, acc[a][b][4 * g + 3] + bv.w);
                *reinterpret_cast<uint2 *>(patch + r * 64 + ((g ^ ((r >> 1) & 3)) << 4) + 8 * (lane >> 5)) = v;
            }
            wave_sync();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int pr = 16 * i + (lane >> 2), row = out_row(a, i);
                uint4 v = *reinterpret_cast<const uint4 *>(patch + pr * 64 + (((lane & 3) ^ ((pr >> 1) & 3)) << 4));
                if (residual) {
                    const u32x4 q = res[a][b][i];
                    v.x = f32x2_to_bf16x2(bf16_lo(v.x) + bf16_lo(q.x), bf16_hi(v.x) + bf16_hi(q.x));
                    v.y = f32x2_to_bf16x2(bf16_lo(v.y) + bf16_lo(q.y), bf16_hi(v.y) + bf16_hi(q.y));
                    v.z = f32x2_to_bf16x2(bf16_lo(v.z) + bf16_lo(q.z), bf16_hi(v.z) + bf16_hi(q.z));
                    v.w = f32x2_to_bf16x2(bf16_lo(v.w) + bf16_lo(q.w), bf16_hi(v.w) + bf16_hi(q.w));
                }
                int sp;
                const int64_t at = out_at(row, b, &sp);
                if (row >= dead) *reinterpret_cast<uint4 *>(out.ptr[sp] + at) = v;
            }
            wave_sync();
        }
}

// ---------------------------------------------------------------------------------------------------
// Few output tiles (a draft position, Sec. 4.1, whose way into a block is draft_in.hip; a short context; the narrow products of a
// longer one): nothing is big, and what counts is the number of trips to memory and of barriers between the launch and the last
// store, and the instructions between them.  One workgroup per 8 CG output columns and 16 MT rows, its NW wavefronts share the
// k range in contiguous pieces of steps of 64, G steps of a wavefront in flight.
// A fragment of v_mfma_f32_16x16x32_bf16 wants row l % 16 in lane l; loaded like that, no two lanes of a quad share a
// 64-byte piece of a line and the address path takes a cycle per lane (60 for the 1 KiB, measured over 192 loads a CU).
// With a row's 64 bytes on the four lanes of a quad it takes 34, with 128 on eight lanes about half of that, so that is
// how rows are loaded; a patch of LDS private to the wavefront turns them into fragments, and later holds its partial tiles.
// A CU's share of that path is what a workgroup of 16 columns and 16 rows takes longest for (K = 1536: 96 such loads), so eight
// columns where that does not make a second round of workgroups (their fragments' other half is never written nor used), and
// tiles of up to 32 columns and 64 rows, which ask for fewer bytes an output, where there are many.
// The partial tiles of the wavefronts meet in LDS, one output per thread; what else an output needs (bias, residual) has been on
// its way since before the main loop.
// us in chains of 24 different weights, replayed (before: 64-byte pieces, the residual waited for where it was fetched, twice the
// LDS; a kernel of its own for 32-column tiles): 12 x 768, K = 1536 3.10 (3.71), 64 x 768 3.4 (3.9), 128 x 3072, K = 768 5.0 (7.0), 333 x
// 768, K = 1536 6.2 (8.5), 1000 x 768 9.0 (11.8), 512 x 512, K = 1024 3.9 (5.9).
typedef float f32x4v __attribute__((ext_vector_type(4)));

// EVEN: K = 64 NW G, one trip of every wavefront; otherwise any K that is a multiple of 8.
// STREAM: w is read once and is large (the LM head on a draft position): its loads are streaming, so that they do not push the
// blocks' weights, which the next position reads again, out of the last-level cache.
template <int MT, int CG, int NW, int G, bool EVEN, bool STREAM>
__global__ void __launch_bounds__(64 * NW)
linear_few_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w, const float *__restrict__ bias,
                  const bf16_t *residual, int M, int N, int K, OutSplit out)
{
    constexpr int kThr = NW * 64;
    constexpr int NT = (CG + 1) / 2;                               // column tiles of 16
    constexpr int kStep = (NT + MT) * 2048;                        // fragments of one step: NT column tiles of w, then MT row tiles
    constexpr int PB = G * NW * kStep <= 32 * 1024 ? G : 1;        // patches in turn: several workgroups to a CU
    constexpr int OPT = (MT * NT * 256 + kThr - 1) / kThr;         // outputs per thread
    // a wavefront's patches, and its partial tiles once it is done with those
    constexpr int kWave = PB * kStep > MT * NT * 1024 ? PB * kStep : MT * NT * 1024;
    __shared__ __attribute__((aligned(16))) unsigned char patch[NW][kWave];
    const unsigned tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned li = lane & 15, lg = lane >> 4;                 // fragment view: row, 16-byte chunk of a k32 half
    const unsigned lrow = lane >> 3, lch = lane & 7;               // load view: row (+ 8 t), 16-byte chunk of the step
    const int n0 = blockIdx.x * (8 * CG), m0 = blockIdx.y * (16 * MT);

    // ---- what the outputs of this thread need besides their sums (nothing is used where it is fetched): tile o / 256 (row tile
    // by row tile), accumulator (o / 64) % 4 of lane o % 64
    int om[OPT], on[OPT];
    uint16_t res[OPT];
    float bias_in[OPT];
#pragma unroll
    for (int j = 0; j < OPT; ++j) {
        const int o6 = wave + j * NW, tile = o6 >> 2;
        om[j] = m0 + tile / NT * 16 + (o6 & 3) + 4 * (int)lg;
        on[j] = n0 + tile % NT * 16 + (int)li;
        const unsigned col = (unsigned)min(on[j], N - 1);
        // (unconditional requests: one under a condition is converted, and so waited for, inside its branch)
        bias_in[j] = (bias ? bias : reinterpret_cast<const float *>(x))[bias ? col : 0u];
        res[j] = (residual ? residual : x)[residual ? (int64_t)min(om[j], M - 1) * N + col : 0];   // single output tensor
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- the wavefront's share of k: steps [s_first, s_end)
    const int steps = EVEN ? NW * G : (K + 63) >> 6, per = EVEN ? G : (steps + NW - 1) / NW;
    const int s_first = wave * per, s_end = EVEN || s_first + per < steps ? s_first + per : steps;
    const unsigned kchunks = (unsigned)K >> 3;                     // K % 8 == 0
    const char *wb = reinterpret_cast<const char *>(w + (int64_t)n0 * K), *xb = reinterpret_cast<const char *>(x + (int64_t)m0 * K);
    unsigned wo[CG], xo[2 * MT];
    int64_t wfar[CG], xfar[2 * MT];
#pragma unroll
    for (unsigned t = 0; t < CG; ++t) {
        const unsigned r = min(8 * t + lrow, (unsigned)(N - 1 - n0));
        wo[t] = r * (2u * (unsigned)K) + 16 * lch;
        wfar[t] = (int64_t)r * 2 * K + 16 * lch;
    }
#pragma unroll
    for (unsigned t = 0; t < 2 * MT; ++t) {
        const unsigned r = min(8 * t + lrow, (unsigned)(M - 1 - m0));   // rows past M repeat the last one, never stored
        xo[t] = r * (2u * (unsigned)K) + 16 * lch;
        xfar[t] = (int64_t)r * 2 * K + 16 * lch;
    }
    const unsigned put = (lrow * 8 + (lch ^ lrow)) * 16;           // + 1024 t: chunks xor-swizzled by the row, no bank conflicts either way
    const unsigned get0 = (li * 8 + (lg ^ (li & 7))) * 16, get1 = (li * 8 + ((lg + 4) ^ (li & 7))) * 16;

    f32x4v acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] = f32x4v(0.0f);
    bool first = true;
    for (int s0 = s_first; EVEN ? first : s0 < s_end; s0 += G) {
        first = false;
        u32x4 wf[G][CG], xf[G][2 * MT];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int s = EVEN || s0 + g < s_end ? s0 + g : 0;
            const unsigned back = EVEN || 8u * (unsigned)s + lch < kchunks ? 0u : 16 * lch;   // chunks past K re-read the step's first one
            const char *ws = wb + (int64_t)s * 128, *xs = xb + (int64_t)s * 128;
#pragma unroll
            for (int t = 0; t < CG; ++t) {
                const u32x4 *p = reinterpret_cast<const u32x4 *>(EVEN ? ws + wo[t] : ws + (wfar[t] - back));
                wf[g][t] = STREAM ? __builtin_nontemporal_load(p) : *p;
            }
#pragma unroll
            for (int t = 0; t < 2 * MT; ++t) xf[g][t] = *reinterpret_cast<const u32x4 *>(EVEN ? xs + xo[t] : xs + (xfar[t] - back));
        }
        __builtin_amdgcn_sched_barrier(0);                         // all of it in flight before any of it is used
        if (s0 == s_first) args_here(out.ptr[0], out.ptr[1], out.ptr[2], out.width[0], out.width[1], out.width[2]);
        auto fill = [&](int g) __attribute__((always_inline)) {
            unsigned char *p = patch[wave] + g % PB * kStep;
            const bool ok = EVEN || (s0 + g < s_end && 8u * (unsigned)(s0 + g) + lch < kchunks);   // else zeros: adds nothing
#pragma unroll
            for (int t = 0; t < CG; ++t) *reinterpret_cast<u32x4 *>(p + 1024 * t + put) = ok ? wf[g][t] : u32x4(0u);
#pragma unroll
            for (int t = 0; t < 2 * MT; ++t) *reinterpret_cast<u32x4 *>(p + 2048 * NT + 1024 * t + put) = ok ? xf[g][t] : u32x4(0u);
        };
        auto product = [&](int g) __attribute__((always_inline)) {
            const unsigned char *p = patch[wave] + g % PB * kStep;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned get = h ? get1 : get0;
                bf16x8 wv[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) wv[n] = *reinterpret_cast<const bf16x8 *>(p + 2048 * n + get);
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const bf16x8 xv = *reinterpret_cast<const bf16x8 *>(p + 2048 * (NT + t) + get);
#pragma unroll
                    for (int n = 0; n < NT; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, wv[n], acc[t][n], 0, 0, 0);
                }
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
    // acc[t][n][i] is C[m = 16 t + 4 (lane / 16) + i][16 n + lane % 16]
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) reinterpret_cast<float *>(patch[wave])[(4 * (t * NT + n) + i) * 64 + lane] = acc[t][n][i];
#pragma unroll
    for (int j = 0; j < OPT; ++j) values_here(bias_in[j]);
    lds_barrier_linear();

#pragma unroll
    for (int j = 0; j < OPT; ++j) {
        const int o6 = wave + j * NW, at = (o6 < 4 * MT * NT ? o6 : 0) * 64 + (int)lane;
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < NW; ++q) v += reinterpret_cast<const float *>(patch[q])[at];
        if (o6 >= 4 * MT * NT || om[j] >= M || on[j] >= N || li >= 8 * CG) continue;
        v = bf16_to_f32(f32_to_bf16(v + (bias ? bias_in[j] : 0.0f)));   // same two roundings as the tiled kernel
        if (residual) {
            out.ptr[0][(int64_t)om[j] * N + on[j]] = (bf16_t)f32_to_bf16(v + bf16_to_f32(res[j]));
            continue;
        }
        int64_t col;
        const int sp = locate(out, on[j], &col);
        (sp == 0 ? out.ptr[0] : sp == 1 ? out.ptr[1] : out.ptr[2])[(int64_t)om[j] * (sp == 0 ? out.width[0] : sp == 1 ? out.width[1] : out.width[2]) + col] =
            (bf16_t)f32_to_bf16(v);
    }
}

template <int MT, int CG, bool STREAM = false>
hipError_t launch_few(const bf16_t *x, const bf16_t *w, const float *bias, const bf16_t *res, const OutSplit &o, int64_t M, int64_t N, int64_t K,
                      hipStream_t stream)
{
    const dim3 grid((unsigned)((N + 8 * CG - 1) / (8 * CG)), (unsigned)((M + 16 * MT - 1) / (16 * MT)));
#define MAMBA_FEW_K(NW, G, EVEN) linear_few_kernel<MT, CG, NW, G, EVEN, STREAM><<<grid, 64 * NW, 0, stream>>>(x, w, bias, res, (int)M, (int)N, (int)K, o)
    const int64_t per = (K + 511) / 512;
    if (K == 256) MAMBA_FEW_K(4, 1, true);
    else if (K < 256) MAMBA_FEW_K(4, 1, false);
    else if (K == 512) MAMBA_FEW_K(8, 1, true);
    else if (K == 768) MAMBA_FEW_K(6, 2, true);
    else if (K == 1024) MAMBA_FEW_K(8, 2, true);
    else if (K == 1536) MAMBA_FEW_K(8, 3, true);
    else if (per <= 2 || per == 4) MAMBA_FEW_K(8, 2, false);
    else MAMBA_FEW_K(8, 3, false);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int STAGES, int PER_CU, bool CONV = false>
hipError_t launch_ring(const bf16_t *x, const bf16_t *w, const float *bias, const bf16_t *res, const OutSplit &o, int64_t M, int64_t N, int64_t K,
                       hipStream_t stream, const ConvTail &conv = ConvTail{})
{
    const int tiles_m = (int)row_blocks(M, BM, CONV), tiles_n = (int)(N / BN);
    // columns of a group: as many as bring about 2 MB of w, half of an XCD's L2, in groups of equal width
    const int64_t most = std::max<int64_t>(1, ((int64_t)9 << 18) / (BN * 2 * K));
    const int64_t groups = (tiles_n + most - 1) / most;
    const unsigned per_xcd = (unsigned)((tiles_m * tiles_n + 7) / 8);
    linear_ring_kernel<BM, BN, WM, WN, STAGES, PER_CU, CONV><<<8 * per_xcd, 64 * WM * WN, 0, stream>>>(
        x, w, bias, res, M, K, tiles_m, tiles_n, (int)((tiles_n + groups - 1) / groups), o, conv);
    return hipGetLastError();
}

template <int BM, int BN, bool CONV = false, int WM = 2, int WN = 2>
hipError_t launch_wide(const bf16_t *x, const bf16_t *w, const float *bias, const bf16_t *res, const OutSplit &o, int64_t M, int64_t N, int64_t K,
                       hipStream_t stream, ConvTail conv = ConvTail{})
{
    const int64_t tiles_n = N / BN, z_blocks = row_blocks(M, BM, false);
    const int64_t n_tiles = z_blocks * tiles_n + (CONV ? (row_blocks(M, BM, true) - z_blocks) * (o.width[0] / BN) : 0);
    conv.z_blocks = (int)z_blocks;
    linear_wide_kernel<BM, BN, CONV, WM, WN><<<(unsigned)(8 * ((n_tiles + 7) / 8)), 64 * WM * WN, 0, stream>>>(x, w, bias, res, o, M, N, K, (int)tiles_n, (int)n_tiles, conv);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_linear(const LinearArgs &a, hipStream_t stream)
{
    OutSplit o;
    for (int s = 0; s < 3; ++s) {
        o.ptr[s] = static_cast<bf16_t *>(a.out[s]);
        o.width[s] = a.width[s];
    }
    const int64_t N = a.width[0] + a.width[1] + a.width[2];
    const int vec = linear_vector_out(a.width) ? 1 : 0;
    const bf16_t *x = static_cast<const bf16_t *>(a.x), *w = static_cast<const bf16_t *>(a.w);
    const bf16_t *res = static_cast<const bf16_t *>(a.residual);
    if (a.norm_w) return launch_draft_in(a, stream);
#define MAMBA_LINEAR(HOW, ...) return launch_##HOW<__VA_ARGS__>(x, w, a.bias, res, o, a.M, N, a.K, stream)
#define MAMBA_TILES(BM, BN, ...)                                                                                                      \
    linear_kernel<BM, BN, __VA_ARGS__><<<dim3((unsigned)((N + BN - 1) / BN), (unsigned)((a.M + BM - 1) / BM)), kThreads, 0, stream>>>( \
        x, w, a.bias, res, o, a.M, N, a.K, vec);                                                                                      \
    return hipGetLastError()
    switch (linear_route(a.M, a.width, a.K)) {
    case kFew16x16Stream: MAMBA_LINEAR(few, 1, 2, true);
    case kFew16x8: MAMBA_LINEAR(few, 1, 1);
    case kFew16x16: MAMBA_LINEAR(few, 1, 2);
    case kFew32x16: MAMBA_LINEAR(few, 2, 2);
    case kFew64x32: MAMBA_LINEAR(few, 4, 4);
    case kFew32x32: MAMBA_LINEAR(few, 2, 4);
    case kRing64: MAMBA_LINEAR(ring, 64, 64, 2, 2, 4, 2);
    case kRing64x128: MAMBA_LINEAR(ring, 64, 128, 2, 4, 6, 1);
    case kRing128: MAMBA_LINEAR(ring, 128, 128, 2, 4, 4, 1);
    case kWide256x192: MAMBA_LINEAR(wide, 256, 192, false, 4, 2);
    case kWide256: MAMBA_LINEAR(wide, 256, 256, false, 2, 4);
    case kWide192: MAMBA_LINEAR(wide, 192, 128);
    case kWide128Eight: MAMBA_LINEAR(wide, 128, 128, false, 2, 4);
    case kWide128: MAMBA_LINEAR(wide, 128, 128);
    case kTiles128: MAMBA_TILES(128, 128, 64);
    case kTiles64x128: MAMBA_TILES(64, 128, 64);
    case kTiles64Deep: MAMBA_TILES(64, 64, 256);
    case kTiles64Stream: MAMBA_TILES(64, 64, 64, true);
    case kTiles64: MAMBA_TILES(64, 64, 64);
    case kNoKernel: break;
    }
    return hipErrorInvalidValue;
#undef MAMBA_TILES
#undef MAMBA_LINEAR
}

hipError_t launch_linear_conv(const LinearArgs &a, hipStream_t stream)
{
    const OutSplit o{{static_cast<bf16_t *>(a.out[0]), static_cast<bf16_t *>(a.out[1]), nullptr}, {a.width[0], a.width[1], 0}};
    const bf16_t *x = static_cast<const bf16_t *>(a.x), *w = static_cast<const bf16_t *>(a.w);
    const ConvTail conv{a.conv_w, a.conv_b, static_cast<const bf16_t *>(a.conv_src), static_cast<bf16_t *>(a.conv_dst), (uint32_t)a.conv_L, 0};
    const int64_t N = a.width[0] + a.width[1];
#define MAMBA_CONV(HOW, ...) return launch_##HOW<__VA_ARGS__, true>(x, w, nullptr, nullptr, o, a.M, N, a.K, stream, conv)
    switch (linear_conv_tiles(a.M, a.width[0], a.K, a.conv_k)) {
    case kConvWide256: return launch_wide<256, 256, true, 2, 4>(x, w, nullptr, nullptr, o, a.M, N, a.K, stream, conv);
    case kConvRing64: MAMBA_CONV(ring, 64, 64, 2, 2, 4, 2);
    case kConvRing64x128: MAMBA_CONV(ring, 64, 128, 2, 4, 6, 1);
    case kConvRing128: MAMBA_CONV(ring, 128, 128, 2, 4, 4, 1);
    case kConvWide128: MAMBA_CONV(wide, 128, 128);
    case kConvWide192: MAMBA_CONV(wide, 192, 128);
    default: return hipErrorInvalidValue;
    }
#undef MAMBA_CONV
}

}  // namespace mamba
