// Token-side ends of the drafter around the blocks (the paper's drafter is a Mamba-130M language
// model, Sec. 3.1; in tree drafting every node proposes N_i children, Sec. 4.1): the embedding
// lookup that turns draft tokens into hidden rows, and the selection of the k most probable next
// tokens of every branch from the LM head's logits.
#include "device_math.h"
#include "launch.h"

namespace mamba {
namespace {

constexpr int kBlock = 256;

// out[m, :] = table[tokens[m], :]; rows of dm bf16 moved as 16-byte vectors (dm % 8 == 0).
// A token outside [0, V) yields a row of NaN instead of an out-of-bounds read.
// (The sizes are one aggregate and come first, so that the kernel fetches its arguments and nobody brings them in registers: 1 token
// 1.80 -> 1.69 us, 12 1.95 -> 1.80, 333 2.03 -> 1.92; 8000 5.43 -> 5.75.)
struct EmbeddingSizes {
    int64_t V, vecs;
};
__global__ void __launch_bounds__(kBlock)
embedding_kernel(EmbeddingSizes sizes, const int32_t *__restrict__ tokens, const uint4 *__restrict__ table, uint4 *__restrict__ out)
{
    const int64_t V = sizes.V, vecs = sizes.vecs;
    const int64_t m = blockIdx.x;
    const int64_t t = tokens[m];
    const bool ok = t >= 0 && t < V;
    for (int64_t v = threadIdx.x; v < vecs; v += kBlock)
        out[m * vecs + v] = ok ? table[t * vecs + v] : make_uint4(~0u, ~0u, ~0u, ~0u);
}

// Ranking works on integer keys that order like (value, then lower index first), a total order, so
// the result is unique.  The upper 16 bits of a key are the bf16 logit's, made to order as a signed
// integer (NaN ranks as -inf and so never wins against a number).  While a lane scans its share of a
// row the lower 16 are the complement of the candidate's sequence number in the lane (the lane meets
// its elements in index order); for the merge over the workgroup they are dropped and the complement
// of the index in the row takes their place in a register of its own.
constexpr int32_t kNoKey = INT32_MIN;                                // below every key (-inf orders as 0x807f....)
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// two logits to two integers that order like them (no NaN), two instructions for both
__device__ __forceinline__ uint32_t ordered2(uint32_t pair)
{
    const uint32_t sign = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, pair) >> 15);
    return pair ^ (sign & 0x7fff7fffu);
}
__device__ __forceinline__ uint32_t nan_to_lowest(uint32_t b) { return (b & 0x7fffu) > 0x7f80u ? 0xff80u : b; }
__device__ __forceinline__ uint32_t nans_to_lowest(uint32_t pair) { return nan_to_lowest(pair & 0xffffu) | nan_to_lowest(pair >> 16) << 16; }
__device__ __forceinline__ u16x2 magnitude2(uint32_t pair) { return __builtin_bit_cast(u16x2, pair & 0x7fff7fffu); }
__device__ __forceinline__ float ordered_value(int32_t o)
{
    const uint32_t b = (uint32_t)(o ^ ((o >> 31) & 0x7fffffff));
    return __uint_as_float(b & 0xffff0000u);
}

__device__ __forceinline__ int32_t middle(int32_t a, int32_t b, int32_t c)
{
    int32_t r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
template <int CTRL> __device__ __forceinline__ int32_t lane_max(int32_t v)
{
    return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false));
}
// largest of 16 lanes, in all of them: quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
__device__ __forceinline__ int32_t row_max(int32_t v) { return lane_max<0x140>(lane_max<0x141>(lane_max<0x4e>(lane_max<0xb1>(v)))); }
// largest of the 64 lanes: row_bcast:15 and row_bcast:31 bring the rows together in the last one
__device__ __forceinline__ int32_t wave_max(int32_t v) { return __builtin_amdgcn_readlane(lane_max<0x143>(lane_max<0x142>(row_max(v))), 63); }

constexpr int kTopkBlock = 1024, kTopkWaves = kTopkBlock / 64;
constexpr int kTopkTurn = 8;                                         // 16-byte vectors of a lane requested together
constexpr uint32_t kSeqHead = 0, kSeqTail = 0xfffe;                  // sequence numbers of the scalar ends

// One workgroup per row.  Every lane keeps the KMAX best keys of its share in a sorted register
// list; the row is read as 16-byte vectors where it is aligned, the few elements before and after
// as scalars.  Then k rounds pick the best head over the workgroup and its owner pops it.
// What a launch takes is instructions: 49 tokens a lane and four wavefronts to a SIMD for a row of 50280, each token about three
// instructions to make a key of and KMAX to sort in (two tokens made to order at once, NaNs looked for by one maximum over the whole
// share), then for every round the best of 1024 lanes, twice six lane exchanges of one instruction each.  us a launch, 1 row k = 3, 3
// rows k = 2, 12 rows k = 1, 64 rows k = 8: 6.8, 5.8, 4.7, 13.8; with 11 and more instructions a token, one vector of a lane in
// flight and 64-bit exchanges through LDS 10.9, 8.0, 7.6, 22.4.
template <int KMAX>
__global__ void __launch_bounds__(kTopkBlock)
topk_kernel(const bf16_t *__restrict__ logits, int32_t *__restrict__ idx, float *__restrict__ val, int64_t V, int k)
{
    const int64_t m = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bf16_t *row = logits + m * V;
    int32_t best[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) best[j] = kNoKey;
    auto offer = [&](uint32_t ordered_up, uint32_t below) {          // the upper 16 bits of the first, the lower of the second
        const int32_t key = (int32_t)((ordered_up & 0xffff0000u) | below);
        // the list is sorted: what stands in a place is the middle one of it, the one above and the newcomer
#pragma unroll
        for (int j = KMAX - 1; j > 0; --j) best[j] = middle(key, best[j - 1], best[j]);
        best[0] = max(key, best[0]);
    };
    const int64_t head = min<int64_t>((8 - (m * V) % 8) % 8, V);     // elements before the first aligned vector
    const int64_t nvec = (V - head) / 8, tail0 = head + nvec * 8;
    const uint4 *vrow = reinterpret_cast<const uint4 *>(row + head);
    const uint32_t first = row[tid < head ? tid : 0], last = row[tail0 + tid < V ? tail0 + tid : 0];
    uint32_t seq = 1;
    for (int64_t v0 = tid; v0 < nvec; v0 += kTopkBlock * kTopkTurn) {
        uint4 q[kTopkTurn];
#pragma unroll
        for (int u = 0; u < kTopkTurn; ++u) q[u] = vrow[min<int64_t>(v0 + u * kTopkBlock, nvec - 1)];
        __builtin_amdgcn_sched_barrier(0);
        // a NaN anywhere (rare) is replaced ahead of the scan
        u16x2 most = magnitude2(q[0].x);
#pragma unroll
        for (int u = 0; u < kTopkTurn; ++u)
            most = __builtin_elementwise_max(most, __builtin_elementwise_max(__builtin_elementwise_max(magnitude2(q[u].x), magnitude2(q[u].y)),
                                                                             __builtin_elementwise_max(magnitude2(q[u].z), magnitude2(q[u].w))));
        if (most.x > 0x7f80 || most.y > 0x7f80) {
#pragma unroll
            for (int u = 0; u < kTopkTurn; ++u)
                q[u] = make_uint4(nans_to_lowest(q[u].x), nans_to_lowest(q[u].y), nans_to_lowest(q[u].z), nans_to_lowest(q[u].w));
        }
#pragma unroll
        for (int u = 0; u < kTopkTurn; ++u, seq += 8) {
            if (v0 + u * kTopkBlock >= nvec) break;
            const uint32_t words[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t o = ordered2(words[i]);
                offer(o << 16, 0xffffu - (seq + 2 * i));
                offer(o, 0xffffu - (seq + 2 * i + 1));
            }
        }
    }
    if (tid < head) offer(ordered2(nan_to_lowest(first)) << 16, 0xffffu - kSeqHead);
    if (tail0 + tid < V) offer(ordered2(nan_to_lowest(last)) << 16, 0xffffu - kSeqTail);

    // value and complement of the index (31 bits) of the lane's list
    int32_t value[KMAX], below[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        const uint32_t sq = 0xffffu - ((uint32_t)best[j] & 0xffffu);
        const int64_t e = sq == kSeqHead ? tid : sq == kSeqTail ? tail0 + tid
                        : head + ((int64_t)tid + (int64_t)((sq - 1) >> 3) * kTopkBlock) * 8 + ((sq - 1) & 7);
        value[j] = best[j] == kNoKey ? kNoKey : best[j] >> 16;
        below[j] = best[j] == kNoKey ? -1 : (int32_t)~((uint32_t)e | 0x80000000u);
    }

    __shared__ int2 heads[2][kTopkWaves];
    for (int r = 0; r < k; ++r) {
        const int32_t wv = wave_max(value[0]), wb = wave_max(value[0] == wv ? below[0] : -1);
        if (lane == 0) heads[r & 1][wave] = make_int2(wv, wb);       // (the other half may still be being read)
        __syncthreads();
        const int2 h = heads[r & 1][lane & (kTopkWaves - 1)];
        const int32_t win = __builtin_amdgcn_readfirstlane(row_max(h.x));
        const int32_t win_below = __builtin_amdgcn_readfirstlane(row_max(h.x == win ? h.y : -1));
        if (tid == 0) {
            idx[m * k + r] = win != kNoKey ? (int32_t)(~(uint32_t)win_below & 0x7fffffffu) : -1;
            val[m * k + r] = win != kNoKey ? ordered_value((int32_t)((uint32_t)win << 16)) : -INFINITY;
        }
        if (win != kNoKey && value[0] == win && below[0] == win_below) {   // candidates are distinct: one owner pops its head
#pragma unroll
            for (int j = 0; j + 1 < KMAX; ++j) value[j] = value[j + 1], below[j] = below[j + 1];
            value[KMAX - 1] = kNoKey;
            below[KMAX - 1] = -1;
        }
    }
}

}  // namespace

hipError_t launch_embedding(const int32_t *tokens, const void *table, void *out, int64_t M, int64_t V, int64_t dm,
                            hipStream_t stream)
{
    embedding_kernel<<<(unsigned)M, kBlock, 0, stream>>>(EmbeddingSizes{V, dm / 8}, tokens, static_cast<const uint4 *>(table),
                                                       static_cast<uint4 *>(out));
    return hipGetLastError();
}

hipError_t launch_topk(const void *logits, int32_t *idx, float *val, int64_t M, int64_t V, int k, hipStream_t stream)
{
    const bf16_t *lg = static_cast<const bf16_t *>(logits);
    switch (k) {
    case 1: topk_kernel<1><<<(unsigned)M, kTopkBlock, 0, stream>>>(lg, idx, val, V, k); break;
    case 2: topk_kernel<2><<<(unsigned)M, kTopkBlock, 0, stream>>>(lg, idx, val, V, k); break;
    case 3: topk_kernel<3><<<(unsigned)M, kTopkBlock, 0, stream>>>(lg, idx, val, V, k); break;
    case 4: topk_kernel<4><<<(unsigned)M, kTopkBlock, 0, stream>>>(lg, idx, val, V, k); break;
    default: topk_kernel<8><<<(unsigned)M, kTopkBlock, 0, stream>>>(lg, idx, val, V, k); break;
    }
    return hipGetLastError();
}

}  // namespace mamba
