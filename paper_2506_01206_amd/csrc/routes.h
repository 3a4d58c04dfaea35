// Conditions under which a launcher takes a kernel that cannot take every call, as plain host functions (no HIP types), so that
// they can be checked without a GPU and without tensors of the sizes they speak of.
#pragma once

#include <stdint.h>

namespace mamba {

// do the byte ranges [p, p + pn) and [q, q + qn) share a byte (null or empty: no)
inline bool overlap(const void *p, int64_t pn, const void *q, int64_t qn)
{
    if (!p || !q || pn <= 0 || qn <= 0) return false;
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b + (uintptr_t)qn && b < a + (uintptr_t)pn;
}

// Scalar-decay scan, second pass stitching the segments itself (the figures are at launch_ssd): every workgroup of a head then
// reads h0, of its batch row, while the last one writes h_final, so the two must not share a byte: not in place, and not
// shifted against each other by a row or a part of one either.  before: pass 1 segments ahead of the last pass 2 segment.
inline bool ssd_folds(int n_seg1, int before, const void *h0, const void *h_final, int64_t state_bytes)
{
    return n_seg1 > 1 && before <= 10 && !overlap(h0, state_bytes, h_final, state_bytes);
}

// The few-row product counts k and columns in 32 bits and a workgroup of 512 threads takes 16 columns: k rounded up to a step
// of 64 has to fit an int, and the grid's threads along x have to stay below 2^32.  What does not fit takes the kernels
// that count in 64 bits (at a draft position: the chain of separate launches).
inline bool linear_few_fits(int64_t N, int64_t K)
{
    return K <= (int64_t)INT32_MAX - 63 && N <= ((int64_t)1 << 27) - 16;
}

// The lanes scan (scan_lanes.hip): its states per channel, and the most dt columns that it takes the projection of.
constexpr int kLanesStates = 16, kLanesLowRank = 64;

// Channels per workgroup: what takes the fewest rounds of 256 workgroups times what one takes (a workgroup of fewer channels has
// fewer wavefronts to a SIMD and is faster, but not in proportion).  us with 2 / 4 / 6 channels, bf16 | float32 (one session):
//   1 x 1000 x  512  10.5*/ 10.6 / 13.8 | 12.3*/ 11.9 / 19.9      1 x  512 x 256   6.3*/  6.9 /  8.9 |  6.6*/  6.7 /  9.1
//   1 x 1000 x  768  14.5 / 11.7*/ 14.2 | 16.0 / 13.2*/ 17.6      1 x 2000 x 1000 26.1 / 19.9*/ 24.0 | 28.5 / 23.0*/ 29.0
//   1 x 2048 x 1536  36.3 / 37.6 / 25.0*| 37.0 / 43.2 / 31.3*     1 x 1000 x 2048 25.3 / 23.0*/ 30.7 | 28.8 / 24.0*/ 32.2
inline int lanes_channels(int64_t batch, int64_t L, int64_t D)
{
    auto cost = [&](int64_t g, double round) { return (double)((batch * ((D + g - 1) / g) + 255) / 256) * round; };
    const double six = cost(6, 1.0), four = cost(4, 0.8), two = cost(2, L <= 256 ? 0.68 : 0.7);
    return two <= four && two <= six ? 2 : four <= six ? 4 : 6;
}

// Workgroups of a launch.  by_xcd: with those that fill the last group of 8 of a row, one to an XCD, as the grid has them
inline int64_t lanes_groups(int64_t batch, int64_t L, int64_t D, bool by_xcd)
{
    const int64_t g = lanes_channels(batch, L, D), row = (D + g - 1) / g;
    return batch * (by_xcd ? (row + 7) / 8 * 8 : row);
}

// ns: rounds of workgroups times what one takes, to which a token adds `six`, `four` or `two` by its channels
inline double lanes_ns(int64_t batch, int64_t L, int64_t D, double six, double four, double two, bool by_xcd = false)
{
    const int64_t g = lanes_channels(batch, L, D), groups = lanes_groups(batch, L, D, by_xcd);
    const double first = g == 6 ? 6000.0 : g == 4 ? 5000.0 : 2500.0, token = g == 6 ? six : g == 4 ? four : two;
    return (double)((groups + 255) / 256) * (first + token * (double)L);
}

// Shapes the lane-scan kernel serves: 16 states, token rows that can be read in 4-byte pieces from any even
// channel, at least one full workgroup; and among those the ones it is expected to finish before the two-pass
// kernels of scan.hip.  Its time is a number of rounds of 256 workgroups, every one walking the whole sequence;
// that of the two-pass kernels goes with all tokens.  The line lies between the two types, since the choice, and with it the size of
// the workspace, is not told the type, and it lies where the two met before the two-pass kernels' exponentials went into runs: those
// have gained more by it than this one, so that between about 7000 tokens of 1536 channels (float32: 2700) and the line they are
// ahead by up to 9 % (float32: 31 %).  But a call that this kernel took needs no workspace, and one made without would be
// refused if the line moved down.  (A whole block brings its workspace and is bf16: scan_lanes_in_block.)
// Down to 33 tokens (a call of fewer keeps the kernel that mamba_scan_kernel has always named for it; a block takes them too): one super-step
// against three launches, 1 x 40 x 1536 6.1 / 16.0, 1 x 40 x 256 3.9 / 15.8, 2 x 40 x 1536 10.8 / 16.4, 1 x 40 x 4096 15.4 / 16.3.
// us, lanes / two-pass, bf16 | float32, one session, four sets of operands in turn (on one set, which stays in the last-level
// cache, 1 x 8192 x 1536 takes 81 | 110 here); * what the line takes:
//   1 x  600 x  768  11.1*/ 20.8 | 12.0*/ 20.9       1 x 2048 x 1536  25.8*/ 35.5 | 31.4*/ 35.9       1 x   64 x 4096  15.4*/ 17.3 |  15.6*/ 17.0
//   1 x 2000 x  768  19.6*/ 30.1 | 22.7*/ 26.5       1 x 6000 x 1536  68.7*/ 73.5 | 93.5*/ 68.5       1 x 8192 x 1536  97.0*/ 92.6 | 123.8*/ 87.0
//   1 x 4000 x  768  34.0 / 37.4*| 41.0 / 37.2*      1 x 7000 x 1536  84.0*/ 83.1 |108.0*/ 79.3       1 x 10240 x 1536 125.7 / 110.7*| 152.0 / 104.2*
//   1 x 2000 x  256  17.0 / 21.8*| 21.8 / 22.0*      1 x 4000 x 1024  34.5*/ 44.3 | 41.7*/ 42.6       1 x 4000 x 512   33.8 / 32.9*| 42.1 / 29.6*
//   1 x 3000 x 1536  34.4*/ 45.5 | 48.4*/ 43.8       1 x 4000 x 1536  43.9*/ 53.9 | 65.3*/ 52.9       1 x 9900 x 1536 120.2*/110.6 | 151.8*/ 104.3
//   4 x 1000 x  768  28.3*/ 35.7 | 34.2*/ 35.5       1 x 2000 x 2048  37.6*/ 43.5 | 43.0*/ 41.6       2 x 3000 x 1536  75.2*/ 73.2 | 98.0*/ 68.4
inline bool scan_lanes_applies(int64_t batch, int64_t L, int64_t D, int64_t N)
{
    if (N != kLanesStates || D % 2 != 0 || D < 6 || L <= 32 || batch > 65535) return false;
    const double two_pass_ns = 24000.0 + 9.8 * (double)L * ((double)batch * (double)D / 1536.0);
    return lanes_ns(batch, L, D, 11.6, 9.7, 12.5) < two_pass_ns;
}

// The same in a whole block, whose scan finds its operands in the last-level cache as long as the block's four tensors of (rows, D) bf16 fit
// its 256 MB: the small pieces of the token rows that this kernel reads come sooner from there, the two passes gain nothing by it.
// What is predicted less than 15 % ahead (8 % where workgroups of fewer channels come in one round) is taken only where the workgroups, dealt
// to the XCDs in whole groups of 8, fill the last round: CUs that stand idle in it, and rows cut to other than whole lines, had cost up to
// 16 % of a block (lanes are thought 4 % ahead on 2 x 9084 x 640, whose 240 workgroups leave one CU in sixteen idle).  1100 blocks of 256 to 6144
// channels, 17 to 22000 tokens, near the line: 5.0 % ahead of the two passes on average, one of 320 taken slower by more than 1.5 % (without that
// 4.7 %, 68 of 430 slower).
// us of a block, two passes / lanes, three sets of operands in turn (* what this takes; a line within 3 us is left to the two passes):
//   1 x 10500 x 1536 260 / 243*      2 x 4000 x 1536 205 / 196*      3 x 3000 x 1536 241 / 219*      1 x  8000 x 1024 140 / 133*      1 x 6000 x 4096 545* / 554
//   1 x 16000 x 1536 368 / 346*      2 x 8000 x 1536 367 / 350*      4 x 1000 x 1536 127*/ 125       1 x 10000 x  768 134*/ 143       1 x 3000 x 2048 133 / 127*
//   1 x 20000 x 1536 458 / 437*      4 x 8000 x 1536 634*/ 724       8 x  500 x 1536 125*/ 139       1 x  9000 x 3072 537 / 518*      2 x 1500 x 2048 133* / 139
//   1 x 32768 x 1536 634*/ 744       4 x 4000 x 1536 370*/ 362       8 x 2000 x 1536 369*/ 377       1 x  6000 x  512  88*/ 81
//   2 x  9084 x  640 162*/ 192       1 x 6653 x 1280 125*/ 140       2 x 1164 x 2048  99*/ 109       1 x 14920 x 1408 332*/ 361       3 x 6795 x 448 157*/ 169
//   1 x    40 x 1536  36 /  22*      2 x   40 x 1536  37 /  28*      4 x   40 x 1536  40*/  39       1 x   493 x 3456  65*/  58       1 x 2041 x 256  43*/  38
// Contexts that the two passes take as one chunk (up to 16 tokens) are one launch there as well, of about 0.4 us a token, and dt has one
// of its own: the lanes kernel is ahead where its workgroups come in one round (dealt to the XCDs in whole groups of 8), and on more
// tokens the more rounds they come in.  400 blocks of 64 to 5120 channels, 4 to 16 tokens: 4.1 % ahead of the two passes, 4.25 the better
// of the two each time.  us of a block, two passes / lanes:
//   1 x  4 x  256  17.7 / 16.9*      1 x  4 x 1536  21.8*/ 22.3      3 x  4 x 1536  21.5*/ 31.7      6 x  8 x  768  22.6*/ 30.5      12 x  8 x 256  20.1*/ 22.8
//   1 x 16 x  256  22.5 / 16.8*      1 x 16 x 1536  26.2 / 21.9*     3 x 16 x 1536  28.1*/ 33.1      2 x 15 x 1024  25.1 / 21.4*     12 x 16 x 256  23.9 / 23.4*
//   1 x  8 x 4096  35.4*/ 44.9       1 x 16 x 2048  28.2 / 24.9*     2 x 16 x 1536  27.0*/ 27.5      4 x 13 x  256  22.4 / 18.1*      1 x  6 x 2048  24.6*/ 24.5
// and with 96 dt columns, whose projection stays apart: 1 x 4 x 768 20.1*/ 21.3, 1 x 15 x 1024 24.8 / 21.1*.
// chunks: what scan_plan cuts such a call into, for which the line above has declined.
inline bool scan_lanes_in_block(int64_t batch, int64_t L, int64_t D, int64_t N, int64_t dt_rank, int64_t chunks)
{
    if (N != kLanesStates || D % 2 != 0 || D < 6 || L < 4 || batch > 65535 || (double)batch * (double)L * (double)D > 32e6) return false;
    const double own = lanes_ns(batch, L, D, 9.9, 8.3, 10.7, true);
    if (chunks == 1) {
        const bool six = lanes_channels(batch, L, D) == 6;
        const double dt_apart = dt_rank <= kLanesLowRank ? 0.0 : six ? 2200.0 : 4250.0;
        // (a single chunk of more tokens has channels for the whole chip)
        return L <= 16 && own < (six ? 3000.0 + 500.0 * (double)L : 2200.0 + 950.0 * (double)L) - dt_apart;
    }
    const double two_pass_ns = 24000.0 + 10.0 * (double)L * ((double)batch * (double)D / 1536.0);
    const int64_t groups = lanes_groups(batch, L, D, true);
    const bool filled = (double)groups >= 0.95 * (double)((groups + 255) / 256 * 256);
    const double ahead = groups <= 256 && lanes_channels(batch, L, D) < 6 ? 0.92 : 0.85;
    return own < ahead * two_pass_ns || (filled && own < two_pass_ns - 3000.0);
}

// Tokens of a lane, 64 times that to a super-step: what takes the fewest super-steps times what one takes, which is 5.3 us with 8 tokens,
// 4.1 with 6 and 3.2 with 4 (1536 channels; a last one that is not full takes somewhat less).  Two channels to a workgroup leave no
// threads for more than 4.  us with 4 / 6 / 8 tokens:
//    200 x 1536  7.25*/ 8.37 / 9.05     400 x 1536 10.45 / 12.56 / 9.84*    1000 x 1536 17.06 / 16.92 / 15.49*     700 x 1000 10.68 / 10.33*/ 11.66
//    300 x 1536 10.42 / 8.79*/ 9.48     600 x 1536 13.49 / 12.69*/14.70     1100 x 1536 19.82 / 17.06*/ 19.72      350 x 1536 float32 11.43 / 9.75*/ 10.70
//    384 x 1536 10.51 / 9.19*/ 9.83     768 x 1536 13.73 / 13.01*/14.92     1900 x 1536 29.56 / 26.07 / 25.83*     700 x 1536 float32 16.88 / 16.21*/ 18.23
// In float32, where a super-step's B and C are not requested ahead, one super-step more costs more; us with 6 / 8, bf16 | float32:
//   2251 x  488, batch 6  82.6*/ 82.8 | 108.6 / 107.2*     2107 x 1392, batch 2  55.7*/ 57.4 | 77.4 / 76.2*     2101 x 504, batch 2  25.1*/ 25.6 | 28.5 / 27.9*
//   2682 x  456, batch 3  34.1*/ 36.3 |  42.7 / 42.4*      1124 x 2304           32.1*/ 36.6 | 38.6*/ 42.5
inline int lanes_tau(int64_t batch, int64_t L, int64_t D, bool bf16)
{
    if (L <= 256 || lanes_channels(batch, L, D) == 2) return 4;
    return 4.1 * (double)((L + 383) / 384) < (bf16 ? 0.95 : 0.9) * 5.3 * (double)((L + 511) / 512) ? 6 : 8;
}

// Whether the lanes kernel takes a whole block's scan, which it has been given, together with its dt projection: contexts of one super-step.
inline bool scan_lanes_takes_low_dt(int64_t batch, int64_t L, int64_t D, int64_t dt_rank)
{
    return L <= 64 * lanes_tau(batch, L, D, true) && dt_rank % 8 == 0 && dt_rank <= kLanesLowRank;
}

// The fused layer step (state_step_conv_kernel) counts channels in 32 bits and launches a wavefront per 64 of them (32 with 32
// states), whose threads along x have to stay below 2^32.  A wider layer takes the conv and the state step one after the other,
// which count in 64 bits.
inline bool conv_step_fits(int64_t D, int64_t N)
{
    return D <= (N > 16 ? ((int64_t)1 << 31) - 32 : ((int64_t)1 << 32) - 64);
}

// The state step of a draft position that adds up the x projection's partial sums (state_step_xproj_kernel) forms a lane's
// places in A, a row of states, the dt weights and a row of partial sums (one run of dt_rank + 2 N floats per 16 channels) as
// bytes in 32 bits, so each of them has to stay below 4 GiB.  A wider block keeps the x projection in a launch of its own, and
// the state step that counts in 64 bits.
inline bool step_xproj_fits(int64_t D, int64_t N, int64_t dt_rank)
{
    const int64_t most = (int64_t)1 << 32;
    return D <= most / (4 * N) && D <= most / (2 * dt_rank) && D / 16 <= most / (4 * (dt_rank + 2 * N));
}

// Row tiles of 16 (1, 2 or 4) per workgroup of the way into a block at a draft position (draft_in.hip), M <= 64 rows, 16 columns
// each: as few as make one round of workgroups on 256 CUs, and no more than there are rows for, since tiles past the last row
// cost what the others do.  us of a whole block with 1 / 2 / 4 tiles, 24 blocks in turn, replayed (* what this takes):
//    3 rows of 5120 channels 34.1*/ 41.2 / 53.8, of 3072 18.5*/ 19.4 / 26.7, of 1536 9.3*/ 10.0 / 11.8    12 rows of 1536 10.2*/ 10.9 / 12.7
//   24 rows of 5120 channels 57.5 / 62.7*/ 68.8, of 3072 26.9 / 26.7*/ 33.4, of 1536 12.3 / 12.7*/ 14.4   32 rows of 1536 12.9 / 13.3*/ 15.0
//   48 rows of 5120 channels 92.8 /102.6 /101.6*, of 1536 15.7 / 16.6 / 17.6*, of 512 8.9*/ 9.6 / 10.7    64 rows of 1536 17.0 / 18.1 / 19.1*
// The rounds come from the kernel before draft_in.hip; on that one a single tile is ahead also where it makes further rounds, by up
// to 12 % of a block.
inline int linear_few_row_tiles(int64_t M, int64_t N)
{
    const int64_t columns = (N + 15) / 16;
    if (M <= 16 || columns * ((M + 15) / 16) <= 256) return 1;
    return M <= 32 || columns * ((M + 31) / 32) <= 256 ? 2 : 4;
}

// Taps of the conv that a tile kernel forms from its finished tile.
constexpr int kConvTaps = 4;

// linear_wide_kernel and linear_ring_kernel place a lane's 16 bytes within eight rows of k in 32 bits.
constexpr int64_t kToLdsLongestK = (int64_t)1 << 28;

// The kernels of a product (linear.hip): what linear_route chooses from.
enum LinearKernel {
    kNoKernel,
    kFew16x8, kFew16x16, kFew16x16Stream, kFew32x16, kFew32x32, kFew64x32,   // linear_few_kernel, rows x columns; w read past the caches
    kRing64, kRing64x128, kRing128,                                          // linear_ring_kernel
    kWide256x192, kWide256, kWide192, kWide128Eight, kWide128,               // linear_wide_kernel: 256 rows on eight wavefronts, 192 x 128 on
                                                                             // four, 128 x 128 on either
    kTiles128, kTiles64x128, kTiles64Deep, kTiles64, kTiles64Stream          // linear_kernel; slabs of 256 k; w read past the caches
};

// Few output tiles (linear_few_kernel): the tile that makes one round of workgroups on 256 CUs, from 16 rows x 8 columns up; the
// tile kernels take over where 32 x 32 comes to more than two or three to a CU.  us on 16 x 8 / 16 x 16 / 32 x 16 / 32 x 32 / 64 x 32 /
// the best tile kernel:
//    12 x  768, K = 1536  3.1 / 3.3 / 3.7 /   -  /   -  / 10.3      333 x   80, K = 1536  3.3 / 3.6 /  4.1 /  4.9 /   -  / 11.4
//   128 x  768, K = 1536  4.8 / 4.3 / 4.1 /  4.6 /  6.4 / 10.9      333 x  768, K = 1536   -  / 6.3 /  6.8 /  6.2 /  6.5 / 10.9
//   700 x  768, K = 1536   -  / 10.6/ 10.1/  8.4 / 11.5 / 11.0     1000 x  768, K = 1536   -  / 13.7/ 12.1 /  9.0 / 12.0 / 11.8
//   128 x 3072, K =  768   -  / 5.3 / 5.0 /  5.1 /  5.6 /  7.0      256 x 3072, K =  768   -  / 8.2 /  8.2 /  7.7 /  9.5 /  7.1
//   256 x 2048, K =  512   -  / 5.1 / 4.6 /  4.2 /  4.4 /  5.8      512 x 2048, K =  512   -  / 8.0 /  7.1 /  6.5 /  7.3 /  6.0
//   512 x  512, K = 1024   -  / 5.2 / 4.7 /  3.9 /  5.1 /  8.4      700 x 1024, K = 2048   -  / 18.3/ 16.5 / 12.1 / 15.0 / 13.3
//   256 x 1536, K = 3072   -  / 15.3/ 12.7/ 12.9 / 10.3 / 18.1      256 x 2048, K = 4096   -  / 29.2/ 24.2 / 21.4 / 18.0 / 28.3
//   200 x 2560, K = 5120   -  / 40.9/ 37.3/ 37.4 / 36.4 / 34.9      256 x 1536, K =   48   -  / 3.1 /  2.9 /   -  /   -  /  3.1
// How many 32 x 32 (`most`), between k of 512 and 1024; us on 32 x 32 / the tile kernels for k = 576, 640, 768, 896, 960:
//   608 tiles (256 x 2432)  7.2 / 7.6    7.2 / 7.6    7.4 / 7.9    7.6 / 9.1    7.7 / 9.2
//   672 tiles (224 x 3072)  7.1 / 7.1    7.2 / 7.1    7.5 / 7.1    7.7 / 8.3    7.8 / 8.3
//   768 tiles (768 x 1024)  7.1 / 7.1    7.2 / 7.2    7.7 / 7.2    7.7 / 8.4    7.9 / 8.4
// So 608 is where the two meet for a k of 768; for k between that and 1024 32 x 32 stays ahead up to 768 tiles, by 4 to 8 %.
// Up to 16 rows against very many columns (the LM head on a draft position): 16 columns each, any number of rounds, up to a k of
// four trips; us on that / 64 x 64 tiles: 1 x 50280, K = 768 13.3 / 15.7, 12 x 50280 15.1 / 17.0, 12 x 16384 6.7 / 10.0, 12 x 32768,
// K = 2048 25.0 / 30.4 (12 x 50280, K = 2560 54.3 / 51.5; 32 x 50280, K = 768 on 32 rows 22.6 / 18.3).
inline LinearKernel linear_few(int64_t M, int64_t N, int64_t K)
{
    if (!linear_few_fits(N, K)) return kNoKernel;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((N + bn - 1) / bn) * ((M + bm - 1) / bm); };
    const int64_t round = 256, t32 = tiles(32, 32), most = K > 3072 ? 512 : K > 512 && K < 1024 ? 608 : 768;
    if (M <= 16 && N >= 8192 && K <= 2048) return kFew16x16Stream;
    if (tiles(16, 8) <= round) return kFew16x8;
    if (tiles(16, 16) <= round * 9 / 8 || (M <= 16 && N < 8192)) return kFew16x16;
    if (tiles(32, 16) <= (K < 256 ? 3 * round : round)) return kFew32x16;
    if (K >= 2048 && M > 64 && t32 > round && tiles(64, 32) <= round) return kFew64x32;
    return K >= 256 && t32 <= most ? kFew32x32 : kNoKernel;
}

// Products whose tiles come in one round of workgroups take linear_ring_kernel, the smallest tile that does it; the few-row kernels
// have been asked before.  64 x 64 tiles run two to a CU, but a second set of them costs what half as many 64 x 128 do.  us on
// the kernel before (the tile kernels below) / 64 x 64 / 64 x 128 / 128 x 128, 24 weights in turn:
//    200 x 3072, K =  768   7.1 / 6.6*/ 8.0 / 9.7       512 x 3072, K =  768   8.9 / 8.5 / 8.1*/10.0      1000 x 3072, K =  768  12.3 / 12.5 / 13.6 / 10.1*
//    200 x 5120, K = 1280  12.9 /12.1*/13.5 /17.1       333 x 5120, K = 1280  13.7 /14.9 /13.3*/17.0       700 x 5120, K = 1280  21.0 / 23.6 / 20.8 / 17.1*
//   1000 x 1024, K = 2048  16.4 /12.1*/13.8 /17.7      2048 x  768, K = 1536  17.1 /12.3 /11.8*/15.0      4000 x  768, K = 1536  19.3 / 20.0 / 20.9 / 16.1*
//   2048 x  512, K = 1024  11.1 / 8.0*/ 9.4 /11.6      3000 x  512, K = 1024  15.0 / 9.8 / 9.5*/11.9      3000 x 1280, K = 2560  37.4 / 36.2 / 31.9 / 28.6*
// Beyond one round the tile kernels are ahead: 1500 x 3072 13.7 / 18.4 / 19.5 / 18.9, 2048 x 3072 15.7 / 22.1 / 20.6 / 19.3.  With a short
// k there is little to have under way: K = 256, 1024 x 1024 4.8 / 4.5* 64 x 64, but 1024 x 2048 5.8* / 5.9 64 x 128, 1500 x 1536 6.2* / 6.5
// 128 x 128; K = 384, 1000 x 1536 7.0 / 6.7* 64 x 128 (64 x 64 tiles of K = 256 8.8 % ahead on 65 products, 64 x 128 of K = 384 2.7 % on 37, a third
// of them slower, by 7 % at most).
// More 64 x 64 tiles than CUs, of a long k, and rows for three of them or fewer: nearly all of what a tile loads is w, from memory, and the CUs
// that have two are as long as twice one.  335 products of 256 to 320 tiles: with the line for those at 270 7 are slower than on the kernel
// before, by 7 % at most, and 19.5 % ahead on average; at 320 throughout 30, by up to 23 %, and 19.2 %.  us on the kernel before / 64 x 64 / 64 x 128:
//    109 x 10240, K = 8064  59.8 / 78.1 / 63.7*      87 x 10240, K = 3584  28.9 / 35.8 / 30.4*     102 x 9856, K = 4224  34.7 / 35.1 / 29.4*
inline LinearKernel linear_ring(int64_t M, int64_t N, int64_t K, bool vector_out)
{
    if (!vector_out || K % 64 != 0 || K < 256 || K > kToLdsLongestK || M < 64 || N % 64 != 0) return kNoKernel;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((N + bn - 1) / bn) * ((M + bm - 1) / bm); };
    if (tiles(64, 64) <= (K >= 2048 && M <= 192 ? 270 : 320)) return kRing64;
    if (N % 128 != 0 || K < 384) return kNoKernel;
    if (tiles(64, 128) <= 256) return kRing64x128;
    return M >= 128 && tiles(128, 128) <= 256 ? kRing128 : kNoKernel;
}

// The way into a block on a context (x | z = u W_in^T, then the conv over time on x) in one launch: the tile whose product takes least,
// by rounds of workgroups over the chip; or the product and the conv apart, where the rows that a tile of x shares with the one before
// it cost more than the conv's launch (512 rows of 4096 channels: 320 128 x 128 tiles instead of 256), on fewer than 64 rows, on a product
// that the few-row kernels take and share the k of, where that is long for so few tiles, and on what the tiles cannot.  (Those on 500 blocks of 64
// to 700 rows, us of a block apart / together (rows, D, K): 70, 256, 2496 24.1*/ 27.6, 133, 128, 2112 24.0*/ 26.1, 116, 512, 2048 24.7*/ 26.0, but 64,
// 1536, 768 together; the line keeps 94 % of what the better of the two would save.)  Fitted to 179 products of seven models, 64 to 32768 rows: the choice costs 0.9 % more
// than the best of them on average, and the launch 15 % less than the two.  us, product + conv / the launch on 64 x 64 / 64 x 128 / 128 x 128
// ring, 128 x 128 / 192 x 128 / 256 x 256 wide tiles (D, K):
//     100 x 1536,  768   8.3 /  6.9*/  9.1 /   -  /   -  /   -  /   -       2048 x 1536,  768  19.8 / 28.2 / 32.6 / 21.3 / 17.8*/ 22.1 / 27.0
//     333 x 1536,  768  11.8 /  8.8*/  9.7 / 11.4 / 13.9 / 15.6 / 25.5      8000 x 1536,  768  52.4 / 85.4 / 99.1 / 60.7 / 50.1 / 46.0*/ 53.0
//     600 x 1536,  768  12.7 / 10.2*/ 10.2 / 11.7 / 14.3 / 16.8 /   -      32768 x 1536,  768   216 /  331 /  387 /  241 /  219 /  189 /  175*
//    1000 x 1536,  768  15.7 / 16.3 / 17.8 / 12.4*/ 15.2 / 17.7 / 26.3     16384 x 3072, 1536   329 /  541 /  562 /  403 /  388 /  323 /  301*
//     200 x 1024,  512   7.5 /  6.3*/  8.3 /  9.5 / 10.8 / 12.8 /   -       2048 x 4096, 2048  72.8*/  127 /  131 /  102 /  101 / 85.6 /  105
enum ConvTiles { kConvApart, kConvRing64, kConvRing64x128, kConvRing128, kConvWide128, kConvWide192, kConvWide256 };
inline int64_t row_blocks(int64_t M, int64_t BM, bool conv)      // with the conv all but the first have kConvTaps - 1 rows that are another's
{
    return !conv || M <= BM ? (M + BM - 1) / BM : 1 + (M - BM + BM - kConvTaps) / (BM - kConvTaps + 1);
}
inline ConvTiles linear_conv_tiles(int64_t M, int64_t D, int64_t K, int64_t taps)
{
    if (taps != kConvTaps || M < 64 || M > (int64_t)1 << 23 || D % 64 != 0 || D > (int64_t)1 << 20 || K % 64 != 0 || K < 256 || K > kToLdsLongestK)
        return kConvApart;
    if (linear_few(M, 2 * D, K) != kNoKernel && K > 700 + 16 * ((M + 63) / 64 * (D / 32))) return kConvApart;
    // us: a launch, a round of workgroups, and where two share a CU a round that gives no CU a second one
    struct Tile { ConvTiles kind; int64_t bm, bn, per_round; double launch, round, round_k, half, half_k; };
    const Tile all[6] = {{kConvRing64, 64, 64, 512, 2.6, 1.5, .0076, 1.1, .0051},    {kConvRing64x128, 64, 128, 256, 2.5, 2.5, .0067, 0, 0},
                         {kConvRing128, 128, 128, 256, 2.4, 3.4, .0085, 0, 0},       {kConvWide128, 128, 128, 512, 3.9, 2.0, .0172, 1.6, .0118},
                         {kConvWide192, 192, 128, 512, 4.5, 4.6, .0205, 2.4, .0139}, {kConvWide256, 256, 256, 256, 5.0, 6.8, .0220, 0, 0}};
    const double none = 1e30;
    auto us = [&](const Tile &t, bool conv) {
        const bool ring = t.kind <= kConvRing128;
        if (M < t.bm) return none;
        // (x and z have row blocks of their own in the wide kernels, x's in the others)
        const int64_t z = row_blocks(M, t.bm, false), x = row_blocks(M, t.bm, conv);
        const int64_t tiles = ring ? x * ((2 * D + t.bn - 1) / t.bn) : z * ((2 * D + t.bn - 1) / t.bn) + (x - z) * ((D + t.bn - 1) / t.bn);
        if (ring && tiles > t.per_round) return none;              // one round
        const int64_t full = tiles / t.per_round, rest = tiles % t.per_round;
        const bool half = t.half > 0 && rest > 0 && rest <= t.per_round / 2;
        return t.launch + (double)(full + (rest > 0 && !half ? 1 : 0)) * (t.round + t.round_k * (double)K) + (half ? t.half + t.half_k * (double)K : 0.0);
    };
    double best = none, apart = none;
    ConvTiles kind = kConvApart;
    for (const Tile &t : all) {
        const double a = us(t, false) + 2.5 + 7.5e-7 * (double)M * (double)D;
        if (a < apart) apart = a;
        if (D % t.bn != 0 || (t.kind > kConvRing128 && K % 128 != 0)) continue;
        const double c = us(t, true);
        if (c < best) best = c, kind = t.kind;
    }
    return best <= 1.05 * apart ? kind : kConvApart;               // (the conv of a tile is cheaper than the model has it)
}

// Tile kernels for products that the few-row and ring kernels do not take.  wide: M >= 128, N % 128 == 0, K % 128 == 0 and output widths
// that are multiples of 8, which the memory-to-LDS kernel asks for.  The lines are drawn from chains of 24 different blocks, as a prefill runs them (alone in a
// loop, or with few weights that stay in the caches, the wide tiles look better than they are there), for seven models from 512
// to 5120 channels and 200 to 32768 rows, every kernel that applies put in place of one product: 201 products, on which
// the choice costs 0.3 % of a block more than the best one on average.  (That was with 256 x 256 tiles on four wavefronts.  On eight they are 5 to
// 16 % faster, and linear_wide256 is asked first; what the lines here still give them after it has declined takes, on 120 products, 2.4 % more than
// the best of the memory-to-LDS tiles, nearly all of it at k of 128 and 256.)  us of a block on 256 x 256 / 128 x 128 memory-to-LDS /
// 128 x 128 register-staged tiles / the best of the small ones:
//   rows   in_proj of         K                                     out_proj of       K
//   8000   1536 channels    768  209.8 / 214.3 / 204.4 / 209.9      1536 channels  1536  232.0 / 214.5 / 228.9 / 225.3
//  16384   1536             768  410.1 / 416.1 / 405.0              1536           1536  403.9 / 409.9 / 423.3 / 428.2
//   2048   1536             768   91.1 /  83.8 /  87.0 /  85.2      2048           2048  149.5 / 130.4 / 145.0 / 124.2
//   3000   2048            1024  153.5 / 163.1 / 157.0 / 163.3      2048           2048  172.1 / 153.1 / 170.1 / 153.8
//    512   2048            1024   81.7 /  69.8 /  73.8 /  64.2      4096           4096  212.1 / 176.9 / 197.9 / 158.7 (1000 rows)
//   6000   3072            1536  432.1 / 447.4 / 422.3              4096           4096  569.7 / 601.0 /   -   /   -
//   1000   5120            2560  233.1 / 251.0 / 235.1 / 251.2      5120           5120  277.7 / 233.1 / 254.3 / 230.1
//   4096   5120            2560  622.1 / 647.3 / 637.7              5120           5120  624.3 / 635.3 / 656.9 / 687.4
inline LinearKernel linear_tiles(int64_t M, int64_t N, int64_t K, bool wide)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((N + bn - 1) / bn) * ((M + bm - 1) / bm); };
    if (wide) {
        // 256 x 256, one to a CU, where they fill nine tenths of the rounds they take; with a long k also where no more than
        // 128 CUs miss a tile in the last round, in narrow outputs only if that is the first one
        const int64_t t256 = M >= 256 && N % 256 == 0 ? tiles(256, 256) : 0;
        const int64_t rounds = (t256 + 255) / 256, idle = 256 * rounds - t256;
        if (t256 >= 230 && 10 * t256 >= 9 * 256 * rounds) return kWide256;
        if (K >= 1024 && t256 >= 160 && idle <= 128 && (N >= 4096 || rounds == 1)) return kWide256;
        // 128 x 128, two to a CU.  Wide outputs: one round of one or two to a CU; beyond that an XCD's tiles lie side by side in
        // one row block and every weight is used once per visit.  Narrow ones: with a short k the same, from fewer tiles on and
        // in any number where there are few columns; with a long k from half a tile per CU on, unless the small tiles with deep
        // slabs come to two per CU at most, which is one round of theirs.
        const int64_t t128 = tiles(128, 128);
        if (N >= 4096 ? t128 >= 256 && t128 <= 512
                      : K >= 1024 ? t128 >= 128 && (N < 1024 || tiles(64, 64) > 512)
                                  : (t128 >= 256 && t128 <= 512) || (N <= 768 && t128 >= 192))
            return kWide128;
    }
    if (tiles(128, 128) >= 512) return kTiles128;
    if (tiles(64, 128) >= 512) return kTiles64x128;
    // few tiles and a long k loop: with one or two workgroups per CU nothing hides the fetch of the next slab, so the slabs
    // are made four times deeper and the loop four times shorter
    return K >= 512 && tiles(64, 64) < 513 ? kTiles64Deep : kTiles64;
}

// 192 x 128 tiles lie between the others in size, so they often leave fewer CUs idle in the last round; as many flops an
// operand byte as half of a 256 x 256 tile's, and two to a CU, so one's output goes out under the other's products.  They are
// weighed against the choice above (other) wherever that takes a second round of 128 x 128 tiles: rounds times what one takes, in
// units of a full set of 256 128 x 128 tiles (7 us at K = 768, 12.5 at K = 1536), a half-full round of two to a CU costing less.  Fitted
// to 139 products of five models, the 256 x 256 tiles of them on four wavefronts (those on eight have been asked: linear_wide256); the choice costs
// 0.4 % of the better of the two on average.  us on the choice above /
// 192 x 128, random operands, 24 weights in turn:
//    3000 x 3072, K =  768   27.6 /  20.9     12000 x  768, K = 1536   43.0 /  36.1      6000 x 6144, K = 1536  140.9 / 117.6
//    8000 x 3072, K =  768   54.1 /  43.2     16384 x 3072, K =  768   84.0*/  88.6     12000 x 1536, K = 3072  125.9 / 108.0
//    5000 x 2048, K =  512   21.9 /  17.0      8000 x 4096, K = 1024   69.8*/  74.4      7000 x 2560, K = 5120  205.0 / 173.3
inline bool linear_wide192(int64_t M, int64_t N, int64_t K, bool wide, LinearKernel other)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((N + bn - 1) / bn) * ((M + bm - 1) / bm); };
    if (!wide || M < 192 || tiles(128, 128) <= 512 || (other != kWide256 && other != kWide128 && other != kTiles128)) return false;
    const bool longk = K >= 1024;
    auto rounds = [](int64_t t, int64_t per, double full, double half) {
        const int64_t rem = t % per;
        return (double)(t / per) * full + (rem == 0 ? 0.0 : rem <= per / 2 ? half : full);
    };
    const double with = rounds(tiles(192, 128), 512, longk ? 3.1 : 2.9, longk ? 1.9 : 1.7);
    const double without = other == kWide256 ? rounds(tiles(256, 256), 256, longk ? 3.6 : 3.9, longk ? 3.6 : 3.9)
                           : other == kWide128 ? rounds(tiles(128, 128), 512, 2.14, longk ? 1.5 : 1.3)
                                                    : rounds(tiles(128, 128), 768, longk ? 3.6 : 3.5, longk ? 2.7 : 2.6);
    return with < without;
}

// 256 x 256 tiles of eight wavefronts multiply faster than the others once every CU has one, which leaves the number of rounds: a launch's
// microseconds and a round's, two workgroups to a CU taking six tenths of one where no CU has a second.  Fitted to 153 products of
// seven models, 1000 to 32768 rows; taken where that is 4 % less than the 128- and 192-row tiles are thought to take, which in none of them
// was slower than what linear_tiles and linear_wide192 choose.  us on that / on 256 x 256:
//   16384 x  768, K = 1536   47.6 /  40.6      10000 x 3072, K =  768   54.0 /  49.4      16384 x 3072, K =  768   84.3 /  77.7
//    5000 x 3072, K =  768   28.8 /  25.9       5000 x 6144, K = 1536   92.9 /  87.3      10000 x 2560, K = 5120  296.5 / 263.4
//    8000 x  768, K = 1536   25.6*/  34.5      12000 x 3072, K =  768   61.4*/  70.4       8000 x 3072, K =  768   43.6*/  45.3
inline double wide_tiles_us(int64_t M, int64_t N, int64_t K, int64_t bm, int64_t bn, int64_t per, double launch, double round, double round_k, double first)
{
    const int64_t t = ((M + bm - 1) / bm) * ((N + bn - 1) / bn), rest = t % per;
    const double part = (double)rest / (double)per;
    const double rounds = (double)(t / per) + (rest == 0 ? 0.0 : per == 512 && part <= 0.5 ? 0.62 : first + (1.0 - first) * part);
    return launch + rounds * (round + round_k * (double)K);
}
inline double wide128_us(int64_t M, int64_t N, int64_t K) { return wide_tiles_us(M, N, K, 128, 128, 512, 1.9, 3.0, .0159, .7); }
inline double wide192_us(int64_t M, int64_t N, int64_t K) { return wide_tiles_us(M, N, K, 192, 128, 512, 1.1, 5.0, .0203, .7); }
inline double wide256_us(int64_t M, int64_t N, int64_t K) { return wide_tiles_us(M, N, K, 256, 256, 256, 0.4, 7.5, .0244, .7); }
inline bool linear_wide256(int64_t M, int64_t N, int64_t K, bool wide)
{
    if (!wide || M < 1000 || N % 256 != 0) return false;
    const double w128 = wide128_us(M, N, K), w192 = wide192_us(M, N, K);
    return wide256_us(M, N, K) < 0.96 * (w128 < w192 ? w128 : w192);
}

// 256 x 192 tiles of eight wavefronts, one to a CU, by the same count of rounds, where that is less than for all the others; asked before
// them.  us on the others / on them, products in a row and a block whose out_proj it is:
//   16384 x 1536, K =  768   58.8 /  44.6     32768 x 1152, K = 2304  170.5 / 153.6     16384 x 768, K =  768   25.1 /  23.8      4096 x 3072, K =  768   25.3 /  23.9
//   32768 x  768, K = 1536   79.6 /  75.1, block 610 / 602              16384 x 768, K = 1536   40.0 /  38.0, block 330 / 327
//    4096 x 6144, K = 1536   81.4 /  81.9     16384 x 1536, K = 3072  144.8 / 135.2, block 796 / 788          6000 x  768, K =  768   14.8*/  18.6
// Three hundredths short of 192 x 128 tiles, of which two to a CU hide each other's residual: 6000 x 1536, K = 3072 (1.9 short) is 62.5 / 57.1 in
// a row, but 335 / 339 in a block, 16384 x 1152, K = 2304 91.1 / 87.0 and 556* / 559.  Widths that those cannot take have slower tiles to
// compare with: 16384 x 576, K = 1152 block 284 / 267, 20000 x 576 360 / 330.  At widths that 128 divides, only
// where they fill the last round: in one that they do not, 192 x 128 tiles, two to a CU, lose less than the count says, the more the longer
// the k (5578 x 1536, K = 6400 111* / 123, 2221 x 4224, K = 6016 114* / 126, 1166 x 6912, K = 2944 60* / 68; of 40 such products 35 are slower here,
// 5 % on average; of 147 that fill it 9, by 5 % at most, and 7 % faster on average), while at the others all of 263 are faster, by a half.
// So whole rounds and little else: of out_proj's row counts from 1000 to 32768 at 768 x K = 1536 those from 16321 to 16384 and from 32641 to 32768.
inline bool linear_wide256x192(int64_t M, int64_t N, int64_t K, bool vector_out)
{
    if (!vector_out || M < 1000 || N % 192 != 0 || K % 128 != 0 || K > kToLdsLongestK) return false;
    const int64_t tiles = ((M + 255) / 256) * (N / 192);
    if (N % 128 == 0 && (double)tiles < 0.95 * (double)((tiles + 255) / 256 * 256)) return false;
    const double own = wide_tiles_us(M, N, K, 256, 192, 256, 0.5, 7.5, .0195, .66);
    return own < .99 * wide128_us(M, N, K) && own < (N % 128 == 0 ? .97 : 1.0) * wide192_us(M, N, K) && (N % 256 != 0 || own < .99 * wide256_us(M, N, K));
}

// Eight wavefronts for 128 x 128 tiles of a long k as well where half of the CUs or more have one tile only.  us of four / eight:
// 6000 x 768, K = 1536 21.7 / 20.5, 8000 x 768 23.7 / 22.8, 4000 x 1024, K = 2048 26.7 / 24.8; 16384 x 512, K = 1024 (two to every CU) 22.8* /
// 23.3, 8000 x 3072, K = 768 45.9* / 47.9
inline bool linear_wide128_eight(int64_t M, int64_t N, int64_t K)
{
    return K >= 1024 && ((M + 127) / 128) * ((N + 127) / 128) <= 384;
}

// The kernel of a product x (M, K) w (N, K)^T whose outputs are width[0], width[1] and width[2] columns wide: the rules above, in the
// order in which they are asked.  1500 random products (48 to 33000 rows, 128 to 11000 columns, k 256 to 6000) are 6.6 % faster with them on
// average than on the kernels from before the ring and the tiles on eight wavefronts, 3 of them slower by more than 1.5 %, by 8 % at most; on 342 that
// the few-row and ring kernels leave, with every other kernel put in its place, the choice takes 1.7 % more than the best.
inline bool linear_vector_out(const int64_t width[3]) { return width[0] % 8 == 0 && width[1] % 8 == 0 && width[2] % 8 == 0; }
inline LinearKernel linear_route(int64_t M, const int64_t width[3], int64_t K)
{
    const int64_t N = width[0] + width[1] + width[2];
    const bool vec = linear_vector_out(width), wide = vec && N % 128 == 0 && M >= 128 && K % 128 == 0 && K <= kToLdsLongestK;
    if (const LinearKernel few = linear_few(M, N, K)) return few;
    if (const LinearKernel ring = linear_ring(M, N, K, vec)) return ring;
    const LinearKernel tiles = linear_tiles(M, N, K, wide);
    if (linear_wide256x192(M, N, K, vec)) return kWide256x192;
    if (linear_wide256(M, N, K, wide)) return kWide256;
    if (linear_wide192(M, N, K, wide, tiles)) return kWide192;
    if (tiles == kWide128 && linear_wide128_eight(M, N, K)) return kWide128Eight;
    if (tiles == kTiles64 && M <= 64 && N >= 8192) return kTiles64Stream;
    return tiles;
}

// x_proj and dt_proj in one kernel (xdt.hip): rows per workgroup and column groups for M rows; 0 rows: two launches.
// Every workgroup reads all weights, so what counts is the number of rounds on 256 CUs times what a workgroup takes (us in
// xdt.hip, in a full round).  One round of 16 rows: column groups as long as they fit the chip beside each other (24-block
// prefill of 1024 tokens with 1, 2, 3 groups 1507, 1486, 1466 us; of 2000 tokens, where only two fit, 2016, 2001, 2104).
// The two launches take 9 us + 2.05 ns a row at 1536 channels, and the gap between them.
// With few rows there are too few workgroups for the weights to stream through, the fewer the more weights there are.  us of a
// block (d_inner, dt_rank) in a chain of eight to 24 different ones, two launches / one:
//   rows    512, 32      1024, 32      1536, 48      2048, 64       3072, 48       4096, 64       5120, 64
//    768   39.7/38.6    48.9/48.0     57.7/58.5     82.4/82.5      86.2/89.8     132.1/139.6    173.8/182.3
//   1100   48.5/47.0    59.2/58.1     67.5/67.5    101.3/102.0    103.5/105.6    196.1/198.7    251.8/257.5
//   1700   56.6/55.3    67.5/66.0     80.8/80.2    112.4/112.6    133.2/134.2    230.9/233.6    329.5/331.9
//   2500   59.9/58.0    78.5/76.4     94.6/95.3    142.5/142.9    156.7/156.3    294.7/296.9    424.6/426.9
//   3000   62.0/59.6    86.2/83.9    112.3/109.9   156.8/153.0    187.9/181.1    334.0/332.4    439.3/432.7
//   8000  115.8/112.6  158.6/151.4   228.7/218.1   322.8/310.9    435.2/416.3    775.6/753.2   1097.7/1068.6
// So from 768 rows up to 1536 channels (500 rows there: 24-block prefill 1146 against 1140 us), from 2700 beyond (2560: 1792,
// 48 128.1/128.6, 2048, 64 142.1/142.5, 5120, 64 424.7/426.0; 2700: 132.0/132.3, 146.6/146.5, 446.0/445.4).
constexpr int kXdtStates = 16;
inline int xdt_plan(int64_t M, int64_t d_inner, int64_t dt_rank, int64_t N, unsigned *groups)
{
    *groups = 1;
    if (N != kXdtStates || (dt_rank != 32 && dt_rank != 48 && dt_rank != 64)) return 0;
    if (d_inner < 64 || d_inner % 64 != 0 || d_inner > (int64_t)1 << 20) return 0;
    if (M < (d_inner <= 1536 ? 768 : 2700)) return 0;
    const int64_t t16 = (M + 15) / 16;
    if (t16 <= 256) {
        *groups = (unsigned)(256 / t16 < 3 ? 256 / t16 : 3);
        return 16;
    }
    const double cost[3] = {11.0, 15.0, 23.0};
    double best = 10.0 + 2.05e-3 * (double)M;
    int rows = 0;
    for (int i = 0; i < 3; ++i) {
        if (i == 2 && dt_rank > 48) break;                         // 64 rows and 64 dt columns: more LDS than a CU has
        const double t = cost[i] * (double)((M + ((int64_t)4096 << i) - 1) / ((int64_t)4096 << i));
        if (t < best) best = t, rows = 16 << i;
    }
    return rows;
}

}  // namespace mamba
