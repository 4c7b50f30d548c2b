// Algorithm 1 of the paper in its own order, for small sequences (an evaluation aid beside the block-level path):
//   k_token_scores     proxy score of every token pair (Eq. 9, fused-head mean of App. B) -> fp32 [N, N]
//   k_link_*, k_pair_links_small  per ordered frame pair (i, j): candidate window (Eq. 7), population mean / std of the scores in
//                      it (Eq. 10), z >= tau_1 / tau_2 by decay state (Eq. 11), keep-one safeguard -> link bytes [N, N]
//   k_aggregate_links  density rule per block pair ("Density control within blocks": a column is active when its
//                      kept-row ratio exceeds theta_c, the block when its active-column ratio exceeds theta_m), plus the
//                      never-pruned t <= 1 zone -> keep bitmaps, which the ordinary CSR emit turns into the mask.
// Definition of the statistics (part of the result, so that masks are bit-exact): fp64; every sum runs column by
// column (query index u ascending inside key column v), then over the column sums with v ascending, one by one, with
// no fused multiply-add.  That order is also the coalesced one: a thread owns a key column, neighbouring threads read
// neighbouring addresses.  gfx950 only.
#include "dr_internal.h"

namespace dr {
namespace {

constexpr int kThreads = 256;

// Four consecutive channels of a row (the row's start need not be aligned).
template <bool BF16>
__device__ __forceinline__ float4 load_channels(const void* base, int64_t at) {
    float4 x;
    if constexpr (BF16) {
        uint16_t u[4];
        __builtin_memcpy(u, reinterpret_cast<const uint16_t*>(base) + at, 8);
        x = make_float4(__uint_as_float((uint32_t)u[0] << 16), __uint_as_float((uint32_t)u[1] << 16),
                        __uint_as_float((uint32_t)u[2] << 16), __uint_as_float((uint32_t)u[3] << 16));
    } else {
        __builtin_memcpy(&x, reinterpret_cast<const float*>(base) + at, 16);
    }
    return x;
}

// scores[b][m][p][q] on the fp32 matrix instruction (fp32 products and sums).  2 x 2 wavefronts of 32 x 32 outputs; 32 channels
// of 64 rows of either operand are staged through LDS, the next 32 on their way in registers.  A lane reads four
// consecutive channels of its row and feeds one to each of four instructions: the order of the contraction is permuted alike
// for both operands.  Bound by latency at the sizes of the search (1024 workgroups of four steps at 2048 tokens x 2 heads of 64
// channels); a 4 x 4-per-thread product on the vector ALU with four-byte loads took 49 us there, this takes 16.7.
// grid: (ceil(N / 64), ceil(N / 64), B * masks).
constexpr int kTile = 64, kChunk = 32, kPitch = 36;      // row pitch 144 B keeps the 16-byte reads of 32 rows off the same banks
typedef float v16f __attribute__((ext_vector_type(16)));

template <bool BF16>
__global__ __launch_bounds__(kThreads) void k_token_scores(const void* __restrict__ Q, const void* __restrict__ K,
                                                           TensorDesc td, int masks, int heads_per_mask,
                                                           float scale, float* __restrict__ scores) {
    __shared__ __attribute__((aligned(16))) float sq[kTile][kPitch];
    __shared__ __attribute__((aligned(16))) float sk[kTile][kPitch];
    const int b = blockIdx.z / masks, m = blockIdx.z % masks;
    const int p0 = blockIdx.y * kTile, q0 = blockIdx.x * kTile;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, half = lane >> 5;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const int chunks = td.d / kChunk, steps = heads_per_mask * chunks;
    const int row = tid >> 3, c4 = (tid & 7) * 4;            // of the first 32 rows; the thread takes row + 32 as well
    float4 xq[2], xk[2];
    auto fetch = [&](int step) {
        const int h = (masks == 1 ? 0 : m) + step / chunks;
        const int64_t at = (int64_t)b * td.stride_b + (int64_t)h * td.stride_h + (step % chunks) * kChunk + c4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {                        // rows past the end are read again from the last one
            xq[i] = load_channels<BF16>(Q, at + (int64_t)min(p0 + row + 32 * i, td.N - 1) * td.stride_n);
            xk[i] = load_channels<BF16>(K, at + (int64_t)min(q0 + row + 32 * i, td.N - 1) * td.stride_n);
        }
    };
    fetch(0);
    for (int step = 0; step < steps; ++step) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<float4*>(&sq[row + 32 * i][c4]) = xq[i];
            *reinterpret_cast<float4*>(&sk[row + 32 * i][c4]) = xk[i];
        }
        __syncthreads();
        if (step + 1 < steps) fetch(step + 1);
#pragma unroll
        for (int g8 = 0; g8 < kChunk; g8 += 8) {
            const float4 a = *reinterpret_cast<const float4*>(&sq[wr + l32][g8 + 4 * half]);
            const float4 bb = *reinterpret_cast<const float4*>(&sk[wc + l32][g8 + 4 * half]);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, bb.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, bb.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, bb.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, bb.w, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // element e of lane (l32, half): row 8 * (e / 4) + 4 * half + e % 4, column l32
    float* out = scores + (int64_t)blockIdx.z * td.N * td.N;
    const int q = q0 + wc + l32;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int p = p0 + wr + 8 * (e >> 2) + 4 * half + (e & 3);
        if (p < td.N && q < td.N) out[(int64_t)p * td.N + q] = acc[e] * scale;
    }
}

#pragma clang fp contract(off)

// ---- links of every ordered frame pair, in three launches.  What bounds this is the serial fp64 chain of a column (the order of
// the sums is part of the definition) and three readings of the score matrix, so the columns of all pairs are spread over the
// whole chip: a workgroup owns 64 key columns of one pair and reads whole row segments, many rows in flight.
//   k_link_sums<0>  column sums of the scores, highest score
//   k_link_sums<1>  column sums of the squared deviations; the last workgroup of a pair then forms its deviation, the test as one
//                   float and the pair that the safeguard keeps (from the columns' highest scores)
//   k_link_blocks   link bytes, and the density rule over them while they are at hand
struct PairStat {
    float threshold;              // a pair is a link when its score is at least this; NaN: none is
    int best;                     // where nothing passes: u * Nt + v of the highest score, which is kept; else -1
};

__device__ __forceinline__ uint32_t score_image(float s) {      // ascending unsigned == ascending float, -0 below +0
    const uint32_t u = __float_as_uint(s);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float image_score(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u); }

// Rank of a candidate for the safeguard: the highest score, the first in row-major order on ties; a NaN ranks below every number.
__device__ __forceinline__ unsigned long long best_key(float s, int index) {
    const uint32_t image = s == s ? score_image(s + 0.0f) : 0u;
    return ((unsigned long long)image << 32) | (0xffffffffu - (uint32_t)index);
}
__device__ __forceinline__ int best_index(unsigned long long key) { return (int)(0xffffffffu - (uint32_t)key); }

struct PairAt {
    int i, j, t, w, flags;
    int64_t mask, pair;           // (b, m) flattened; index into per-pair arrays
    bool judged;                  // t >= 2 and retained: its links are decided by score
};
// kScalar: the flags come by a scalar load of their word (of a byte there is none), ahead of all else; k_link_sums gains 0.3 % by it,
// k_pair_links_small, which has other work meanwhile, loses 2 to 5 %.
template <bool kScalar>
__device__ __forceinline__ PairAt pair_at(const FrameTab& tab, int Nf, int pair) {
    PairAt p;
    p.i = pair / Nf;
    p.j = pair % Nf;
    p.t = abs(p.i - p.j);
    if constexpr (kScalar) {
        uint32_t word;
        __builtin_memcpy(&word, tab.flags + (p.t & ~3), 4);
        p.flags = (int)(word >> (8 * (p.t & 3))) & 255;
    } else {
        p.flags = tab.flags[p.t];
    }
    p.w = tab.w[p.t];
    p.mask = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    p.pair = p.mask * Nf * Nf + pair;
    p.judged = p.t > 1 && (p.flags & 1);
    return p;
}

// The sum of Nt doubles, one by one in ascending order.  lay_out (all threads of the workgroup, a barrier behind it) puts them into LDS,
// up to a multiple of 16; ordered_sum is one wavefront's.  The next sixteen are read while the current ones are added: the
// chain waits for the additions alone (2.4 ns each).  (Every wavefront for itself: the reads of three workgroups fill a
// compute unit's LDS, 52 us a launch at 8 x 1024 tokens.)
template <bool kSameLaunch, int kSumThreads, class Meanwhile>      // whether other workgroups of this launch wrote them; what to do while they are on their way
__device__ __forceinline__ void lay_out(const double* col, int Nt, double* sh, Meanwhile&& meanwhile) {
    const int padded = (Nt + 15) & ~15;
    for (int v0 = threadIdx.x; v0 < padded || v0 == (int)threadIdx.x; v0 += kSumThreads * 4) {
        double x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double* at = col + min(v0 + kSumThreads * e, Nt - 1);
            x[e] = kSameLaunch ? __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *at;
        }
        if (v0 == (int)threadIdx.x) meanwhile();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = v0 + kSumThreads * e;
            if (v < padded) sh[v] = v < Nt ? x[e] : -0.0;         // (x + -0.0 is x, bit for bit)
        }
    }
}
__device__ __forceinline__ double ordered_sum(int Nt, const double* sh) {
    const int padded = (Nt + 15) & ~15;
    double total = 0.0, x[2][16];
    auto read = [&](double (&dst)[16], int v) {
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[e] = sh[v + e];
        __builtin_amdgcn_sched_barrier(0);
    };
    auto add = [&](const double (&src)[16]) {
#pragma unroll
        for (int e = 0; e < 16; ++e) total = total + src[e];
        __builtin_amdgcn_sched_barrier(0);
    };
    read(x[0], 0);
    int v = 16;
    for (; v + 16 < padded; v += 32) {
        read(x[1], v);
        add(x[0]);
        read(x[0], v + 16);
        add(x[1]);
    }
    if (v < padded) {
        read(x[1], v);
        add(x[0]);
        add(x[1]);
    } else {
        add(x[0]);
    }
    return total;
}
// token pairs of a candidate set: Nt of one place each, and Nt - k at distance k either way, up to w
__device__ __forceinline__ double window_size(int Nt, int w) {
    const long long m = min(w, Nt - 1);
    return (double)(Nt + 2 * (m * Nt - m * (m + 1) / 2));
}

__device__ __forceinline__ float highest(const float* __restrict__ tops, int Nt) {      // (one wavefront)
    const int lane = threadIdx.x & 63;
    float top = __builtin_nanf("");
    for (int v0 = lane; v0 < Nt; v0 += 64 * 16) {
        float x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = tops[min(v0 + 64 * e, Nt - 1)];
#pragma unroll
        for (int e = 0; e < 16; ++e) top = fmaxf(top, x[e]);
    }
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
    return top;
}
constexpr int kRun = 16;                  // rows of a run: what k_link_sums remembers of the place of a column's highest score
__device__ __forceinline__ void set_stats(const float* __restrict__ S, const PairAt& p, int N, int Nt, double mu, double denom, double tau,
                                          float top, const float* __restrict__ tops, const int32_t* __restrict__ rows, PairStat* __restrict__ stats) {
    const int lane = threadIdx.x & 63;
    auto passes = [&](float s) { return ((double)s - mu) / denom >= tau; };
    // images lo .. none - 1 are the finite floats; the first that passes lies in [lo, lo + span]
    const uint32_t none = score_image(3.402823466e38f) + 1u;
    uint32_t lo = score_image(-3.402823466e38f), span = none - lo;
    while (span > 0u) {
        const uint32_t step = span / 64u + 1u;                             // lane l asks at lo + l * step
        const uint32_t at = lo + (uint32_t)lane * step;
        const uint64_t yes = __ballot((uint64_t)lane * step < span && passes(image_score(at)));
        // the answer lies behind the last place that fails, up to the first that passes (or the end)
        const int first = yes ? __ffsll((unsigned long long)yes) - 1 : (int)((span - 1u) / step) + 1;
        if (first == 0) break;                                             // lo itself passes
        const uint32_t end = yes ? (uint32_t)first * step : span;
        const uint32_t from = (uint32_t)(first - 1) * step + 1u;
        lo += from;
        span = end - from;
    }
    const float threshold = lo < none ? image_score(lo) : __builtin_nanf("");
    int best = -1;
    if (!(top >= threshold)) {
        // nothing passes: the highest score, the first in row-major order on ties (-0 equals +0; in a set of NaN alone any is).  A lane
        // takes a column that holds it and looks at the run of rows that is known to; a later column counts only by an earlier
        // row.  (Column after column, a row of the wavefront's after the other, cost 0.5 us for each that shares the highest score:
        // scores that depend on their row alone, nothing passing, 8 x 1024 tokens 587 us where this takes 123, 4 x 4096 7412 / 410.)
        int best_u = top == top ? Nt : 0, best_v = 0;
        for (int v0 = lane; v0 < Nt + lane; v0 += 64 * 8) {
            float x[8];
            int first[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] = tops[p.pair * Nt + min(v0 + 64 * e, Nt - 1)];
                first[e] = rows[p.pair * Nt + min(v0 + 64 * e, Nt - 1)];
            }
#pragma unroll 1
            for (int e = 0; e < 8; ++e) {
                const int v = v0 + 64 * e, vc = min(v, Nt - 1);
                const bool asks = v < Nt && x[0] == top && first[0] < best_u;
                const int u0 = first[0];
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    x[k] = x[k + 1];
                    first[k] = first[k + 1];
                }
                if (!__any(asks)) continue;
                const int lo = max(0, vc - p.w), hi = min(Nt - 1, vc + p.w);
                float s[kRun];
#pragma unroll
                for (int k = 0; k < kRun; ++k) s[k] = S[(int64_t)min(max(u0 + k, lo), hi) * N + vc];
                int at = Nt;
#pragma unroll
                for (int k = kRun - 1; k >= 0; --k)
                    if (asks && u0 + k >= lo && u0 + k <= hi && s[k] == top) at = u0 + k;
                int least = at;
                for (int off = 32; off > 0; off >>= 1) least = min(least, __shfl_xor(least, off));
                if (least < best_u) {                                      // the same in every lane
                    best_u = least;
                    best_v = v - lane + __ffsll((unsigned long long)__ballot(at == least)) - 1;
                }
            }
        }
        best = best_u * Nt + best_v;
    }
    if (lane == 0) {
        stats[p.pair].threshold = threshold;
        stats[p.pair].best = best;
    }
}

// grid: (Nf * Nf * ceil(Nt / 64), masks, B).  sums, devs, tops, rows: [B * masks][Nf * Nf][Nt]; a column's highest score
// and the first run of kRun rows that holds it, for the safeguard.
// A column's rows are walked over the union of the workgroup's windows, so that all lanes read one row; a row outside a
// lane's own window adds +0.0, which leaves its running sum bit for bit as it is (it starts at +0.0 and is never -0.0).
// At 8 x 1024 tokens 672 workgroups have work, so a wavefront that did it all alone (one to a SIMD at most) would pay for every
// wait and every instruction one after the other: 20 and 29 us, and 10 for the statistics in a launch of their own.  Only the
// additions have to be serial, so kFeeders wavefronts fetch the rows and lay them out in LDS, kRun rows in turn, and
// one adds up the round before.  Three feeders: 15 us, and 32 with the statistics, of which the two chains of 1024 sums and what they
// wait for take 18; 256 tokens a frame (8 frames) 10.8, 11.8 and 6.4 -> 7.6 and 12.  (More rows on their way, in registers or in
// LDS, up to four rounds: 16 to 18 and 33 to 45.)  Where workgroups wait for a place a feeder each is enough, and more of them
// are in flight: whole calls, alone / three feeders / one, by the number of workgroups, 192: 128 / 98 / 126 us; 384: 335 / 309 / 389;
// 672: 101 / 89 / 104; 880: 61.4 / 54.7 / 57.2; 1344: 70.1 / 68.8 / 70.0; 1680: 102 / 104 / 98; 2024: 78.7 / 77.5 / 72.4; 2394: 120 / 112 / 108;
// 3720: 101 / 111 / 100; 6486: 98.1 / 98.9 / 87.8.  Drawn at six workgroups on each of 256 compute units, as measured: what LDS lets a unit hold of
// three feeders' workgroups is six in pass 0, but four in pass 1 at 1024 tokens a frame and two at 4096, and yet three are faster there (8 frames of
// 2048, 1344 workgroups: 308 / 322 us with three / one, 4 of 4096 x 4 masks, 1536: 1005 / 1083, 10 of 1600, 1800: 321 / 340), while short frames
// would have the line lower (20 of 256, 1304: 65.1 / 63.8, 15 of 512, 1456: 97.9 / 95.2).
// Pass 1: the workgroup that is last of its pair to store its sums forms the pair's statistics (arrivals are counted in the
// `best` of the pair, which pass 0 clears); nobody waits for another.  Pass 0 also clears the kept counts of the mask's rows, to
// which k_link_blocks adds.
constexpr int64_t kSumGrid = 6 * 256;
template <int PASS, int kFeeders>
__global__ __launch_bounds__(64 * (kFeeders + 1)) void k_link_sums(const float* __restrict__ scores, FrameTab tab, int N, int Nt, int Nf, int Sb,
                                                                   double tau_near, double tau_far, double* __restrict__ sums, double* devs,
                                                                   float* __restrict__ tops, int32_t* __restrict__ rows, PairStat* stats,
                                                                   int32_t* __restrict__ counts) {
    constexpr int kSumThreads = 64 * (kFeeders + 1), kRound = kFeeders * kRun;
    extern __shared__ double s_sums[];
    __shared__ float s_rows[2][kRound][64];
    __shared__ float s_top[kFeeders][64];
    __shared__ int s_row[kFeeders][64];
    __shared__ int s_last;
    const int tiles = (Nt + 63) / 64;
    const int pair = blockIdx.x / tiles, v0 = (blockIdx.x % tiles) * 64;
    const PairAt p = pair_at<true>(tab, Nf, pair);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (PASS == 0) {
        for (int r = (int)(blockIdx.x * kSumThreads + threadIdx.x); r < Sb; r += (int)gridDim.x * kSumThreads) counts[p.mask * Sb + r] = 0;
        if (v0 == 0 && threadIdx.x == 0) stats[p.pair].best = 0;
    }
    if (!p.judged) return;
    const int v = v0 + lane, vc = min(v, Nt - 1), v_last = min(v0 + 63, Nt - 1);
    const int lo = max(0, vc - p.w), hi = min(Nt - 1, vc + p.w);
    const int u_first = max(0, v0 - p.w), u_last = min(Nt - 1, v_last + p.w);      // of the workgroup
    const int every_first = max(0, v_last - p.w), every_last = min(Nt - 1, v0 + p.w);      // rows in all its windows
    const int rounds = (u_last - u_first) / kRound + 1;
    const float* S = scores + p.mask * N * N + ((int64_t)p.i * Nt) * N + (int64_t)p.j * Nt;
    // a feeder's rows of a round: u_first + round * kRound + wave * kRun ..  (past the window: its last row again)
    const uint32_t row_bytes = (uint32_t)N * 4u, at_last = (uint32_t)u_last * row_bytes + (uint32_t)vc * 4u;
    uint32_t at = (uint32_t)(u_first + wave * kRun) * row_bytes + (uint32_t)vc * 4u;      // (a frame's rows: below 2^32 bytes)
    float x[kRun];
    auto fetch = [&]() {
#pragma unroll
        for (int e = 0; e < kRun; ++e) x[e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(S) + min(at + (uint32_t)e * row_bytes, at_last));
        at += (uint32_t)kRound * row_bytes;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto first_rows = [&]() {
        if (wave < kFeeders) fetch();
    };
    if constexpr (PASS == 1) lay_out<false, kSumThreads>(sums + p.pair * Nt, Nt, s_sums, first_rows);
    else first_rows();
    double acc = 0.0;
    float top = __builtin_nanf("");
    int row = 0;                                                     // of the first run of rows that holds `top`
    auto feed = [&](int round) {
        const int u0 = u_first + round * kRound + wave * kRun;
        float most = __builtin_nanf("");                             // (fmaxf passes NaN by: it ranks below every number)
        float (*out)[64] = &s_rows[round & 1][wave * kRun];
#pragma unroll
        for (int e = 0; e < kRun; ++e) out[e][lane] = x[e];
        if constexpr (PASS == 0) {
            if (u0 >= every_first && u0 + kRun - 1 <= every_last) {  // the same in every lane
#pragma unroll
                for (int e = 0; e < kRun; ++e) most = fmaxf(most, x[e]);
            } else {
#pragma unroll
                for (int e = 0; e < kRun; ++e) most = fmaxf(most, u0 + e >= lo && u0 + e <= hi ? x[e] : __builtin_nanf(""));      // (hi <= u_last)
            }
            const bool higher = most > top || (top != top && most == most);
            top = higher ? most : top;
            row = higher ? u0 : row;
        }
    };
    double mu = 0.0;                                                 // (of the wavefront that adds)
    auto term = [&](float x) {
        if constexpr (PASS == 0) return (double)x;
        const double dev = (double)x - mu;
        return dev * dev;
    };
    auto add = [&](int round) {
        const float (*in)[64] = s_rows[round & 1];
        float y[2][kRun];
        auto read = [&](int f) {
#pragma unroll
            for (int e = 0; e < kRun; ++e) y[f & 1][e] = in[f * kRun + e][lane];
            __builtin_amdgcn_sched_barrier(0);
        };
        read(0);
#pragma unroll
        for (int f = 0; f < kFeeders; ++f) {
            if (f + 1 < kFeeders) read(f + 1);
            const int u0 = u_first + round * kRound + f * kRun;
            if (u0 >= every_first && u0 + kRun - 1 <= every_last) {  // the same in every lane
#pragma unroll
                for (int e = 0; e < kRun; ++e) acc = acc + term(y[f & 1][e]);
            } else {
#pragma unroll
                for (int e = 0; e < kRun; ++e) {
                    const double t = term(y[f & 1][e]);
                    acc = acc + (u0 + e >= lo && u0 + e <= hi ? t : 0.0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // A round is laid out while the one before it is added, so that a barrier a round is enough.
    if (wave < kFeeders) {
        feed(0);
        fetch();
        __syncthreads();
        for (int round = 0; round < rounds; ++round) {
            if (round + 1 < rounds) feed(round + 1);
            fetch();
            __syncthreads();
        }
    } else {
        __syncthreads();
        if constexpr (PASS == 1) mu = ordered_sum(Nt, s_sums) / window_size(Nt, p.w);
        for (int round = 0; round < rounds; ++round) {
            add(round);
            __syncthreads();
        }
    }
    if constexpr (PASS == 0) {
        if (wave < kFeeders) {
            s_top[wave][lane] = top;
            s_row[wave][lane] = row;
        }
        __syncthreads();
        if (wave != kFeeders || v >= Nt) return;
#pragma unroll
        for (int f = 0; f < kFeeders; ++f) {
            const float t = s_top[f][lane];
            const int r = s_row[f][lane];
            const bool higher = t > top || (top != top && t == t);
            row = higher || (t == top && r < row) ? r : row;
            top = higher ? t : top;
        }
        sums[p.pair * Nt + v] = acc;
        tops[p.pair * Nt + v] = top;
        rows[p.pair * Nt + v] = row;
    } else {
        if (wave == kFeeders) {
            // Agent-scope stores are written through to where all XCDs see them, and are waited for before they are counted; the
            // last workgroup reads them by agent-scope loads, behind the count.  (A release fence instead writes back all that the
            // XCD's L2 holds, 672 times: 75 us.)
            if (v < Nt) __hip_atomic_store(&devs[p.pair * Nt + v], acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) s_last = __hip_atomic_fetch_add(&stats[p.pair].best, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tiles - 1;
        }
        __syncthreads();
        if (!s_last) return;
        lay_out<true, kSumThreads>(devs + p.pair * Nt, Nt, s_sums, []() {});
        if (wave == 0) s_top[0][0] = highest(tops + p.pair * Nt, Nt);
        __syncthreads();
        if (wave != kFeeders) return;
        const double denom = sqrt(ordered_sum(Nt, s_sums) / window_size(Nt, p.w)) + 1e-6;
        const double tau = ((p.flags >> 1) & 3) == 1 ? tau_near : tau_far;     // class 1 = NEAR (decay length >= block size)
        set_stats(S, p, N, Nt, mu, denom, tau, s_top[0][0], tops, rows, stats);
    }
}

// Link bytes and the density rule in one pass over the scores.  A workgroup owns a query block (Bs rows) and 1024 key columns;
// a thread takes four consecutive columns, of every kGroups-th row, and keeps their numbers of links in the bytes of one
// word (a count is at most 128), so that a wavefront reads 1 KB runs and writes 256-byte ones and the link bytes are not read
// again; only scores inside some row's window are read.  Bound by memory: at 8192 tokens 41 us, 67 MB written and some 65 MB
// read.  (Link bytes, safeguard and density in three launches took 90 us.)
// kGroups = 4 (1024 threads) up to kSmallGrid workgroups, two per compute unit: calls at 128 workgroups 42 us against 49, at 512
// 152 against 171 (block size 128) and 62 against 62 (32), at 750 73 against 68.  grid: (Sb * ceil(N / 1024), masks, B).
constexpr int kBlockCols = 1024;
constexpr int64_t kSmallGrid = 512;
// kPast: link bytes go past the caches, which they and the scores no longer fit: whole calls through them / past them, 4 frames of 4096 tokens
// (268 million link bytes) 317 / 263 us, 16 of 1024 327 / 312, 8 of 1792 (205) 251 / 233, 12 of 1024 (151) 166.5 / 163.8, 33 of 256 x 2 masks (143)
// 195.4 / 190.9, 8 of 1020 x 2 (133) 198.0 / 204.4, 10 of 1024 (105) 128.1 / 130.4.
constexpr int64_t kPastCaches = 140000000;
template <int kGroups, bool kPast = false>
__global__ __launch_bounds__(256 * kGroups) void k_link_blocks(const float* __restrict__ scores, FrameTab tab, const PairStat* __restrict__ stats,
                                                               const uint8_t* __restrict__ class_map, Geometry g,
                                                               uint8_t* __restrict__ links, uint32_t* __restrict__ keepbits,
                                                               int32_t* __restrict__ counts) {
    __shared__ uint32_t s_cnt[kGroups][256];
    __shared__ uint32_t s_bits;
    const int tid = threadIdx.x & 255, group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int N = g.N, Nt = g.Nt, steps = (N + kBlockCols - 1) / kBlockCols;
    const int qb = (int)blockIdx.x / steps, c_step = (int)blockIdx.x % steps;
    const int64_t mask = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    const int r0 = qb * g.Bs, nr = min(g.Bs, N - r0), c0 = c_step * kBlockCols, c = c0 + tid * 4, n = min(4, N - c);
    if (threadIdx.x == 0) s_bits = 0u;
    uint32_t cnt = 0u;
    if (n > 0) {
        // per column: its frame and place there; for the rows of frame `i`, the window, the threshold and the safeguard's row
        int j[4], v[4], from[4], kept_u[4];
        uint32_t width[4], all = 0u;
        float threshold[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = min(c + e, N - 1);
            j[e] = q / Nt;
            v[e] = q - j[e] * Nt;
        }
        const uint32_t present = n == 4 ? ~0u : (1u << (8 * n)) - 1u;
        auto enter_frame = [&](int i) {
            all = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = abs(i - j[e]);
                const int flags = tab.flags[t];
                if (t <= 1) all |= 1u << (8 * e);
                from[e] = 0x40000000;                                    // an empty window: no row lies in it
                width[e] = 0u;
                threshold[e] = 0.f;
                kept_u[e] = -1;
                if (t > 1 && (flags & 1)) {
                    const PairStat st = stats[(mask * g.Nf + i) * g.Nf + j[e]];
                    from[e] = v[e] - tab.w[t];
                    width[e] = 2u * (uint32_t)tab.w[t];
                    threshold[e] = st.threshold;
                    if (st.best >= 0 && st.best % Nt == v[e]) kept_u[e] = st.best / Nt;
                }
            }
            all &= present;
        };
        const int64_t at0 = mask * N * N + (int64_t)r0 * N + c;
        int frame = min(r0 + group, N - 1) / Nt, frame_row0 = frame * Nt - r0;      // the same in every lane (a group may be without rows)
        enter_frame(frame);
        constexpr int kAhead = 4;
        for (int r = group; r < nr; r += kGroups * kAhead) {
            // only columns whose window some row of the batch lies in are read (all, where the batch leaves the frame)
            const int row_last = min(r + (kAhead - 1) * kGroups, nr - 1);
            const int u_first = r - frame_row0, u_last = row_last - frame_row0;
            bool asks = u_last >= Nt;
#pragma unroll
            for (int e = 0; e < 4; ++e) asks = asks || (from[e] <= u_last && u_first - from[e] <= (int)width[e]);
            float x[kAhead][4];
#pragma unroll
            for (int a = 0; a < kAhead; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[a][e] = 0.f;
            if (asks) {
#pragma unroll
                for (int a = 0; a < kAhead; ++a) {
                    const int64_t at = at0 + (int64_t)min(r + a * kGroups, nr - 1) * N;
                    if (n == 4) __builtin_memcpy(x[a], scores + at, 16);      // (4-byte aligned)
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[a][e] = scores[at + min(e, n - 1)];
                    }
                }
            }
            const bool any_asks = __any(asks);                            // the same in every lane
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const int row = r + a * kGroups;
                if (row >= nr) break;
                while (row - frame_row0 >= Nt) {
                    ++frame;
                    frame_row0 += Nt;
                    enter_frame(frame);
                }
                const int u = row - frame_row0;
                uint32_t out = all;
                if (any_asks) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool link = u == kept_u[e] || ((uint32_t)(u - from[e]) <= width[e] && x[a][e] >= threshold[e]);
                        out |= link ? 1u << (8 * e) : 0u;
                    }
                    out &= present;
                }
                const int64_t at = at0 + (int64_t)row * N;
                if constexpr (kPast) __builtin_nontemporal_store(out, reinterpret_cast<uint32_t*>(links + at));      // (n is 4: rows of whole words)
                else if (n == 4) __builtin_memcpy(links + at, &out, 4);
                else for (int e = 0; e < n; ++e) links[at + e] = (uint8_t)(out >> (8 * e));
                cnt += out;
            }
        }
    }
    s_cnt[group][tid] = cnt;
    __syncthreads();
    if (group != 0) return;
    for (int k = 1; k < kGroups; ++k) cnt += s_cnt[k][tid];
    const int row_min = nr == g.Bs ? g.row_min_full : g.row_min_tail;
    int active = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) active += (e < n && (int)((cnt >> (8 * e)) & 255u) >= row_min) ? 1 : 0;
    const int per_block = g.Bs / 4;                                       // threads of a key block: 8, 16 or 32
    for (int off = 1; off < per_block; off <<= 1) active += __shfl_xor(active, off);
    const int kb = c / g.Bs;
    if (n > 0 && tid % per_block == 0) {
        const int nc = min(g.Bs, N - kb * g.Bs);
        const int col_min = nc == g.Bs ? g.col_min_full : g.col_min_tail;
        // a block that holds a token pair with t <= 1 is kept whatever its density
        if (class_map[(int64_t)qb * g.Sb + kb] == 3 || active >= col_min) atomicOr(&s_bits, 1u << (kb - c0 / g.Bs));
    }
    __syncthreads();
    // the step's 8, 16 or 32 bits as bytes of the row's bitmap; the last step clears what is left of the last word
    const int64_t row = mask * g.Sb + qb;
    const int words = (g.Sb + 31) / 32, step_bytes = kBlockCols / g.Bs / 8, at = c_step * step_bytes;
    uint8_t* bytes = reinterpret_cast<uint8_t*>(keepbits + row * words);
    const int to = c_step + 1 == steps ? words * 4 : at + step_bytes;
    if (tid < to - at && at + tid < words * 4) bytes[at + tid] = tid < step_bytes ? (uint8_t)(s_bits >> (8 * tid)) : (uint8_t)0;
    if (tid == 0 && s_bits) atomicAdd(&counts[row], __popc(s_bits));
}

// The same for pairs of small frames in one launch: a workgroup holds the pair's scores in LDS (two such workgroups share a CU at
// 128 tokens, three from 115 down) and makes the statistics, the bytes and the safeguard itself; the density rule follows.  Where
// there is little work three launches cost more than two, where there is much the serial chains of a workgroup do, and for one
// mask of frames above 115 tokens they do as well: whole calls, the three launches above / these two, 16 frames of 64 tokens 27.9 / 20.2 us;
// 33 of 64: 30.1 / 25.8; 20 of 96: 34.9 / 34.9; 33 of 96 (10 million token pairs): 47.0 / 44.9; 50 of 96 (23 million): 60.9 / 65.6; 33 of 121: 53.3 / 70.8;
// 9 of 120: 30.7 / 33.0; 16 of 128: 31.0 / 35.9; 24 of 128 (9 million): 42.0 / 46.9; 60 of 128: 80 / 133; several masks, 16 of 117 x 2: 47.9 / 46.5;
// 10 of 120 x 4: 43.8 / 40.3.  (In another run the latter two measured 36.5 / 38.9 and 43.1 / 39.3, 16 of 128 x 2 33.3 / 42.1, 19 of 128 x 2 45.0 / 63.8,
// 13 of 128 x 4 44.6 / 64.1, 9 of 128 x 8 46.4 / 51.3: several masks keep the two launches, as they always have, although the three are the
// faster ones at most sizes.)
constexpr int64_t kSmallPairs = 12 << 20;
constexpr int kThreePerCu = 115;
inline bool small_frames(int B, int masks, int N, int Nf) {
    const int Nt = N / Nf;
    return Nt <= kSmallFrame && (int64_t)B * masks * N * N <= kSmallPairs && (Nt <= kThreePerCu || (int64_t)B * masks > 1);
}
// grid: (Nf * Nf, masks, B).  LDS: Nt doubles | Nt * Nt floats.
__global__ __launch_bounds__(kThreads) void k_pair_links_small(const float* __restrict__ scores, FrameTab tab, int N, int Nt, int Nf,
                                                               double tau_near, double tau_far, uint8_t* __restrict__ links) {
    extern __shared__ double col[];
    __shared__ double s_total;
    __shared__ unsigned long long s_best;
    __shared__ unsigned int s_kept;
    float* S = reinterpret_cast<float*>(col + Nt);
    const PairAt p = pair_at<false>(tab, Nf, (int)blockIdx.x);
    const int64_t at0 = p.mask * N * N + (int64_t)p.i * Nt * N + (int64_t)p.j * Nt;
    const int tid = threadIdx.x, size = Nt * Nt;
    if (!p.judged) {
        for (int q = tid; q < size; q += kThreads) links[at0 + (int64_t)(q / Nt) * N + q % Nt] = p.t <= 1 ? 1 : 0;
        return;
    }
    if (tid == 0) { s_kept = 0u; s_best = 0ull; }
#pragma unroll 4
    for (int q = tid; q < size; q += kThreads) S[q] = scores[at0 + (int64_t)(q / Nt) * N + q % Nt];
    __syncthreads();
    // sums of the columns' windows, then of the columns, one by one
    auto total_of = [&](auto&& term) -> double {
        if (tid < Nt) {
            const int lo = max(0, tid - p.w), hi = min(Nt - 1, tid + p.w);
            double acc = 0.0;
#pragma unroll 8
            for (int u = lo; u <= hi; ++u) acc = acc + term(S[u * Nt + tid]);
            col[tid] = acc;
        }
        __syncthreads();
        if (tid == 0) {
            double total = 0.0;
#pragma unroll 8
            for (int v = 0; v < Nt; ++v) total = total + col[v];
            s_total = total;
        }
        __syncthreads();
        return s_total;
    };
    const double n = window_size(Nt, p.w);
    const double mu = total_of([](float s) { return (double)s; }) / n;
    const double denom = sqrt(total_of([&](float s) {
        const double dev = (double)s - mu;
        const double sq = dev * dev;
        return sq;
    }) / n) + 1e-6;
    const double tau = ((p.flags >> 1) & 3) == 1 ? tau_near : tau_far;     // class 1 = NEAR (decay length >= block size)
    unsigned int kept = 0u;
    unsigned long long best = 0ull;
    for (int q = tid; q < size; q += kThreads) {
        const int u = q / Nt, v = q - u * Nt;
        uint8_t out = 0;
        if (abs(u - v) <= p.w) {
            const float s = S[q];
            out = ((double)s - mu) / denom >= tau ? 1 : 0;
            kept += out;
            best = max(best, best_key(s, q));
        }
        links[at0 + (int64_t)u * N + v] = out;
    }
    for (int off = 32; off > 0; off >>= 1) {
        kept += __shfl_xor(kept, off);
        best = max(best, (unsigned long long)__shfl_xor(best, off));
    }
    if ((tid & 63) == 0) { atomicAdd(&s_kept, kept); atomicMax(&s_best, best); }
    __syncthreads();
    if (s_kept == 0u && tid == 0) {
        const int q = best_index(s_best);
        links[at0 + (int64_t)(q / Nt) * N + q % Nt] = 1;
    }
}

// Density rule.  One workgroup per query block; a thread sums the link bytes of sixteen consecutive key columns over the
// block's rows, four to a 32-bit word (a count is at most 128), so that a wavefront reads 1 KB runs; the threads of a key
// block then add their numbers of active columns.  Bound by reading the link bytes once.  (A lane per column, one byte at a
// time and half the lanes idle at block size 32, took 380 us at 8192 tokens; this takes 20.)  Where a row has fewer than
// 128 such units the rows are shared out over the idle threads and their counts added up in LDS; the last unit of a row
// whose length is no multiple of sixteen is the row's last sixteen bytes, of which its own columns count.
// grid: (Sb, masks, B).
__global__ __launch_bounds__(kThreads) void k_aggregate_links(const uint8_t* __restrict__ links,
                                                              const uint8_t* __restrict__ class_map, Geometry g,
                                                              uint32_t* __restrict__ keepbits, int32_t* __restrict__ counts) {
    constexpr int kCols = 16 * kThreads;                    // columns of a step: 32, 64 or 128 key blocks
    __shared__ uint32_t s_bits[4];
    __shared__ uint4 s_part[kThreads];
    __shared__ int s_count;
    const int qb = blockIdx.x, tid = threadIdx.x;
    const int words = (g.Sb + 31) / 32;
    const int64_t mask_id = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    const int64_t row = mask_id * g.Sb + qb;
    const int r0 = qb * g.Bs, nr = min(g.Bs, g.N - r0);
    const uint8_t* L = links + mask_id * g.N * g.N + (int64_t)r0 * g.N;
    const int row_min = nr == g.Bs ? g.row_min_full : g.row_min_tail;
    const int per_block = g.Bs / 16;                        // threads of a key block: 2, 4 or 8
    // threads per row: a power of two, whole key blocks; the others take rows of their own
    int span = per_block;
    while (span < kThreads && span * 16 < g.N) span <<= 1;
    const int unit = tid & (span - 1), first = tid / span, groups = kThreads / span;
    if (tid == 0) s_count = 0;
    for (int c_step = 0; c_step < g.N; c_step += kCols) {
        if (tid < 4) s_bits[tid] = 0u;
        __syncthreads();
        const int c = c_step + unit * 16, n = min(16, g.N - c);      // n <= 0: past the last column
        const int at = min(c, g.N - 16);                             // where the unit's sixteen bytes start (N >= 16)
        uint32_t cnt[4] = {0u, 0u, 0u, 0u};
        auto add_row = [&](int r) {
            uint32_t x[4];
            __builtin_memcpy(x, L + (int64_t)r * g.N + at, 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) cnt[e] += x[e];
        };
        if (n > 0 && at >= 0 && groups == 1) {                       // (apart from the other: a fixed step, eight loads in flight)
#pragma unroll 8
            for (int r = 0; r < nr; ++r) add_row(r);
        } else if (n > 0 && at >= 0) {
#pragma unroll 4
            for (int r = first; r < nr; r += groups) add_row(r);
        } else {                                                     // (fewer than sixteen tokens in all)
            for (int e = 0; e < n; ++e)
                for (int r = first; r < nr; r += groups) cnt[(16 - n + e) >> 2] += (uint32_t)L[(int64_t)r * g.N + c + e] << (8 * ((16 - n + e) & 3));
        }
        if (groups > 1) {                                            // (a single step: the row fits the span)
            s_part[tid] = make_uint4(cnt[0], cnt[1], cnt[2], cnt[3]);
            __syncthreads();
            for (int i = 1; i < groups; ++i) {
                const uint4 p = s_part[(tid + i * span) & (kThreads - 1)];
                cnt[0] += p.x; cnt[1] += p.y; cnt[2] += p.z; cnt[3] += p.w;
            }
        }
        int active = 0;                                              // the unit's own columns are the last n of its sixteen
#pragma unroll
        for (int e = 0; e < 16; ++e) active += (e >= 16 - n && (int)((cnt[e >> 2] >> (8 * (e & 3))) & 255u) >= row_min) ? 1 : 0;
        for (int off = 1; off < per_block; off <<= 1) active += __shfl_xor(active, off);
        const int kb = c / g.Bs;
        if (kb < g.Sb && tid < span && unit % per_block == 0) {
            const int nc = min(g.Bs, g.N - kb * g.Bs);
            const int col_min = nc == g.Bs ? g.col_min_full : g.col_min_tail;
            // a block that holds a token pair with t <= 1 is kept whatever its density
            if (class_map[(int64_t)qb * g.Sb + kb] == 3 || active >= col_min) atomicOr(&s_bits[(kb - c_step / g.Bs) >> 5], 1u << (kb & 31));
        }
        __syncthreads();
        const int w0 = c_step / g.Bs / 32, n_words = kCols / g.Bs / 32;
        if (tid < n_words && w0 + tid < words) {
            keepbits[row * words + w0 + tid] = s_bits[tid];
            atomicAdd(&s_count, __popc(s_bits[tid]));
        }
        __syncthreads();
    }
    if (tid == 0) counts[row] = s_count;
}

}  // namespace

hipError_t launch_token_scores(const void* Q, const void* K, bool bf16, const TensorDesc& td, int masks,
                               int heads_per_mask, float* scores, hipStream_t s) {
    const int tiles = (td.N + kTile - 1) / kTile;
    const float scale = (float)(1.0 / ((double)heads_per_mask * sqrt((double)td.d)));
    hipLaunchKernelGGL(bf16 ? k_token_scores<true> : k_token_scores<false>, dim3(tiles, tiles, td.B * masks), dim3(kThreads), 0, s, Q, K, td,
                       masks, heads_per_mask, scale, scores);
    return hipGetLastError();
}

size_t pair_links_scratch_bytes(int B, int masks, int N, int Nf) {
    if (small_frames(B, masks, N, Nf)) return 0;
    return (size_t)B * masks * ((size_t)Nf * N * (2 * sizeof(double) + sizeof(float) + sizeof(int32_t)) + (size_t)Nf * Nf * sizeof(PairStat));
}

hipError_t launch_token_mask(const float* scores, const FrameTab& tab, const uint8_t* class_map, const Geometry& g, int B, int masks,
                             double tau_near, double tau_far, void* scratch, uint8_t* links, uint32_t* keepbits, int32_t* counts,
                             hipStream_t s) {
    const int N = g.N, Nt = g.Nt, Nf = g.Nf;
    if (small_frames(B, masks, N, Nf) || !scratch) {      // (the caller has no scratch: Nt <= kSmallFrame)
        const size_t lds = (size_t)Nt * sizeof(double) + (size_t)Nt * Nt * sizeof(float);
        if (lds > 64 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pair_links_small), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_pair_links_small, dim3((unsigned)Nf * Nf, masks, B), dim3(kThreads), lds, s, scores, tab, N, Nt, Nf,
                           tau_near, tau_far, links);
        hipLaunchKernelGGL(k_aggregate_links, dim3(g.Sb, masks, B), dim3(kThreads), 0, s, links, class_map, g, keepbits, counts);
        return hipGetLastError();
    }
    const size_t columns = (size_t)B * masks * Nf * N;
    double* sums = static_cast<double*>(scratch);
    double* devs = sums + columns;
    PairStat* stats = reinterpret_cast<PairStat*>(devs + columns);
    float* tops = reinterpret_cast<float*>(stats + (size_t)B * masks * Nf * Nf);
    int32_t* rows = reinterpret_cast<int32_t*>(tops + columns);
    const unsigned pairs = (unsigned)Nf * Nf, cols = (Nt + 63) / 64;
    int64_t judged = 0;                                     // pairs of a mask
    for (int t = 2; t < Nf; ++t) judged += (tab.flags[t] & 1) ? 2 * (Nf - t) : 0;
    const size_t lds = (size_t)((Nt + 15) & ~15) * sizeof(double);
    auto sum_up = [&](auto pass0, auto pass1, int threads) {
        const dim3 grid(pairs * cols, masks, B);
        hipLaunchKernelGGL(pass0, grid, dim3(threads), 0, s, scores, tab, N, Nt, Nf, g.Sb, tau_near, tau_far, sums, devs, tops, rows, stats, counts);
        hipLaunchKernelGGL(pass1, grid, dim3(threads), lds, s, scores, tab, N, Nt, Nf, g.Sb, tau_near, tau_far, sums, devs, tops, rows, stats, counts);
    };
    if (judged * cols * masks * B <= kSumGrid) sum_up(k_link_sums<0, 3>, k_link_sums<1, 3>, 256);
    else sum_up(k_link_sums<0, 1>, k_link_sums<1, 1>, 128);
    const dim3 grid((unsigned)g.Sb * ((N + kBlockCols - 1) / kBlockCols), masks, B);
    if ((int64_t)grid.x * masks * B <= kSmallGrid)
        hipLaunchKernelGGL(k_link_blocks<4>, grid, dim3(1024), 0, s, scores, tab, stats, class_map, g, links, keepbits, counts);
    else if ((int64_t)B * masks * N * N >= kPastCaches && N % 4 == 0 && (reinterpret_cast<uintptr_t>(links) & 3) == 0)
        hipLaunchKernelGGL((k_link_blocks<1, true>), grid, dim3(256), 0, s, scores, tab, stats, class_map, g, links, keepbits, counts);
    else
        hipLaunchKernelGGL(k_link_blocks<1>, grid, dim3(256), 0, s, scores, tab, stats, class_map, g, links, keepbits, counts);
    return hipGetLastError();
}

}  // namespace dr
