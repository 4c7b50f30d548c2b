// Stage (c) at fp32 accuracy: block-sparse softmax attention (paper Eqs. 12-13, epsilon -> 0) for fp32 storage and for
// the bf16 shapes that k_attn_mfma* do not cover (d = 64), on the bf16 matrix instructions.  gfx950 only.
//
// What bounds it: the fp32 matrix instruction does 1/16 of the bf16 one's operations per cycle, the vector ALU no more.
// So every 32-bit operand is split into three bf16 parts, x = h + m + l, which is exact down to 2^-110 (8 + 8 + 8 significant
// bits, each part the rounding of what the parts before it leave), and a product is summed from part products on the bf16
// matrix cores with fp32 accumulation.  Of the nine part products the three of order 2^-26 and below (m l, l m, l l)
// are left out: 6 bf16 instructions for one, 2.7 times the rate of the fp32 instruction.  Inputs stored as bf16 are one
// part (their products are exact); the probabilities stay 32-bit and are always three parts.
// Times and errors against 64 bits are at the kernel's definition below.
//
// One workgroup owns one query block of one (batch, head).  It has kQ * kS wavefronts: wavefront (q, s) owns 32 queries
// and walks every kS-th group of 32-key tiles, so that block sizes 64 and 32, whose rows share no key list, still fill
// four or eight wavefronts (the streams' partial sums are merged at the end, in a fixed order).  Keys and values of a
// stage (kT tiles per stream) are fetched to registers while the stage before is computed, split once by the workgroup and
// left in LDS as bf16 parts (bf16 rows at d = 64 go straight to LDS); at block size 32 no wavefront shares a tile with another, and each
// fetches and splits its own.  The logits are produced transposed, S^T = K Q^T (32x32x16), so that a lane's sixteen values
// belong to one query, and the split probabilities are already the B operand of O^T += V^T P^T; V^T fragments come
// from the row-major parts with the transposing LDS read.
// Softmax is online in fp32; the exponent reference of a query is moved only when a tile's probabilities outgrow it by
// 2^10, which costs no accuracy (fp32 sums are scale free), so the steady state forms no maximum and rescales nothing.
//
// Infinite inputs (or values that round to infinity in bf16) make inf - inf in a split, and values far below 1 lose their
// third part (kTiny).  A workgroup that finds a result that is not finite, or one that may have lost bits, takes its query
// block again with plain fp32 arithmetic on the vector ALU, whose answer stands.
#include "attn_mfma_common.h"
#include "dr_internal.h"

#include <type_traits>

namespace dr {
namespace {

using namespace mfma;

constexpr float kSumLimit = 1024.0f;      // a lane's sixteen probabilities of a tile may sum to at most this
// Three parts hold a value to 2^-134 at best (bf16 ends at 2^-133), that is, exactly down to 2^-110.  What that does to fp32
// results: an output that is not 0 and below kTiny is taken again in plain fp32, and so is a block whose logits could feel
// it, that is, where values of Q beyond kHuge, or nonzero ones below kTiny against keys beyond kHuge, leave an error of more
// than 2^-34 in a product.
constexpr float kTiny = 0x1p-108f, kHuge = 0x1p100f;

typedef __attribute__((address_space(3))) const v8bf* lds_v8;
typedef __attribute__((address_space(3))) v4s* lds_v4;
typedef float v4f32 __attribute__((ext_vector_type(4)));

// L: launches of few query blocks, of at most one workgroup a compute unit (bf16, d = 64, block size 32), or of many (fp32, d = 64, block size
// 128); the results are the same bits
constexpr int kAnyLaunch = 0, kFewBlocks = 1, kManyBlocks = 2;
template <bool BF16, int D, int BS, int L = kAnyLaunch>
struct Plan {
    static constexpr int kIn = BF16 ? 1 : 3;                        // parts of Q, K, V
    static constexpr int kQ = BS / 32;                              // wavefronts along the queries
    // block size 32: nobody shares a wavefront's key tiles, so each walks alone (keys straight to registers, values through
    // an LDS region of its own, no barrier), eight to a workgroup where their regions fit two per SIMD
    static constexpr bool kAlone = BS == 32;
    // Two streams of four query groups and a second buffer: a query block's list takes half as many steps, and a launch of up to one
    // workgroup a compute unit leaves no SIMD with a single wavefront.  Against one stream (two workgroups of four wavefronts a
    // compute unit): 96 blocks of 1024 tokens 57.9 -> 43.6 us, 240 of 2048 84 -> 65, of 10 240 169 -> 126, 720 258 -> 247.  (At block size 64,
    // where two streams are the rule, four measured 44.0 -> 34.4 at 84 blocks, 75 -> 81 at 320, 531 -> 555 at 1760: they stay two.)
    static constexpr bool kTwo = !BF16 && D == 64 && BS == 128, kEight = kTwo && L != kManyBlocks;
    // Where many blocks wait, two independent workgroups of four wavefronts a compute unit get more done than one of eight that keep step:
    // one stream / eight wavefronts / in turn, 4000 blocks of 5120 tokens 1135 / 1191 / 1138 us, of 2048 785 / 841 / 790, 1440 of 1024 180 / 194 / 181,
    // 320 of 256 26.9 / 33.1 / 27.4.  They take the two streams in turn, with the first one's sums in registers meanwhile.
    static constexpr int kTurns = kTwo && !kEight ? 2 : 1;
    static constexpr int kS = kAlone ? (!BF16 && D == 128 ? 4 : 8) : (kEight ? 8 : 4) / kQ;        // streams of key tiles
    static constexpr int kThreads = 64 * kQ * kS;
    // bf16 rows straight from memory to LDS, the keys as well: fewer instructions and registers (120, four wavefronts a SIMD), a longer
    // way for a key.  17 550 tokens x 12 heads 815 -> 724 us, 6144 x 8 119 -> 100, 384 query blocks 21.9 -> 18.9; 192 and 168 blocks, with
    // a few tiles a wavefront, 12.7 -> 13.1 and 11.9 -> 12.5: launches of up to one workgroup a compute unit keep the registers
    // (the results are the same bits).
    static constexpr bool kAloneDirect = kAlone && BF16 && D == 64 && L != kFewBlocks;
    static constexpr int kTileBytes = 32 * (kAlone && !kAloneDirect ? 1 : 2) * kIn * 2 * D;          // 32 keys of (K and) V, all parts
    // bf16 rows go to LDS as they are, straight from memory, a stage of 64 keys ahead
    static constexpr bool kDirect = BF16 && D == 64 && !kAlone;
    static constexpr int kT = (kDirect && kS == 1) || kTurns == 2 ? 2 : 1;      // 32-key tiles per stream and stage
    static constexpr int kTiles = kS * kT;                          // of a stage
    static constexpr int kRows = kAlone ? 32 : kTiles * 32;         // of an LDS region
    static constexpr int kStageBytes = kTiles * kTileBytes;
    // one wavefront per SIMD (fp32, d = 128: 96 registers of Q parts) has nobody to hide its vector instructions behind: they go
    // between the matrix instructions, with a second buffer, where two fit
    static constexpr int kBuffers = kDirect || kEight || (!kAlone && !BF16 && D == 128 && 2 * kStageBytes <= 128 * 1024) ? 2 : 1;
    static constexpr int kPerSimd = !BF16 && D == 128 ? 1 : kDirect || kAloneDirect ? 4 : 2;      // wavefronts, at least
    static constexpr int kPlainRows = kThreads / 8, kPlainKeys = BS == 32 ? 32 : 64;
    static constexpr int kPlainBytes = 4 * (kPlainRows * D + kPlainKeys * (D + 1) + kPlainRows * kPlainKeys);
    static constexpr int kMergeBytes = (kS - 1) * kQ * 32 * D * 4 + kS * kQ * 64 * 4;
    static constexpr int kMax1 = kBuffers * kStageBytes > kPlainBytes ? kBuffers * kStageBytes : kPlainBytes;
    static constexpr int kLdsBytes = kMax1 > kMergeBytes ? kMax1 : kMergeBytes;
    static constexpr int kRowUnits = D / 8;                         // a unit = 8 channels of one row
    static constexpr int kFetch = kAlone ? 64 : kThreads;           // threads that fetch a region's rows
    static constexpr int kPasses = kRows * kRowUnits / kFetch;      // units per thread, K and V each
    static constexpr int kRowBytes = 2 * D;
    static_assert(kRows * kRowUnits % kFetch == 0 && kLdsBytes <= 160 * 1024, "stage layout");
};

// 16-byte piece of row r at which channel piece p of a K part row is kept: the sixteen rows a ds_read_b128 touches per
// cycle fall in distinct bank groups
template <int D> __device__ __forceinline__ int k_piece(int p, int r) { return D == 128 ? p ^ (r & 15) : p ^ ((r >> 1) & 7); }
// the same for V: the four rows of a transposing read's patch fall in distinct 64-byte groups
template <int D> __device__ __forceinline__ int v_piece(int p, int r) { return D == 128 ? p ^ ((r & 3) << 2) : p ^ (((r >> 1) & 1) << 2); }

// (the converted pair is unpacked again from its packed word, which costs two bit operations)
__device__ __forceinline__ void split2(float r0, float r1, uint32_t (&part)[3]) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        union { v2bf v; uint32_t u; } pk;
        pk.v[0] = (__bf16)r0;
        pk.v[1] = (__bf16)r1;
        asm("" : "+v"(pk.u));                                // keeps the pair packed
        part[p] = pk.u;
        r0 -= __uint_as_float(pk.u << 16);
        r1 -= __uint_as_float(pk.u & 0xffff0000u);
    }
}
__device__ __forceinline__ void split8(const float (&x)[8], v8bf (&part)[3]) {
    union { uint32_t u[4]; v8bf v; } w[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t t[3];
        split2(x[2 * i], x[2 * i + 1], t);
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p].u[i] = t[p];
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) part[p] = w[p].v;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// c += a b with both operands in parts: the six part products of order above 2^-26 (three when b is one part), small ones first
template <int NA, int NB>
__device__ __forceinline__ v16f mfma_parts(const v8bf (&a)[NA], const v8bf (&b)[NB], v16f c) {
#pragma unroll
    for (int order = 2; order >= 0; --order)
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int j = order - i;
            if (j >= 0 && j < NB) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], c, 0, 0, 0);
        }
    return c;
}

template <bool BF16, int D>
__device__ __forceinline__ void load_plain(const char* src, float* dst, int g) {
    if (BF16) {
        const uint16_t* p = reinterpret_cast<const uint16_t*>(src);
        for (int c = g; c < D; c += 8) dst[c] = __uint_as_float((uint32_t)p[c] << 16);
    } else {
        const float* p = reinterpret_cast<const float*>(src);
        for (int c = g; c < D; c += 8) dst[c] = p[c];
    }
}

// |x| of a value that is not 0 as an integer, ascending like |x|; a zero gives the largest of all
__device__ __forceinline__ uint32_t nonzero_magnitude(float x) { return (__float_as_uint(x) << 1) - 1u; }
constexpr uint32_t kTinyMagnitude = (__builtin_bit_cast(uint32_t, kTiny) << 1) - 1u;

struct Item {
    const char *Q, *K, *V;      // of this (batch, head)
    char* O;
    float* lse;                 // of this (batch, head), or NULL
    const int32_t* list;        // the row's key blocks
    int n_list, qb, Sb, N;
    int64_t row_bytes;
};

// The query block in plain fp32 on the vector ALU (thread (r, g): row r, every eighth logit of a chunk, D / 8 output
// channels).  Only for blocks with infinities or NaN, or beyond the range that three parts hold (kTiny).  A chunk is 64 keys
// where the block has them: a row is lost only when every logit of its first chunk is -inf (nothing finite to subtract), and
// shorter chunks lose more rows.  Keys and values take turns in one LDS area, so that this pass, which is rarely made, asks
// for little more than the walk does.
template <bool BF16, int D, int BS, int L>
__device__ __forceinline__ void plain_block(const Item& it, float* lds) {
    using P = Plan<BF16, D, BS, L>;
    constexpr int R = P::kPlainRows, C = P::kPlainKeys, DC = D / 8, LPT = C / 8;
    float* sQ = lds;
    float* sX = sQ + R * D;                    // keys, then values
    float* sP = sX + C * (D + 1);
    const int tid = threadIdx.x, r = tid >> 3, g = tid & 7;
    const float scale = 1.0f / sqrtf((float)D);
    for (int row0 = it.qb * BS; row0 < min(it.N, it.qb * BS + BS); row0 += R) {
        const bool row_ok = row0 + r < min(it.N, it.qb * BS + BS);
        __syncthreads();
        if (row_ok) load_plain<BF16, D>(it.Q + (int64_t)(row0 + r) * it.row_bytes, sQ + r * D, g);
        else for (int c = g; c < D; c += 8) sQ[r * D + c] = 0.f;
        float m_run = -INFINITY, l_run = 0.f, o[DC];
#pragma unroll
        for (int i = 0; i < DC; ++i) o[i] = 0.f;
        for (int e = 0; e < it.n_list; ++e) {
            const int kb = min(max(it.list[e], 0), it.Sb - 1);
            const int k_end = min(it.N, (kb + 1) * BS);
            for (int k0 = kb * BS; k0 < k_end; k0 += C) {
                const int nk = min(C, k_end - k0);
                auto load = [&](const char* X) {
                    for (int kr = tid >> 3; kr < C; kr += R) {
                        if (kr < nk) load_plain<BF16, D>(X + (int64_t)(k0 + kr) * it.row_bytes, sX + kr * (D + 1), g);
                        else for (int c = g; c < D; c += 8) sX[kr * (D + 1) + c] = 0.f;
                    }
                };
                __syncthreads();
                load(it.K);
                __syncthreads();
                float s[LPT];
#pragma unroll
                for (int j = 0; j < LPT; ++j) s[j] = 0.f;
                for (int c = 0; c < D; ++c) {
                    const float qv = sQ[r * D + c];
#pragma unroll
                    for (int j = 0; j < LPT; ++j) s[j] = fmaf(qv, sX[(g + 8 * j) * (D + 1) + c], s[j]);
                }
                float mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < LPT; ++j) {
                    s[j] = (g + 8 * j < nk) ? s[j] * scale : -INFINITY;
                    mx = fmaxf(mx, s[j]);
                }
                for (int off = 1; off < 8; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
                const float m_new = fmaxf(m_run, mx);
                const float alpha = expf(m_run - m_new);
                float ps = 0.f;
#pragma unroll
                for (int j = 0; j < LPT; ++j) {
                    const float p = expf(s[j] - m_new);
                    sP[r * C + g + 8 * j] = p;
                    ps += p;
                }
                for (int off = 1; off < 8; off <<= 1) ps += __shfl_xor(ps, off);
                l_run = l_run * alpha + ps;
                m_run = m_new;
                __syncthreads();
                load(it.V);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < DC; ++i) o[i] *= alpha;
                for (int k = 0; k < nk; ++k) {
                    const float p = sP[r * C + k];
#pragma unroll
                    for (int i = 0; i < DC; ++i) o[i] = fmaf(p, sX[k * (D + 1) + g * DC + i], o[i]);
                }
            }
        }
        if (!row_ok) continue;
        const float inv = (l_run > 0.f) ? 1.0f / l_run : 0.f;
        char* dst = it.O + (int64_t)(row0 + r) * it.row_bytes;
#pragma unroll
        for (int i = 0; i < DC; ++i) {
            const float val = o[i] * inv;
            if (BF16) reinterpret_cast<uint16_t*>(dst)[g * DC + i] = f32_to_bf16_rne(val);
            else reinterpret_cast<float*>(dst)[g * DC + i] = val;
        }
        if (it.lse && g == 0) it.lse[row0 + r] = (l_run > 0.f) ? m_run + logf(l_run) : -INFINITY;
    }
}

// whether this thread's share of the listed keys (fp32) holds one beyond kHuge
template <int D, int BS>
__device__ __forceinline__ bool holds_huge_keys(const Item& it) {
    float most = 0.f;
    for (int e = 0; e < it.n_list; ++e) {
        const int kb = min(max(it.list[e], 0), it.Sb - 1), rows = min(BS, it.N - kb * BS);
        for (int u = threadIdx.x; u < rows * (D / 4); u += blockDim.x) {
            const v4f32 x = *reinterpret_cast<const v4f32*>(it.K + (int64_t)(kb * BS + u / (D / 4)) * it.row_bytes + u % (D / 4) * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) most = fmaxf(most, fabsf(x[i]));
        }
    }
    return most >= kHuge;
}

template <bool BF16, int D, int BS, int L>
__device__ __forceinline__ void attn_split_body(const AttnArgs& a) {
    using P = Plan<BF16, D, BS, L>;
    constexpr int kDB = D / 32, kKS = D / 16;       // channel blocks of O, contraction steps of a logit tile
    constexpr int kPart = P::kRows * P::kRowBytes;  // bytes of one part of K (or V) of a stage
    constexpr int kTPB = BS / 32;                   // 32-key tiles of a key block
    constexpr float kScaleLog2 = (float)(1.4426950408889634 / (D == 128 ? 11.313708498984760 : 8.0));
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    // Twelve idle instructions that only move the code behind them: a lone wavefront per SIMD with a loop of 9.5 KB waits for
    // instruction fetches, and with the place of that loop, in steps of 4 bytes over a line of 64, the same code took 650 to
    // 700 us (6144 tokens x 8 heads, 40 % kept).
    if constexpr (!BF16 && D == 128 && BS == 32) asm volatile(".fill 12, 4, 0xbf800000");
    const int wq = wave % P::kQ, ws = wave / P::kQ;

    // one XCD walks a contiguous run of (batch, head, query block) items: neighbours share K and V in its L2
    constexpr int kXcds = 8;
    const int total = a.Sb * a.td.H * a.td.B, per_xcd = (total + kXcds - 1) / kXcds;
    const int item = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if ((int)(blockIdx.x / kXcds) >= per_xcd || item >= total) return;
    const int qb = item % a.Sb, h = (item / a.Sb) % a.td.H, b = item / (a.Sb * a.td.H);
    constexpr int ES = BF16 ? 2 : 4;
    const int N = a.td.N;
    const int64_t head_off = ((int64_t)b * a.td.stride_b + (int64_t)h * a.td.stride_h) * ES;
    Item it;
    it.Q = reinterpret_cast<const char*>(a.Q) + head_off;
    it.K = reinterpret_cast<const char*>(a.K) + head_off;
    it.V = reinterpret_cast<const char*>(a.V) + head_off;
    it.O = reinterpret_cast<char*>(a.O) + head_off;
    it.lse = a.lse ? a.lse + ((int64_t)b * a.td.H + h) * N : nullptr;
    it.row_bytes = a.td.stride_n * ES;
    it.qb = qb; it.Sb = a.Sb; it.N = N;
    const int mh = (a.mask_heads == 1) ? 0 : h;
    const int32_t* rp = a.rowptr + ((int64_t)b * a.mask_heads + mh) * (a.Sb + 1);
    // row range, clipped to the colidx array of this mask (a list cut short by a too small capacity stays in bounds)
    const int lim = (int)min(a.colidx_stride, (int64_t)0x7fffffff);
    const int beg = min(max(__builtin_amdgcn_readfirstlane(rp[qb]), 0), lim);
    it.n_list = min(max(__builtin_amdgcn_readfirstlane(rp[qb + 1]), beg), lim) - beg;
    it.list = a.colidx + ((int64_t)b * a.mask_heads + mh) * a.colidx_stride + beg;

    // Q^T fragments (B operand): lane holds query l32, channels ks * 16 + 8 * half .. + 7
    const int q_wave0 = qb * BS + wq * 32, qrow = q_wave0 + l32;
    v8bf qf[kKS][P::kIn];
    {
        const char* src = it.Q + (int64_t)min(qrow, N - 1) * it.row_bytes + half * (8 * ES);
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            if constexpr (BF16) {
                qf[ks][0] = *reinterpret_cast<const v8bf*>(src + ks * 32);
            } else {
                const v4f32 x0 = *reinterpret_cast<const v4f32*>(src + ks * 64), x1 = *reinterpret_cast<const v4f32*>(src + ks * 64 + 16);
                const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
                split8(x, qf[ks]);
            }
        }
    }

    // ---- the walk.  Tile t of the row = keys (t % kTPB) * 32 .. + 31 of its key block t / kTPB; stage g holds tiles
    // g * kTiles .., stream s the kT consecutive ones from s * kT on (in turns: every second tile, from the turn's own on).  The list is
    // held in a 64-entry register window. ----
    const int n_tiles = it.n_list * kTPB, stages = (n_tiles / P::kTurns + P::kTiles - 1) / P::kTiles;
    int turn = 0;
    auto tile_of = [&](int g, int i) { return (g * P::kTiles + i) * P::kTurns + turn; };
    int wbase = 0, win = it.n_list > 0 ? it.list[min(lane, it.n_list - 1)] : 0;
    auto tile_row0 = [&](int t) {          // t < n_tiles, its key block inside the window; clamped: a malformed list cannot address outside K / V
        const int kb = min(max(__builtin_amdgcn_readlane(win, t / kTPB - wbase), 0), a.Sb - 1);
        return kb * BS + (t % kTPB) * 32;
    };
    const int64_t lane_off = (int64_t)(lane / P::kRowUnits) * it.row_bytes + (lane % P::kRowUnits) * (8 * ES);
    struct Raw { v4f32 x[BF16 ? 1 : 2]; };
    Raw rk[P::kPasses], rv[P::kPasses];
    int row0_next[P::kT], row0[P::kT];
    auto fetch = [&](int g) {
        const int e_first = tile_of(g, 0) / kTPB, e_last = min(tile_of(g, P::kTiles - 1) / kTPB, it.n_list - 1);
        if (e_last - wbase >= 64) {          // wavefront-uniform
            wbase = e_first;
            win = it.list[min(wbase + lane, it.n_list - 1)];
        }
#pragma unroll
        for (int c = 0; c < P::kT; ++c) row0_next[c] = tile_row0(min(tile_of(g, ws * P::kT + c), n_tiles - 1));
#pragma unroll
        for (int p = 0; p < P::kPasses; ++p) {
            constexpr int kWaveRows = 64 / P::kRowUnits;          // rows of one wavefront and pass: they lie in one tile
            static_assert(32 % kWaveRows == 0, "a wavefront's rows lie in one tile");
            const int wave_row = (p * P::kThreads + wave * 64) / P::kRowUnits;
            const int r = tile_row0(min(tile_of(g, wave_row / 32), n_tiles - 1)) + wave_row % 32;      // the same in every lane
            const int64_t base = (int64_t)r * it.row_bytes;
            int64_t off = base + lane_off;
            if (r + kWaveRows > N) off = (int64_t)min(r + lane / P::kRowUnits, N - 1) * it.row_bytes + (lane % P::kRowUnits) * (8 * ES);
#pragma unroll
            for (int i = 0; i < (BF16 ? 1 : 2); ++i) {
                rk[p].x[i] = *reinterpret_cast<const v4f32*>(it.K + off + i * 16);
                rv[p].x[i] = *reinterpret_cast<const v4f32*>(it.V + off + i * 16);
            }
        }
    };
    // split the fetched rows into their LDS parts, sixteen bytes of a row at a time (u: pass, K or V, half of the unit)
    constexpr int kPieces = P::kPasses * 2 * (BF16 ? 1 : 2);
    auto store_piece = [&](int u, int buffer) {
        const int i = BF16 ? 0 : u & 1, v = (BF16 ? u : u >> 1) & 1, p = BF16 ? u >> 1 : u >> 2;
        const int row = (p * P::kThreads + tid) / P::kRowUnits, piece = tid % P::kRowUnits;
        unsigned char* dst = smem + buffer * P::kStageBytes + row * P::kRowBytes +
                             (v ? P::kIn * kPart + v_piece<D>(piece, row) * 16 : k_piece<D>(piece, row) * 16);
        const v4f32 x = v ? rv[p].x[i] : rk[p].x[i];
        if constexpr (BF16) {
            *reinterpret_cast<v4f32*>(dst) = x;
        } else {
            uint32_t a01[3], a23[3];
            split2(x[0], x[1], a01);
            split2(x[2], x[3], a23);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(dst + q * kPart + i * 8) = make_uint2(a01[q], a23[q]);
        }
    };
    auto store = [&](int buffer) {
#pragma unroll
        for (int u = 0; u < kPieces; ++u) store_piece(u, buffer);
    };

    v16f o[kDB];
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
    float ref = -INFINITY, l_run = 0.f;      // exponent reference of this lane's query (log2 units), this half's normaliser

    const uint32_t lds0 = lds_addr(smem);
    const uint32_t v_base = P::kAlone ? (uint32_t)ws * P::kTileBytes + (P::kAloneDirect ? kPart : 0) : (uint32_t)P::kIn * kPart;
    const uint32_t stream = P::kDirect ? (uint32_t)(ws * P::kT * 32 * P::kRowBytes) : 0u, alone = P::kAloneDirect ? (uint32_t)ws * P::kTileBytes : 0u;      // (the others add it to a tile's place)
    uint32_t k_addr[kKS], v_addr[kDB];
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) k_addr[ks] = lds0 + stream + alone + l32 * P::kRowBytes + k_piece<D>(ks * 2 + half, l32) * 16;
    {
        const int v_e = (lane & 15) >> 2, v_c = lane & 3, v_grp = (lane >> 4) & 1;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
            v_addr[db] = lds0 + v_base + stream + (half * 4 + v_e) * P::kRowBytes + v_piece<D>(db * 4 + v_grp * 2 + (v_c >> 1), v_e) * 16 + (v_c & 1) * 8;
    }

    // softmax of a logit tile (keys x queries) and its share of O; `tile`: LDS offset of its values
    auto use_tile = [&](v16f& s, int valid, uint32_t tile, auto&& before_values) {
                    if (valid < 32) {
                        int base = half * 4;
                        asm volatile("" : "+v"(base));                   // (a branch, not sixteen selects on every tile)
#pragma unroll
                        for (int j = 0; j < 16; ++j)
                            if ((j >> 2) * 8 + base + (j & 3) >= valid) s[j] = -INFINITY;
                    }
                    // The exponentials are taken against the reference as it stands; their sum, which joins the normaliser anyway,
                    // is also the guard: beyond 2^10 (or not a number, as before the first tile) the reference is moved to the row
                    // maximum and they are taken again, once.
                    float p[2][8], sum = 0.f;
                    auto exps = [&]() {
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int i = 0; i < 8; ++i) p[t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t * 8 + i], kScaleLog2, -ref));
                        // (the tile's share first: fewer roundings at the running sum's size)
                        sum = (((p[0][0] + p[0][1]) + (p[0][2] + p[0][3])) + ((p[0][4] + p[0][5]) + (p[0][6] + p[0][7]))) +
                              (((p[1][0] + p[1][1]) + (p[1][2] + p[1][3])) + ((p[1][4] + p[1][5]) + (p[1][6] + p[1][7])));
                    };
                    exps();
                    if (__any(!(sum <= kSumLimit))) {
                        float mx = s[0];
#pragma unroll
                        for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
                        mx = max_across_halves(mx) * kScaleLog2;             // finite for finite inputs: the tile holds at least one key
                        const float ref_new = fmaxf(ref, mx);
                        const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);      // first tile: exp2(-inf) = 0
                        ref = ref_new;
                        l_run *= alpha;
#pragma unroll
                        for (int db = 0; db < kDB; ++db)
#pragma unroll
                            for (int j = 0; j < 16; ++j) o[db][j] *= alpha;
                        exps();
                    }
                    l_run += sum;
                    if constexpr (!BF16 && D == 128) {
#pragma unroll
                        for (int db = 0; db < kDB; ++db) asm volatile("" : "+v"(o[db]));
                    }
                    before_values();
                    v8bf pf[2][3];
                    split8(p[0], pf[0]);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
#pragma unroll
                        for (int db = 0; db < kDB; ++db) {
                            v8bf vf[P::kIn];
#pragma unroll
                            for (int i = 0; i < P::kIn; ++i) {
                                union { struct { v4s a, b; } s2; v8bf v; } u;
                                const uint32_t at = v_addr[db] + tile + i * kPart + t * 16 * P::kRowBytes;
                                u.s2.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(uintptr_t)at);
                                u.s2.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(uintptr_t)(at + 8 * P::kRowBytes));
                                vf[i] = u.v;
                            }
                            o[db] = mfma_parts<P::kIn, 3>(vf, pf[t], o[db]);
                        }
                        if (t == 0) split8(p[1], pf[1]);          // (between the products of the first half)
                    }
                    constexpr int kPvMfma = kDB * (P::kIn == 3 ? 6 : 3);          // of one half
                    __builtin_amdgcn_sched_group_barrier(0x100, 2 * P::kIn, 1);
#pragma unroll
                    for (int i = 0; i < 2 * kPvMfma; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2 * P::kIn * kDB / kPvMfma, 1);
                        if (i < kPvMfma) __builtin_amdgcn_sched_group_barrier(0x002, (44 + kPvMfma - 1) / kPvMfma, 1);
                    }
    };

    auto to_lds = [&](const char* from, uint32_t to) {          // sixteen bytes a lane; counted by hand
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(from), "s"(to) : "memory", "m0");
    };
    if constexpr (P::kAloneDirect) {
        // A stream's tiles one after the other through a place of its own, without a barrier: the next tile's keys are fetched as soon as
        // this one's are read, its values when the products with this one's are made, so either has half a tile's time to arrive.
        // Four loads each, in turn: where four are on their way at most, the ones before them have arrived.
        const int own = (it.n_list - ws + P::kS - 1) / P::kS;
        int base = 0, at = own > 0 ? it.list[min(ws + lane * P::kS, it.n_list - 1)] : 0;
        asm volatile("" : "+v"(at));
        auto row_of = [&](int j) {             // clamped: a malformed list cannot address outside K / V
            if (j - base >= 64) {              // wavefront-uniform
                base = j;
                at = it.list[min(ws + (base + lane) * P::kS, it.n_list - 1)];
                asm volatile("" : "+v"(at));   // (waited for here, and not counted among the tiles' loads)
            }
            return min(max(__builtin_amdgcn_readlane(at, j - base), 0), a.Sb - 1) * 32;
        };
        const int r0 = lane >> 3;              // + 8 i in load i; the swizzles are their own inverses, that of V the same for every i
        const char* from_k[2];
        const char* from_v = it.V + (int64_t)r0 * it.row_bytes + v_piece<D>(lane & 7, r0) * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) from_k[i] = it.K + (int64_t)r0 * it.row_bytes + k_piece<D>(lane & 7, r0 + 8 * i) * 16;
        const uint32_t to0 = __builtin_amdgcn_readfirstlane(lds0 + alone);
        auto issue = [&](int row0, bool values) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const char* from = (values ? from_v : from_k[i & 1]) + (int64_t)(row0 + 8 * i) * it.row_bytes;
                if (row0 + 32 > N) from -= (int64_t)max(row0 + 8 * i + r0 - (N - 1), 0) * it.row_bytes;      // past the end: the last row again
                to_lds(from, to0 + (values ? kPart : 0) + i * 1024u);
            }
        };
        int row = 0;
        if (own > 0) {
            row = row_of(0);
            issue(row, false);
            issue(row, true);
        }
        for (int j = 0; j < own; ++j) {
            const int row_next = row_of(min(j + 1, own - 1));      // (behind the last tile: that tile again, read by nobody)
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory");       // the keys are there
            v8bf kf[kKS];
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) kf[ks] = *(lds_v8)(uintptr_t)k_addr[ks];
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(kf[0]), "+v"(kf[1]), "+v"(kf[2]), "+v"(kf[3]) :: "memory");      // and read
            issue(row_next, false);
            v16f s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks][0], s, 0, 0, 0);
            use_tile(s, N - row, 0u, []() { asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); });      // the values are there
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // and read
            issue(row_next, true);
            row = row_next;
        }
        DR_WAIT_VMCNT0();                      // none may land in what the merge lays out
    } else if constexpr (P::kAlone) {
        // stream s takes tiles s, s + kS, ..: lane i of the window holds the stream's entry base + i
        constexpr int kWaveRows = 64 / P::kRowUnits, NX = BF16 ? 1 : 2;
        const int own = (it.n_list - ws + P::kS - 1) / P::kS;
        unsigned char* region = smem + ws * P::kTileBytes;
        v4f32 xk[kKS][NX], xv[P::kPasses][NX];
        int base = 0, at = own > 0 ? it.list[min(ws + lane * P::kS, it.n_list - 1)] : 0, next_row0 = 0;
        auto fetch_own = [&](int j) {
            if (j - base >= 64) {
                base = j;
                at = it.list[min(ws + (base + lane) * P::kS, it.n_list - 1)];
            }
            next_row0 = min(max(__builtin_amdgcn_readlane(at, j - base), 0), a.Sb - 1) * 32;      // clamped, as above
            const char* k = it.K + (int64_t)min(next_row0 + l32, N - 1) * it.row_bytes + half * (8 * ES);
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
                for (int i = 0; i < NX; ++i) xk[ks][i] = *reinterpret_cast<const v4f32*>(k + ks * (16 * ES) + i * 16);
#pragma unroll
            for (int p = 0; p < P::kPasses; ++p) {
                const int r = min(next_row0 + p * kWaveRows + lane / P::kRowUnits, N - 1);
                const char* v = it.V + (int64_t)r * it.row_bytes + (lane % P::kRowUnits) * (8 * ES);
#pragma unroll
                for (int i = 0; i < NX; ++i) xv[p][i] = *reinterpret_cast<const v4f32*>(v + i * 16);
            }
        };
        if (own > 0) fetch_own(0);
        for (int j = 0; j < own; ++j) {
            const int valid = N - next_row0;
            // a wavefront's LDS operations execute in order; the fences keep the compiler from moving them past each other
#pragma unroll
            for (int p = 0; p < P::kPasses; ++p) {
                const int row = p * kWaveRows + lane / P::kRowUnits;
                unsigned char* dst = region + row * P::kRowBytes + v_piece<D>(lane % P::kRowUnits, row) * 16;
                if constexpr (BF16) {
                    *reinterpret_cast<v4f32*>(dst) = xv[p][0];
                } else {
                    const float x[8] = {xv[p][0][0], xv[p][0][1], xv[p][0][2], xv[p][0][3], xv[p][1][0], xv[p][1][1], xv[p][1][2], xv[p][1][3]};
                    v8bf part[3];
                    split8(x, part);
#pragma unroll
                    for (int i = 0; i < 3; ++i) *reinterpret_cast<v8bf*>(dst + i * kPart) = part[i];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            v16f s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                v8bf kf[P::kIn];
                if constexpr (BF16) {
                    union { v4f32 x; v8bf v; } u;
                    u.x = xk[ks][0];
                    kf[0] = u.v;
                } else {
                    const float x[8] = {xk[ks][0][0], xk[ks][0][1], xk[ks][0][2], xk[ks][0][3], xk[ks][1][0], xk[ks][1][1], xk[ks][1][2], xk[ks][1][3]};
                    split8(x, kf);
                }
                s = mfma_parts<P::kIn, P::kIn>(kf, qf[ks], s);
            }
            if (j + 1 < own) fetch_own(j + 1);
            use_tile(s, valid, 0u, []() {});
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    } else if constexpr (P::kDirect) {
        // Stage g = rows 64 g .. of the listed blocks one after the other, two buffers: the next stage's rows are on their way, without
        // a register, while this one is multiplied, and a barrier a stage keeps the four wavefronts together.  A wavefront fetches
        // sixteen rows of K and of V, eight rows an instruction; the swizzles are folded into the lanes' addresses.
        static_assert(P::kTiles == 2 && P::kRowUnits == 8 && P::kThreads == 256, "stages of 64 rows");
        constexpr int kStagesPerBlock = BS / 64;
        const int n_stages = it.n_list * kStagesPerBlock;
        auto row_of = [&](int g) {             // clamped: a malformed list cannot address outside K / V
            const int e = g / kStagesPerBlock;
            if (e - wbase >= 64) {             // wavefront-uniform
                wbase = e;
                win = it.list[min(wbase + lane, it.n_list - 1)];
                asm volatile("" : "+v"(win));
            }
            return min(max(__builtin_amdgcn_readlane(win, e - wbase), 0), a.Sb - 1) * BS + g % kStagesPerBlock * 64;
        };
        const char *from_k[2], *from_v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = wave * 16 + i * 8 + (lane >> 3);
            from_k[i] = it.K + (int64_t)r * it.row_bytes + k_piece<D>(lane & 7, r) * 16;      // (the swizzles are their own inverses)
            from_v[i] = it.V + (int64_t)r * it.row_bytes + v_piece<D>(lane & 7, r) * 16;
        }
        const uint32_t to0 = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)wave * 2048u);
        auto issue = [&](int row0, uint32_t buffer) {
            const int64_t at = (int64_t)row0 * it.row_bytes;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const char *k = from_k[i] + at, *v = from_v[i] + at;
                if (row0 + 64 > N) {           // wavefront-uniform: rows past the sequence's end are read again from its last
                    const int r = wave * 16 + i * 8 + (lane >> 3);
                    const int64_t back = (int64_t)max(row0 + r - (N - 1), 0) * it.row_bytes;
                    k -= back;
                    v -= back;
                }
                to_lds(k, to0 + buffer + i * 1024u);
                to_lds(v, to0 + buffer + kPart + i * 1024u);
            }
        };
        int row_next = 0;
        if (n_stages > 0) {
            row_next = row_of(0);
            issue(row_next, 0u);
        }
        auto stage = [&](int g, auto which) {
            constexpr uint32_t kHere = decltype(which)::value * P::kStageBytes, kThere = P::kStageBytes - kHere;
            const int row = row_next;
            DR_WAIT_VMCNT0();                  // this wavefront's rows of the stage have arrived; behind the barrier, everyone's
            DR_BARRIER();                      // (and everyone has read the stage before, whose place is filled next)
            if (g + 1 < n_stages) {
                row_next = row_of(g + 1);
                issue(row_next, kThere);
            }
#pragma unroll
            for (int c = 0; c < P::kT; ++c) {
                const uint32_t tile = kHere + (uint32_t)(c * 32 * P::kRowBytes);
                const int valid = N - row - (ws * P::kT + c) * 32;      // keys of the tile (only the sequence's end has fewer than 32)
                if (valid <= 0) continue;                               // wavefront-uniform
                v16f s;
#pragma unroll
                for (int j = 0; j < 16; ++j) s[j] = 0.f;
                v8bf kf[kKS];
#pragma unroll
                for (int ks = 0; ks < kKS; ++ks) kf[ks] = *(lds_v8)(uintptr_t)(k_addr[ks] + tile);
#pragma unroll
                for (int ks = 0; ks < kKS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks][0], s, 0, 0, 0);
                use_tile(s, valid, tile, []() {});
            }
        };
        for (int g = 0; g < n_stages; g += 2) {
            stage(g, std::integral_constant<uint32_t, 0>{});
            if (g + 1 < n_stages) stage(g + 1, std::integral_constant<uint32_t, 1>{});
        }
    } else if constexpr (P::kBuffers == 2 && !P::kEight) {
        // One wavefront per SIMD issues in order, so the vector instructions of a tile (the exponentials, the split of its
        // probabilities, the split of the rows fetched for later tiles) stand between matrix instructions that do not wait for
        // them, some five to each: the softmax of tile g under the logits of tile g + 1, the splits of rows under the products
        // with the values of tile g.  Keys of tile t are in the key part of buffer t % 2, its values in the value part.
        // The four wavefronts read every fragment, so the LDS is nearly as busy as the matrix pipes: values are kept
        // transposed (a channel's 32 keys in 64 bytes, in the order in which the probabilities lie in a lane), which a fragment
        // reads with one 16-byte load instead of two transposing 8-byte ones, at twice the rate.
        static_assert(P::kS == 1 && P::kT == 1 && kPieces == 8 && kKS == 8 && kDB == 4 && D == 128 && P::kThreads == 256,
                      "eight steps of six matrix instructions each, four pieces of sixteen bytes a thread");
        typedef float v2f32 __attribute__((ext_vector_type(2)));
        // keys: a thread splits eight channels of two rows.  Rows past the sequence's end are read again from its last.
        auto key_offsets = [&](int row0, int64_t (&off)[2]) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int r = p * 16 + wave * 4 + (lane >> 4);
                off[p] = (int64_t)(min(row0 + r, N - 1) - row0) * it.row_bytes + (lane & 15) * 32;
            }
        };
        auto fetch_k = [&](int row0, const int64_t (&off)[2]) {
            const char* base = it.K + (int64_t)row0 * it.row_bytes;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int i = 0; i < 2; ++i) rk[p].x[i] = *reinterpret_cast<const v4f32*>(base + off[p] + i * 16);
        };
        // values: a thread splits two channels of the eight keys that one lane half of a product takes, key e of them being
        // (wave / 2) * 16 + (wave % 2) * 4 + e % 4 + 8 * (e / 4): a wavefront reads whole rows
        v2f32 xv[8];
        const int v_row = (wave >> 1) * 16 + (wave & 1) * 4;
        constexpr int kVRow[8] = {0, 1, 2, 3, 8, 9, 10, 11};
        auto load_v = [&](uint64_t row, int e) {
            asm("" : "+s"(row));                   // (a scalar base and the lane's offset, not a 64-bit product per lane)
            xv[e] = *reinterpret_cast<const __attribute__((address_space(1))) v2f32*>(row + (uint32_t)lane * 8u);
        };
        auto fetch_v = [&](int row0) {             // rows past the sequence's end are read again from its last
#pragma unroll
            for (int e = 0; e < 8; ++e) load_v((uint64_t)(it.V + (int64_t)min(row0 + v_row + kVRow[e], N - 1) * it.row_bytes), e);
        };
        // LDS place of a thread's four pieces: keys of pass 0 and 1, values of channel 2 * lane and 2 * lane + 1
        auto v_unit = [](int channel, int unit) { return channel * 64 + ((unit ^ ((channel >> 2) & 3)) << 4); };
        uint32_t put[4];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int row = p * 16 + wave * 4 + (lane >> 4);
            put[p] = row * P::kRowBytes + k_piece<D>(lane & 15, row) * 16;
            put[2 + p] = P::kIn * kPart + v_unit(2 * lane + p, wave);
        }
        auto pair_of = [&](int u, int j, int h) -> float {      // element h of pair j of piece u
            return u < 2 ? rk[u].x[j >> 1][2 * (j & 1) + h] : xv[2 * j + h][u - 2];
        };
        auto row_of = [&](int t) { return tile_row0(min(t, n_tiles - 1)); };      // first row of tile t (past the end: of the last)
        auto at_buffer = [&](uint32_t addr, uint32_t buffer) {      // (opaque: the parts' offsets stay immediates of the reads)
            uint32_t at = addr + buffer;
            asm("" : "+v"(at));
            return at;
        };
        uint32_t vt_addr[2];                       // of the lane's unit of either half tile; channel block db is 2 KB further
#pragma unroll
        for (int t = 0; t < 2; ++t) vt_addr[t] = lds0 + P::kIn * kPart + v_unit(l32, t * 2 + half);
        auto read_k = [&](uint32_t at, int i, v8bf (&kf)[P::kIn]) { kf[i] = *(lds_v8)(uintptr_t)(at + i * kPart); };
        auto read_v = [&](uint32_t at, int c, int i, v8bf (&vf)[P::kIn]) {      // step c: keys 16 * (c / 4) .., channels 32 * (c % 4) ..
            vf[i] = *(lds_v8)(uintptr_t)(at + i * kPart + (c & 3) * 2048);
        };
        // first: cvt of part q of a pair; second: what the part leaves.  (A conversion's result is read an instruction later at
        // the earliest, so the two are apart.)
        auto convert = [](float r0, float r1) {
            union { v2bf v; uint32_t u; } pk;
            pk.v[0] = (__bf16)r0;
            pk.v[1] = (__bf16)r1;
            asm("" : "+v"(pk.u));                  // keeps the pair packed
            return pk.u;
        };
        auto subtract = [](float (&r)[2], uint32_t part) {
            r[0] -= __uint_as_float(part << 16);
            r[1] -= __uint_as_float(part & 0xffff0000u);
        };
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        v4u word[3];                               // a piece's parts
        float rest[2][2];
        // Slot i (0 .. 11) of the split of piece u into buffer `to`: two pairs at a time, six slots each
        auto split_slot = [&](int u, int i, uint32_t to) {
            const int a = i < 6 ? 0 : 2, b = a + 1, k = i % 6;
            if (k == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h) { rest[0][h] = pair_of(u, a, h); rest[1][h] = pair_of(u, b, h); }
                word[0][a] = convert(rest[0][0], rest[0][1]);
                word[0][b] = convert(rest[1][0], rest[1][1]);
            } else if (k == 1) {
                subtract(rest[0], word[0][a]);
            } else if (k == 2) {
                word[1][a] = convert(rest[0][0], rest[0][1]);
                subtract(rest[1], word[0][b]);
            } else if (k == 3) {
                word[1][b] = convert(rest[1][0], rest[1][1]);
                subtract(rest[0], word[1][a]);
            } else if (k == 4) {
                word[2][a] = convert(rest[0][0], rest[0][1]);
                subtract(rest[1], word[1][b]);
            } else {
                word[2][b] = convert(rest[1][0], rest[1][1]);
            }
            if (i == 8 || i == 10 || i == 11) {
                const int q = i == 8 ? 0 : i == 10 ? 1 : 2;
                *reinterpret_cast<v4u*>(smem + put[u] + to + q * kPart) = word[q];
            }
        };
        auto split_piece = [&](int u, uint32_t to) {
#pragma unroll
            for (int i = 0; i < 12; ++i) split_slot(u, i, to);
        };
        // operands of the six part products in the order of mfma_parts
        constexpr int kPartA[6] = {0, 1, 2, 0, 1, 0}, kPartB[6] = {2, 1, 0, 1, 0, 0};
        v16f s;
        v16f bias;                                 // what the logits of tile g + 1 start from: -inf for keys past the sequence's end
        int row_1 = 0, row_2 = 0, row_3 = 0;       // first rows of tiles g + 1, g + 2, g + 3
        int64_t off_k[2];                          // of tile g + 3
        uint32_t edge = 0u;                        // bits 1, 2, 3: tiles g + 1, g + 2, g + 3 reach past the sequence's end
        bool look = true;                          // something of the next lines' is due
        auto past_end = [&](int row0) { return row0 + 32 > N ? 1u : 0u; };
        auto bias_of = [&](int row0) {
            int base = half * 4 + row0 - N;
            asm volatile("" : "+v"(base));
#pragma unroll
            for (int j = 0; j < 16; ++j) bias[j] = (j >> 2) * 8 + (j & 3) + base >= 0 ? -INFINITY : 0.f;
        };
        if (stages > 0) {
            const int row_0 = row_of(0);
            key_offsets(row_0, off_k);
            fetch_k(row_0, off_k);
            fetch_v(row_0);
#pragma unroll
            for (int u = 0; u < 4; ++u) split_piece(u, 0u);
            row_1 = row_of(1);
            key_offsets(row_1, off_k);
            fetch_k(row_1, off_k);
#pragma unroll
            for (int u = 0; u < 2; ++u) split_piece(u, P::kStageBytes);
            row_2 = row_of(2);
            key_offsets(row_2, off_k);
            fetch_k(row_2, off_k);
            fetch_v(row_1);
            row_3 = row_of(3);
            edge = past_end(row_1) << 1 | past_end(row_2) << 2 | past_end(row_3) << 3;
            __syncthreads();
            bias_of(row_0);
            s = bias;
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                v8bf kf[P::kIn];
#pragma unroll
                for (int i = 0; i < P::kIn; ++i) read_k(k_addr[ks], i, kf);
                s = mfma_parts<P::kIn, P::kIn>(kf, qf[ks], s);
            }
            __syncthreads();                       // tile 0's keys are read by all: the loop's first pass puts tile 2's over them
        }
        for (int g = 0; g < stages; ++g) {
            // the Q parts are only ever operands of matrix instructions, and O leaves them only where the reference moves: they
            // live in accumulation registers
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
                for (int i = 0; i < P::kIn; ++i) asm volatile("" : "+a"(qf[ks][i]));
#pragma unroll
            for (int db = 0; db < kDB; ++db) asm volatile("" : "+a"(o[db]));
            asm volatile("" : "+a"(bias));
            const uint32_t buffer = (uint32_t)(g & 1) * P::kStageBytes, other = P::kStageBytes - buffer;
            v8bf kf[2][P::kIn], vf[2][P::kIn];
            {
                const uint32_t at = at_buffer(k_addr[0], other);
#pragma unroll
                for (int i = 0; i < P::kIn; ++i) read_k(at, i, kf[0]);
            }
            if (__builtin_expect(look, 0)) {        // wavefront-uniform, and rare: one branch for all that is, out of the loop's line
                if ((g + 4) / kTPB - wbase >= 64) {
                    wbase = min((g + 4) / kTPB, it.n_list - 1);      // (the tiles past the end are of the last entry)
                    win = it.list[min(wbase + lane, it.n_list - 1)];
                    asm volatile("" : "+v"(win));   // (waited for here: behind the branch the wait would be for every load)
                }
                key_offsets(row_3, off_k);
                if (edge & 2u) {                    // the loop's own loads took another row
                    fetch_v(row_1);
#pragma unroll
                    for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(xv[e]));
                }
                bias_of(row_1);
            }
            // tile g + 2's values: row by row from v_at on; where a row would lie past the end, the sequence's first row instead
            const int64_t whole = (int64_t)((edge >> 2) & 1u) - 1;      // all bits, or none: without a branch
            uint64_t v_at = (uint64_t)(it.V + (whole & ((int64_t)(row_2 + v_row) * it.row_bytes)));
            const int64_t v_step = whole & it.row_bytes;
            v16f s_next = bias;
            float p[16], quad[4], sum = 0.f;
            union { uint32_t u[4]; v8bf v; } pf[2][3];
            auto exp_of = [&](int e) { p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], kScaleLog2, -ref)); };
            auto quad_of = [&](int c) { quad[c] = (p[4 * c] + p[4 * c + 1]) + (p[4 * c + 2] + p[4 * c + 3]); };
            float left[2][2];
            auto split_p = [&](int a, int k) {      // slot k (0 .. 5) of the split of pairs a and a + 1 of the probabilities, as in split_slot
                auto w = [&](int j, int q) -> uint32_t& { return pf[j >> 2][q].u[j & 3]; };
                if (k == 0) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) { left[0][h] = p[2 * a + h]; left[1][h] = p[2 * a + 2 + h]; }
                    w(a, 0) = convert(left[0][0], left[0][1]);
                    w(a + 1, 0) = convert(left[1][0], left[1][1]);
                } else if (k == 1) {
                    subtract(left[0], w(a, 0));
                } else if (k == 2) {
                    w(a, 1) = convert(left[0][0], left[0][1]);
                    subtract(left[1], w(a + 1, 0));
                } else if (k == 3) {
                    w(a + 1, 1) = convert(left[1][0], left[1][1]);
                    subtract(left[0], w(a, 1));
                } else if (k == 4) {
                    w(a, 2) = convert(left[0][0], left[0][1]);
                    subtract(left[1], w(a + 1, 1));
                } else {
                    w(a + 1, 2) = convert(left[1][0], left[1][1]);
                }
            };
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                const uint32_t at = ks + 1 < kKS ? at_buffer(k_addr[ks + 1], other) : at_buffer(vt_addr[0], buffer);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const int slot = ks * 6 + i;
                    s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks & 1][kPartA[i]], qf[ks][kPartB[i]], s_next, 0, 0, 0);
                    if (i < P::kIn) {
                        if (ks + 1 < kKS) read_k(at, i, kf[(ks + 1) & 1]);
                        else read_v(at, 0, i, vf[0]);
                    }
                    if (slot < 16) exp_of(slot);
                    else if (slot < 40) split_p(2 * ((slot - 16) / 6), (slot - 16) % 6);
                    if (slot >= 40 && slot < 44) quad_of(slot - 40);
                    if (slot == 44) sum = (quad[0] + quad[1]) + (quad[2] + quad[3]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // The exponentials are taken against the reference as it stands; their sum, which joins the normaliser anyway, is also
            // the guard: beyond 2^10 (or not a number, as before the first tile) the reference is moved to the row maximum and
            // they are taken again, once.
            if (__builtin_expect(__any(!(sum <= kSumLimit)), 0)) {
                float mx = s[0];
#pragma unroll
                for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
                mx = max_across_halves(mx) * kScaleLog2;             // finite for finite inputs: the tile holds at least one key
                const float ref_new = fmaxf(ref, mx);
                const float alpha = __builtin_amdgcn_exp2f(ref - ref_new);      // first tile: exp2(-inf) = 0
                ref = ref_new;
                l_run *= alpha;
                // O is rescaled where it lies (the compiler would move it out of the accumulation registers on every tile).  Its
                // last matrix instruction is a phase of 48 others back; the wait states behind cover the one that reads it next.
#pragma unroll
                for (int db = 0; db < kDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        float x = o[db][j], t;
                        asm volatile("v_accvgpr_read_b32 %1, %0\n\tv_mul_f32 %1, %1, %2\n\tv_accvgpr_write_b32 %0, %1"
                                     : "+a"(x), "=&v"(t) : "v"(alpha));
                        o[db][j] = x;
                    }
                asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
                for (int e = 0; e < 16; ++e) exp_of(e);
#pragma unroll
                for (int c = 0; c < 4; ++c) quad_of(c);
#pragma unroll
                for (int j = 0; j < 24; ++j) split_p(2 * (j / 6), j % 6);
                sum = (quad[0] + quad[1]) + (quad[2] + quad[3]);
            }
            l_run += sum;
            const v8bf pt[2][3] = {{pf[0][0].v, pf[0][1].v, pf[0][2].v}, {pf[1][0].v, pf[1][1].v, pf[1][2].v}};
            __builtin_amdgcn_sched_barrier(0);
            uint32_t at = at_buffer(vt_addr[0], buffer);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if (c == 3) at = at_buffer(vt_addr[1], buffer);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const int slot = c * 6 + i;
                    o[c & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c & 1][kPartA[i]], pt[c >> 2][kPartB[i]], o[c & 3], 0, 0, 0);
                    if (c + 1 < 8 && i < P::kIn) read_v(at, c + 1, i, vf[(c + 1) & 1]);
                    // values of tile g + 1 first, keys of tile g + 2 behind them (past the last tile: rows that nobody reads)
                    split_slot(slot < 24 ? 2 + slot / 12 : slot / 12 - 2, slot % 12, slot < 24 ? other : buffer);
                    if (slot >= 24 && slot < 32) {
                        load_v(v_at, slot - 24);
                        if (slot < 31) v_at += slot == 27 ? 5 * v_step : v_step;
                    }
                    if (slot == 47) fetch_k(row_3, off_k);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const int row_4 = row_of(g + 4);
            const uint32_t was = edge;
            edge = edge >> 1 | past_end(row_4) << 3;
            row_1 = row_2;
            row_2 = row_3;
            row_3 = row_4;
            look = ((was | edge) & 14u) != 0u || (g + 5) / kTPB - wbase >= 64;
            s = s_next;
            __syncthreads();
        }
    } else {
    // a tile's logits, its softmax and its share of O; `at`: LDS offset of the stage
    auto take_tile = [&](int g, int c, int row, uint32_t at) {
        const int valid = N - row;                               // keys of the tile (only the sequence's end has fewer than 32)
        if (!(tile_of(g, ws * P::kT + c) < n_tiles && valid > 0)) return;      // wavefront-uniform
        const uint32_t tile = at + (uint32_t)((ws * P::kT + c) * 32 * P::kRowBytes);
        v16f s;
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = 0.f;
        // the fragments of a step are read while the step before is multiplied
        v8bf kf[2][P::kIn];
#pragma unroll
        for (int i = 0; i < P::kIn; ++i) kf[0][i] = *(lds_v8)(uintptr_t)(k_addr[0] + tile + i * kPart);
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            if (ks + 1 < kKS) {
#pragma unroll
                for (int i = 0; i < P::kIn; ++i) kf[(ks + 1) & 1][i] = *(lds_v8)(uintptr_t)(k_addr[ks + 1] + tile + i * kPart);
            }
            s = mfma_parts<P::kIn, P::kIn>(kf[ks & 1], qf[ks], s);
        }
        use_tile(s, valid, tile, []() {});
    };
    if constexpr (P::kEight) {
        // One workgroup of eight wavefronts fills a compute unit, so nobody else runs while it waits: a second buffer, a barrier a
        // stage, the next stage split and the one after it on its way ahead of this one's products.
        if (stages > 0) {
            fetch(0);
            store(0);
#pragma unroll
            for (int c = 0; c < P::kT; ++c) row0[c] = row0_next[c];
            if (stages > 1) fetch(1);
        }
        for (int g = 0; g < stages; ++g) {
            __syncthreads();                     // the stage is laid out, the one before is consumed
            int row[P::kT];
#pragma unroll
            for (int c = 0; c < P::kT; ++c) {
                row[c] = row0[c];
                row0[c] = row0_next[c];
            }
            if (g + 1 < stages) store((g + 1) & 1);
            if (g + 2 < stages) fetch(g + 2);
#pragma unroll
            for (int c = 0; c < P::kT; ++c) take_tile(g, c, row[c], (uint32_t)(g & 1) * P::kStageBytes);
        }
    } else {
    auto walk = [&]() {
    if (stages > 0) fetch(0);
    for (int g = 0; g < stages; ++g) {
        if constexpr (!BF16 && D == 128) {
            // the Q parts are only ever operands of matrix instructions: they live in accumulation registers
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
                for (int i = 0; i < P::kIn; ++i) asm volatile("" : "+a"(qf[ks][i]));
#pragma unroll
            for (int db = 0; db < kDB; ++db) asm volatile("" : "+v"(o[db]));
        }
        __syncthreads();                     // the stage before is consumed
        store(0);
#pragma unroll
        for (int c = 0; c < P::kT; ++c) row0[c] = row0_next[c];
        __syncthreads();
        if (g + 1 < stages) fetch(g + 1);
#pragma unroll
        for (int c = 0; c < P::kT; ++c) take_tile(g, c, row0[c], 0u);
    }
    };
    walk();
    if constexpr (P::kTurns == 2) {
        v16f o_first[kDB];
#pragma unroll
        for (int db = 0; db < kDB; ++db) {
            o_first[db] = o[db];
#pragma unroll
            for (int j = 0; j < 16; ++j) o[db][j] = 0.f;
        }
        const float ref_first = ref, l_first = l_run + __shfl_xor(l_run, 32);
        ref = -INFINITY;
        l_run = 0.f;
        turn = 1;
        wbase = 0;
        if (it.n_list > 0) win = it.list[min(lane, it.n_list - 1)];
        walk();
        // as two streams are merged below
        const float l_second = l_run + __shfl_xor(l_run, 32), top = fmaxf(fmaxf(-INFINITY, ref_first), ref);
        const float first = (ref_first == top) ? 1.0f : __builtin_amdgcn_exp2f(ref_first - top);
        const float second = (ref == top) ? 1.0f : __builtin_amdgcn_exp2f(ref - top);
        l_run = __builtin_fmaf(l_first, first, l_second * second);
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int j = 0; j < 16; ++j) o[db][j] = __builtin_fmaf(o_first[db][j], first, o[db][j] * second);
        ref = top;
    }
    }
    }

    // ---- merge the streams of a query group (stream order), normalise, store ----
    float l = P::kTurns == 2 ? l_run : l_run + __shfl_xor(l_run, 32);
    if constexpr (P::kS > 1) {
        __syncthreads();
        float* sO = reinterpret_cast<float*>(smem);                           // [kS - 1][kQ][32 channels-and-queries x kDB]
        float* sM = sO + (P::kS - 1) * P::kQ * 32 * D;                        // [kS][kQ][64]: reference, normaliser
        sM[(ws * P::kQ + wq) * 64 + lane] = half ? l : ref;
        __syncthreads();
        float top = -INFINITY;
#pragma unroll
        for (int s = 0; s < P::kS; ++s) top = fmaxf(top, sM[(s * P::kQ + wq) * 64 + l32]);
        const float mine = (ref == top) ? 1.0f : __builtin_amdgcn_exp2f(ref - top);      // (both -inf: nothing listed)
        if (ws > 0) {
            float* dst = sO + ((ws - 1) * P::kQ + wq) * 32 * D + lane;
#pragma unroll
            for (int db = 0; db < kDB; ++db)
#pragma unroll
                for (int j = 0; j < 16; ++j) dst[(db * 16 + j) * 64] = o[db][j] * mine;
        }
        __syncthreads();
        if (ws == 0) {
            l *= mine;
#pragma unroll
            for (int db = 0; db < kDB; ++db)
#pragma unroll
                for (int j = 0; j < 16; ++j) o[db][j] *= mine;
#pragma unroll
            for (int s = 1; s < P::kS; ++s) {
                const float r_s = sM[(s * P::kQ + wq) * 64 + l32], l_s = sM[(s * P::kQ + wq) * 64 + 32 + l32];
                l += l_s * ((r_s == top) ? 1.0f : __builtin_amdgcn_exp2f(r_s - top));
                const float* src = sO + ((s - 1) * P::kQ + wq) * 32 * D + lane;
#pragma unroll
                for (int db = 0; db < kDB; ++db)
#pragma unroll
                    for (int j = 0; j < 16; ++j) o[db][j] += src[(db * 16 + j) * 64];
            }
        }
        ref = top;
    }
    // Nothing is stored before every wavefront's results are known to stand: the plain pass reads Q again, which O may overlay.
    const bool writer = ws == 0 && qrow < N;
    const float inv = (l > 0.f) ? 1.0f / l : 0.f;
    bool bad = false, q_tiny = false;
    if constexpr (!BF16) {
        // the first parts tell (a value that is 0 in all of them is below 2^-134 and lost to no purpose beside keys under kHuge)
        typedef unsigned short v2us __attribute__((ext_vector_type(2)));
        v2us least = {0xffff, 0xffff}, most = {0, 0};
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks)
            if (ks % P::kS == ws) {                              // (the streams hold the same rows)
                union { v8bf v; v2us u[4]; } w;
                w.v = qf[ks][0];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const v2us twice = w.u[i] << 1;
                    least = __builtin_elementwise_min(least, (v2us)(twice - 1));
                    most = __builtin_elementwise_max(most, twice);
                }
            }
        q_tiny = min(least[0], least[1]) < (kTinyMagnitude >> 16);
        bad = max(most[0], most[1]) >= (__builtin_bit_cast(uint32_t, kHuge) >> 15);
    }
    if (writer) {
        float check = l;
        uint32_t least = ~0u;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float val = o[db][j] * inv;
                check += fabsf(val) * 0.f;                       // NaN as soon as one value is not finite
                if constexpr (!BF16) least = min(least, nonzero_magnitude(val));
            }
        bad = bad || !(check > 0.f && check < INFINITY) || least < kTinyMagnitude;
    }
    bad = bad && it.n_list > 0;
    bool plain = __syncthreads_or((bad || (q_tiny && it.n_list > 0)) ? 1 : 0) != 0;
    if constexpr (!BF16) {
        // (tiny values of Q are at home among zeros; they matter beside huge keys alone)
        if (plain && !__syncthreads_or(bad ? 1 : 0)) plain = __syncthreads_or(holds_huge_keys<D, BS>(it) ? 1 : 0) != 0;
    }
    if (writer && !plain) {
        char* dst = it.O + (int64_t)qrow * it.row_bytes;
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int ch = db * 32 + q4 * 8 + half * 4;
                v4f32 val;
#pragma unroll
                for (int i = 0; i < 4; ++i) val[i] = o[db][q4 * 4 + i] * inv;
                if constexpr (BF16) {
                    v4bf r;
#pragma unroll
                    for (int i = 0; i < 4; ++i) r[i] = (__bf16)val[i];
                    *reinterpret_cast<v4bf*>(dst + ch * 2) = r;
                } else {
                    *reinterpret_cast<v4f32*>(dst + ch * 4) = val;
                }
            }
        if (it.lse && half == 0)      // the two terms in 64 bits: the reference is a rounded multiple of the scale
            it.lse[qrow] = (l > 0.f) ? (float)((double)ref * 0.69314718055994531 + log((double)l)) : -INFINITY;
    }
    if (plain) plain_block<BF16, D, BS, L>(it, reinterpret_cast<float*>(smem));
}

// Measured against the vector-ALU kernel before it (one thread, eight logits and D / 8 channels of a row; 16 TFLOP/s at
// d = 64, 7 at d = 128): bf16 d = 64, 17 550 tokens x 12 heads, block 64, 32 % of the blocks kept (0.30 TFLOP)
// 18.43 -> 0.70 ms, bound by the vector ALU (some 150 instructions a tile, 16 of them exponentials, beside 16 matrix
// instructions); fp32 d = 128, 6144 tokens x 8 heads, block 128, 48 % (0.073 TFLOP, 384 workgroups: a round and a half)
// 10.21 -> 0.53 ms, and 0.53 -> 0.45 with the exponentials, both splits and their LDS traffic placed between the matrix
// instructions (5000 cycles a tile for 96 of 33: what is left is the issue of 800 instructions by one wavefront).  The packed split (one conversion per pair and part), the guard by the sum and the two buffers at
// d = 128 were worth 0.784 -> 0.70 and 0.617 -> 0.51.  Error against 64 bits (2-norm): fp32 d = 128 O 1.9e-6 -> 1.4e-6,
// d = 64 1.15e-6 -> 0.7e-6; log-sum-exp 3.3e-8..4.8e-8 -> 2.9e-8..3.8e-8.
// Block size 32, fp32 d = 64, 2048 tokens x 2 heads, all blocks: 700 us with the vector ALU, 45 us with four wavefronts that
// share stages behind barriers, 24 to 30 us with eight that walk alone.
// The fp32 kernels at d = 128 hold 96 registers of Q parts and run one wavefront per SIMD; those at d = 64 run two, bf16 at d = 64,
// which fits 128 registers, four, bf16 at d = 128 two or three.
template <bool BF16, int D, int BS, int L>
__global__ __launch_bounds__((Plan<BF16, D, BS, L>::kThreads)) __attribute__((amdgpu_waves_per_eu(Plan<BF16, D, BS, L>::kPerSimd)))
void k_attn_split(AttnArgs a) { attn_split_body<BF16, D, BS, L>(a); }

template <bool BF16, int D, int BS, int L = kAnyLaunch>
hipError_t launch_t(const AttnArgs& a, hipStream_t s) {
    using P = Plan<BF16, D, BS, L>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_attn_split<BF16, D, BS, L>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, P::kLdsBytes);
    if (e != hipSuccess) return e;
    const int total = a.Sb * a.td.H * a.td.B, grid = (total + 7) / 8 * 8;          // every XCD gets the same number of slots
    hipLaunchKernelGGL((k_attn_split<BF16, D, BS, L>), dim3(grid), dim3(P::kThreads), P::kLdsBytes, s, a);
    return hipGetLastError();
}

template <bool BF16, int D>
hipError_t launch_d(const AttnArgs& a, hipStream_t s) {
    return a.Bs == 128 ? launch_t<BF16, D, 128>(a, s) : a.Bs == 64 ? launch_t<BF16, D, 64>(a, s) : launch_t<BF16, D, 32>(a, s);
}

}  // namespace

// fp32, d = 64, block size 128: the number of query blocks beyond which their workgroups take the streams in turn.  The shorter a walk, the more
// its ends, where all eight wavefronts wait, weigh: blocks per compute unit at which eight wavefronts cease to be faster, one or two rows of
// blocks (256 tokens) 1.0, 8 rows 1 to 3, 16 rows 2 to 4.5, 24 and 32 rows 6.5 to 7.5, 40 and 80 rows 8.  (Eight / in turn: 800 blocks of 256
// tokens 68.8 / 53.8 us, 320 of 1024 69.4 / 72.6 and 91.5 / 82.9, 1040 of 2048 262 / 253, 1200 272 / 287, 1536 of 3072 403 / 415, 1920 543 / 523,
// 1800 of 5120 592 / 603, 2560 779 / 743.)
static int64_t many_blocks(const AttnArgs& a) { return (int64_t)a.cus * (a.Sb <= 8 ? 1 : a.Sb <= 16 ? 4 : a.Sb <= 32 ? 7 : 8); }

hipError_t launch_attn_split(const AttnArgs& a, hipStream_t s) {
    const int64_t blocks = (int64_t)a.Sb * a.td.H * a.td.B;
    if (a.td.d == 64 && a.bf16 && a.Bs == 32 && blocks <= a.cus) return launch_t<true, 64, 32, kFewBlocks>(a, s);
    if (a.td.d == 64 && !a.bf16 && a.Bs == 128 && blocks > many_blocks(a)) return launch_t<false, 64, 128, kManyBlocks>(a, s);
    if (a.td.d == 64) return a.bf16 ? launch_d<true, 64>(a, s) : launch_d<false, 64>(a, s);
    if (a.td.d == 128) return a.bf16 ? launch_d<true, 128>(a, s) : launch_d<false, 128>(a, s);
    return hipErrorNotSupported;
}

}  // namespace dr
