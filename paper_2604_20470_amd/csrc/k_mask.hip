// Stage (b): candidate geometry, per-row selection and CSR emission.  gfx950 only.
//
//   k_class_map  integer interval arithmetic on the radial window (paper Eqs. 3, 6, 7 and the
//                density rule); one wavefront classifies one (query block, key block) pair,
//                lanes own columns, ballots count active columns.
//   k_select     one workgroup per (batch, mask, query block) row: compacts the selectable
//                blocks into LDS as 64-bit keys (score descending, key block ascending), then
//                (rows of more than 1024 key blocks; below, one wavefront per row: k_select_wave, k_select_mass)
//                static top-k: radix selection of the k-th smallest key, keep every key up to it
//                (paper Eq. 8 k rule); dynamic: bitonic sort and the cumulative-mass prefix
//                (keep-one fallback of Eq. 11 / Algorithm 1).
//                In the seeded uniform mode (Eq. 8 as worded in the paper) the key is a
//                counter-based hash of (seed, query block, key block) instead of the score.
//   k_select_zscore  the paper's dynamic rule (Eqs. 10-11) per row: lanes own candidate sets
//                (frame distance, side), standardise the scores of a set in fp64 and keep
//                z >= tau_1 / tau_2, with the keep-one fallback.
//   k_emit*      per row: offset = sum of the previous rows' counts, bit-expansion to
//                ascending key-block indices.
//   k_mask_short both, for masks of at most 32 rows.
#include "dr_internal.h"

namespace dr {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// grid: (Sb)   one workgroup per query block, waves stride over key blocks
__global__ __launch_bounds__(kThreads) void k_class_map(Geometry g, FrameTab tab, uint8_t* __restrict__ class_map,
                                                        int32_t* __restrict__ row_sel,
                                                        unsigned long long* __restrict__ totals) {
    __shared__ int s_sel, s_cand;
    const int qb = blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = lane_id();
    if (threadIdx.x == 0) { s_sel = 0; s_cand = 0; }
    __syncthreads();
    const int r0 = qb * g.Bs, r1 = min(g.N, r0 + g.Bs);
    const int i0 = r0 / g.Nt, i1 = (r1 - 1) / g.Nt;
    const int row_min = (r1 - r0 == g.Bs) ? g.row_min_full : g.row_min_tail;
    int n_sel = 0, n_cand = 0;
    for (int kb = wave; kb < g.Sb; kb += kWaves) {
        const int c0 = kb * g.Bs, c1 = min(g.N, c0 + g.Bs);
        const int j0 = c0 / g.Nt, j1 = (c1 - 1) / g.Nt;
        const int gap = max(0, max(j0 - i1, i0 - j1));
        int cls;
        if (gap <= 1) {
            cls = 3;
        } else {
            int n_active = 0;
            for (int cbase = 0; cbase < c1 - c0; cbase += 64) {
                const int col = cbase + lane;
                bool active = false;
                if (col < c1 - c0) {
                    const int q = c0 + col;
                    const int j = q / g.Nt, v = q - j * g.Nt;
                    int cnt = 0;
                    for (int i = i0; i <= i1; ++i) {
                        const int t = abs(i - j);
                        if (tab.flags[t] & 1) {
                            const int w = tab.w[t];
                            const int u_lo = max(r0, i * g.Nt) - i * g.Nt;
                            const int u_hi = min(r1, (i + 1) * g.Nt) - 1 - i * g.Nt;
                            cnt += max(0, min(u_hi, v + w) - max(u_lo, v - w) + 1);
                        }
                    }
                    active = cnt >= row_min;
                }
                n_active += __popcll(__ballot(active));
            }
            const int col_min = (c1 - c0 == g.Bs) ? g.col_min_full : g.col_min_tail;
            cls = (n_active >= col_min) ? ((tab.flags[gap] >> 1) & 3) : 0;
        }
        if (lane == 0) class_map[(int64_t)qb * g.Sb + kb] = (uint8_t)cls;
        n_cand += (cls != 0);
        n_sel += (cls == 1 || cls == 2);
    }
    if (lane == 0) { atomicAdd(&s_sel, n_sel); atomicAdd(&s_cand, n_cand); }
    __syncthreads();
    if (threadIdx.x == 0) {
        row_sel[qb] = s_sel;
        atomicAdd(&totals[0], (unsigned long long)s_cand);
        atomicMax(&totals[1], (unsigned long long)s_sel);
    }
}

// Sort key, ascending order == (NEAR before FAR when ranked separately), score descending, kb ascending.
//   bit 63      far flag (only when the two classes are ranked separately)
//   bits 62..31 bitwise complement of the order-preserving integer image of the score
//   bits 30..0  key-block index
__device__ __forceinline__ uint64_t make_key(float s, int kb, bool far_bit) {
    s = s + 0.0f;                                  // -0 -> +0
    uint32_t u = __float_as_uint(s);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending unsigned == ascending float
    u = ~u;                                        // descending
    return ((uint64_t)(far_bit ? 1 : 0) << 63) | ((uint64_t)u << 31) | (uint64_t)(uint32_t)kb;
}
__device__ __forceinline__ float key_score(uint64_t key) {
    uint32_t u = ~(uint32_t)(key >> 31);
    u = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
    return __uint_as_float(u);
}
__device__ __forceinline__ int key_block(uint64_t key) { return (int)(key & 0x7fffffffu); }

// MurmurHash3's 32-bit finaliser; the sample key of block pair (qb, kb) under a seed
__device__ __forceinline__ uint32_t fmix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}
__device__ __forceinline__ uint64_t make_sample_key(uint32_t seed, int qb, int kb, bool far_bit) {
    const uint32_t h = fmix32(fmix32(seed ^ fmix32((uint32_t)qb)) + (uint32_t)kb);
    return ((uint64_t)(far_bit ? 1 : 0) << 63) | ((uint64_t)h << 31) | (uint64_t)(uint32_t)kb;
}

// keep bitmask of one row -> global memory, and the row's count
template <int kT = kThreads>
__device__ __forceinline__ void store_row(const uint32_t* keep, int words, int64_t row, uint32_t* __restrict__ keepbits,
                                          int32_t* __restrict__ counts, int* s_cnt) {
    int c = 0;
    for (int i = threadIdx.x; i < words; i += kT) {
        const uint32_t wv = keep[i];
        keepbits[row * words + i] = wv;
        c += __popc(wv);
    }
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
    if (lane_id() == 0) atomicAdd(s_cnt, c);
    __syncthreads();
    if (threadIdx.x == 0) counts[row] = *s_cnt;
}

__device__ __forceinline__ int keep_count(int n, double ratio) {
    if (n == 0) return 0;
    const int k = (int)floor((double)n * ratio);
    return max(1, k);
}

// The k-th smallest (k = 1 .. n) of n distinct 64-bit keys in LDS: most-significant-digit-first radix selection,
// eight bits per pass.  A pass counts, among the keys that agree with the digits fixed so far, how many fall in each
// of the 256 values of the next digit (thread t owns bin t), scans the counts and descends into the bin that holds
// rank k.  O(n) per pass instead of the O(n log^2 n) of a full sort: the static rules only need the set of the k
// smallest keys, not their order.  All threads of the workgroup call it and all receive the key.
__device__ uint64_t kth_smallest(const uint64_t* keys, int n, int k, uint32_t* hist, int* s_wave, int* s_pick) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    uint64_t prefix = 0ull, mask = 0ull;
    int rank = k;
    for (int shift = 56; shift >= 0; shift -= 8) {
        hist[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < n; i += kThreads) {
            const uint64_t key = keys[i];
            if ((key & mask) == prefix) atomicAdd(&hist[(uint32_t)(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        const int h = (int)hist[tid];
        int incl = h;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        for (int i = 0; i < wave; ++i) incl += s_wave[i];
        if (incl - h < rank && rank <= incl) { s_pick[0] = tid; s_pick[1] = rank - (incl - h); }
        __syncthreads();
        prefix |= (uint64_t)(uint32_t)s_pick[0] << shift;
        mask |= 0xffull << shift;
        rank = s_pick[1];
    }
    return prefix;
}

// grid: (Sb, masks, B).  LDS: keys[sort_cap] u64 | mass[sort_cap] f64 (dynamic mode) | keep[words] u32
__global__ __launch_bounds__(kThreads) void k_select(const uint8_t* __restrict__ class_map,
                                                     const float* __restrict__ scores, int masks, int Sb,
                                                     SelectArgs a, uint32_t* __restrict__ keepbits,
                                                     int32_t* __restrict__ counts) {
    extern __shared__ unsigned char smem[];
    uint64_t* keys = reinterpret_cast<uint64_t*>(smem);
    double* mass = reinterpret_cast<double*>(smem + (size_t)a.sort_cap * 8);
    const int words = (Sb + 31) / 32;
    uint32_t* keep = reinterpret_cast<uint32_t*>(smem + (size_t)a.sort_cap * (a.mode == 1 ? 16 : 8));
    __shared__ int s_n, s_near, s_k, s_cnt;

    const int qb = blockIdx.x, m = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int64_t row = ((int64_t)b * masks + m) * Sb + qb;
    const float* srow = scores + row * Sb;
    const uint8_t* crow = class_map + (int64_t)qb * Sb;

    for (int i = tid; i < words; i += kThreads) keep[i] = 0u;
    if (tid == 0) { s_n = 0; s_near = 0; s_k = 0x7fffffff; s_cnt = 0; }
    __syncthreads();
    for (int kb = tid; kb < Sb; kb += kThreads) {
        const int c = crow[kb];
        if (c == 3) {
            atomicOr(&keep[kb >> 5], 1u << (kb & 31));
        } else if (c != 0) {
            const int pos = atomicAdd(&s_n, 1);
            const bool far_bit = a.two_ratio && c == 2;
            if (a.two_ratio && c == 1) atomicAdd(&s_near, 1);
            keys[pos] = (a.mode == 3) ? make_sample_key(a.seed, qb, kb, far_bit) : make_key(srow[kb], kb, far_bit);
        }
    }
    __syncthreads();
    const int n = s_n;
    if (n > 0 && a.mode != 1) {
        // static top-k / seeded sample: keep the k smallest keys (with two ratios: the k_near smallest NEAR keys and the
        // k_far smallest FAR keys; every NEAR key is below every FAR key)
        __shared__ uint32_t s_hist[kThreads];
        __shared__ int s_wave4[kWaves], s_pick[2];
        const int n_near = a.two_ratio ? s_near : n;
        const int k_near = keep_count(n_near, a.ratio);
        const int k_far = a.two_ratio ? keep_count(n - n_near, a.ratio_far) : 0;
        const uint64_t none = 0ull;
        const uint64_t t_near = k_near > 0 ? kth_smallest(keys, n, k_near, s_hist, s_wave4, s_pick) : none;
        const uint64_t t_far = k_far > 0 ? kth_smallest(keys, n, n_near + k_far, s_hist, s_wave4, s_pick) : none;
        for (int i = tid; i < n; i += kThreads) {
            const uint64_t key = keys[i];
            const bool far_key = (key >> 63) != 0;
            const bool sel = far_key ? (k_far > 0 && key <= t_far) : (k_near > 0 && key <= t_near);
            if (sel) { const int kb = key_block(key); atomicOr(&keep[kb >> 5], 1u << (kb & 31)); }
        }
    } else if (n > 0) {
        int P = 1;
        while (P < n) P <<= 1;
        for (int i = n + tid; i < P; i += kThreads) keys[i] = ~0ull;
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = tid; i < P; i += kThreads) {
                    const int ixj = i ^ j;
                    if (ixj > i) {
                        const uint64_t x = keys[i], y = keys[ixj];
                        const bool up = (i & k) == 0;
                        if ((x > y) == up) { keys[i] = y; keys[ixj] = x; }
                    }
                }
                __syncthreads();
            }
        }
        {
            const double top = (double)key_score(keys[0]);
            for (int i = tid; i < n; i += kThreads) mass[i] = exp((double)key_score(keys[i]) - top);
            __syncthreads();
            if (tid == 0) {          // one-by-one summation in the total order: the order is part of the definition
                double cum = 0.0;
                int i = 0;
                for (; i + 8 <= n; i += 8) {          // eight loads in flight, then the dependent chain of additions
                    double v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = mass[i + e];
#pragma unroll
                    for (int e = 0; e < 8; ++e) { cum = cum + v[e]; v[e] = cum; }
#pragma unroll
                    for (int e = 0; e < 8; ++e) mass[i + e] = v[e];
                }
                for (; i < n; ++i) { cum = cum + mass[i]; mass[i] = cum; }
            }
            __syncthreads();
            const double target = a.tau * mass[n - 1];
            for (int i = tid; i < n; i += kThreads)
                if (mass[i] >= target && (i == 0 || !(mass[i - 1] >= target))) atomicMin(&s_k, i + 1);
            __syncthreads();
            const int k = max(1, min(n, s_k));
            for (int i = tid; i < k; i += kThreads) {
                const int kb = key_block(keys[i]);
                atomicOr(&keep[kb >> 5], 1u << (kb & 31));
            }
        }
    }
    __syncthreads();
    store_row(keep, words, row, keepbits, counts, &s_cnt);
}

// a wave's LDS operations execute in order; the fence keeps the compiler from moving reads above writes
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Static top-k / seeded sample for rows of at most 1024 key blocks: ONE wave per row, four rows per workgroup, no
// barrier.  Lane l holds the keys of key blocks l, l + 64, ... in registers, complemented (kSlots 64-bit values; 0
// where there is no key).  The classes arrive as lane masks (k_class_bits), so counting the selectable and the FAR
// keys, dropping the others and adding the forced ones are scalar operations on those masks.  The rules need the SET
// of the k smallest keys, not their order, and the keys are distinct, so any threshold that exactly k complemented
// keys reach describes it.  The threshold is built bit by bit from the top: with the bits kept so far and the next
// one set, count the keys that reach it -- per register one unsigned compare into a lane mask and a population
// count, nothing is rewritten; keep the bit when at least k do, and stop as soon as exactly k do (at the highest bit
// in which the k-th and the (k+1)-th key differ: 15 to 20 steps on real scores).  Only when keys with equal high
// words straddle rank k (equal scores) does the search go on in the low words of that group; the key-index bits
// above log2(Sb) are equal in every key and take no vote.  For a small k the search runs on a short list of one
// register instead (kth_smallest_wave_short_list).  A ballot of "selected" over the wave IS the pair of keep words
// of those 64 key blocks.  Same keys, same counts as k_select: the keep bitmaps are identical.  With one workgroup
// per row, k_select holds 8 rows per CU in flight, each waiting on its barriers; this holds up to 32.
// grid: ceil(B * masks * Sb / 4).
constexpr int kWaveSelectMaxSlots = kWaveSelectMaxBlocks / 64;
constexpr int64_t kWaveSelectMinRows = 1;
constexpr int64_t kWaveSelectPackRows = 2048;
static_assert(kWaveSelectMaxSlots <= 64, "one bit per slot in a 64-bit word");

template <int kSlots>
struct WaveKeys {
    uint64_t c[kSlots];                           // ~key; 0 = no key here
};

// selected <=> the complemented key, as a 64-bit number, is at least (hi, lo); never (0, 0)
struct WaveThreshold {
    uint32_t hi, lo;
};

template <int kSlots>
__device__ __forceinline__ WaveThreshold kth_smallest_wave(const WaveKeys<kSlots>& w, int k, int index_bits) {
    uint32_t t_hi = 0u;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t t = t_hi | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < kSlots; ++i) cnt += __popcll(__ballot((uint32_t)(w.c[i] >> 32) >= t));
        if (cnt == k) return WaveThreshold{t, 0u};    // wave-uniform
        if (cnt > k) t_hi = t;
    }
    // t_hi is the high word of the k-th largest complemented key, and more keys than rank k asks for share it
    int above = 0;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) above += __popcll(__ballot((uint32_t)(w.c[i] >> 32) > t_hi));
    const int k_low = k - above;
    uint32_t t_lo = 0x7fffffffu & ~((1u << index_bits) - 1u);   // ones in every key: the index bits no key block has
    auto vote = [&](uint32_t bit_mask) -> bool {
        const uint32_t t = t_lo | bit_mask;
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < kSlots; ++i)
            cnt += __popcll(__ballot((uint32_t)(w.c[i] >> 32) == t_hi && (uint32_t)w.c[i] >= t));
        if (cnt >= k_low) t_lo = t;
        return cnt == k_low;
    };
    if (vote(1u << 31)) return WaveThreshold{t_hi, t_lo};
    for (int bit = index_bits - 1; bit >= 0; --bit)
        if (vote(1u << bit)) break;
    return WaveThreshold{t_hi, t_lo};
}

// The same answer for a small k, by way of a short list.  The k-th largest of the 64 lanes' own maxima is a lower
// bound of the k-th largest key, so the keys that reach it hold the k largest; when they are at most 64 (a few more
// than k on real scores) they are packed one per lane through `list` (64 words of LDS that belong to this wave)
// and the search runs on one register instead of kSlots.  Only the high words take part in the bound, so keys with
// equal high words all make the list.  Returns false, with nothing decided, when the list would not fit or fewer
// than k lanes hold a key.
constexpr int kShortListMaxK = 40;

template <int kSlots>
__device__ __forceinline__ bool kth_smallest_wave_short_list(const WaveKeys<kSlots>& w, int k, int index_bits,
                                                             uint64_t* list, WaveThreshold* out) {
    uint32_t lane_max = 0u;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) lane_max = max(lane_max, (uint32_t)(w.c[i] >> 32));
    uint32_t bound = 0u;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t t = bound | (1u << bit);
        const int cnt = __popcll(__ballot(lane_max >= t));
        if (cnt >= k) bound = t;
        if (cnt == k) break;
    }
    if (bound == 0u) return false;
    uint64_t reach[kSlots];
    int listed = 0;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        reach[i] = __ballot((uint32_t)(w.c[i] >> 32) >= bound);
        listed += __popcll(reach[i]);
    }
    if (listed > 64) return false;
    if (listed == k) {                            // the list is the answer
        *out = WaveThreshold{bound, 0u};
        return true;
    }
    int at = 0;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        const int mine = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(reach[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)reach[i], 0u));
        if (__builtin_amdgcn_inverse_ballot_w64(reach[i])) list[mine] = w.c[i];
        at += __popcll(reach[i]);
    }
    wave_lds_fence();
    WaveKeys<1> shortlist;
    shortlist.c[0] = (lane_id() < listed) ? list[lane_id()] : 0ull;
    __builtin_amdgcn_wave_barrier();
    // more keys than k are listed, so the threshold found lies above the bound and counts the same keys in the row
    *out = kth_smallest_wave<1>(shortlist, k, index_bits);
    return true;
}

// The class map as lane masks, for the one-wave-per-row selection: class_bits[qb][slot][3] holds, for the 64 key
// blocks of a slot, one bit per key block: selectable (NEAR or FAR), FAR, forced.  A row has `slots` entries, the
// register slots of the selection kernel that will read it; those past the row's end are 0.  Written once per
// geometry.  grid: ceil(Sb / 4); one wave per row.
__global__ __launch_bounds__(kThreads) void k_class_bits(const uint8_t* __restrict__ class_map, int Sb, int slots,
                                                         uint64_t* __restrict__ class_bits) {
    const int lane = lane_id(), qb = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (qb >= Sb) return;
    for (int i = 0; i < slots; ++i) {
        const int kb = i * 64 + lane;
        const int c = (kb < Sb) ? class_map[(int64_t)qb * Sb + kb] : 0;
        const uint64_t sel = __ballot(c == 1 || c == 2), far = __ballot(c == 2), forced = __ballot(c == 3);
        if (lane < 3) class_bits[((int64_t)qb * slots + i) * 3 + lane] = lane == 0 ? sel : lane == 1 ? far : forced;
    }
}

// Reductions and scans over a wavefront in the vector ALU's own lane moves (a shuffle goes through the LDS, some 120 cycles
// each, and a row's selection is a chain of them).  `none`: what lanes without a source read.
template <int kCtrl, int kRows, typename T>
__device__ __forceinline__ T moved(T none, T x) {
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_update_dpp((int)none, (int)x, kCtrl, kRows, 0xf, false);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)none, (int)(uint32_t)x, kCtrl, kRows, 0xf, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(none >> 32), (int)(uint32_t)(x >> 32), kCtrl, kRows, 0xf, false);
        return (T)(((uint64_t)hi << 32) | lo);
    }
}
// inclusive scan: rows of sixteen (row_shr 1, 2, 4, 8), then the rows' last lanes into the rows behind (row_bcast 15, 31)
template <typename T, class Op>
__device__ __forceinline__ T wave_scan(T x, T none, Op&& op) {
    x = op(x, moved<0x111, 0xf>(none, x));
    x = op(x, moved<0x112, 0xf>(none, x));
    x = op(x, moved<0x114, 0xf>(none, x));
    x = op(x, moved<0x118, 0xf>(none, x));
    x = op(x, moved<0x142, 0xa>(none, x));
    x = op(x, moved<0x143, 0xc>(none, x));
    return x;
}
template <typename T>
__device__ __forceinline__ T from_lane(T x, int lane) {                 // lane: the same in every lane
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_readlane((int)x, lane);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
        return (T)(((uint64_t)hi << 32) | lo);
    }
}
template <typename T> __device__ __forceinline__ T wave_max(T x) { return from_lane(wave_scan(x, (T)0, [](T a, T b) { return a > b ? a : b; }), 63); }
template <typename T> __device__ __forceinline__ T wave_min(T x) { return from_lane(wave_scan(x, (T)~(T)0, [](T a, T b) { return a < b ? a : b; }), 63); }
template <typename T> __device__ __forceinline__ T wave_prefix(T x) { return wave_scan(x, (T)0, [](T a, T b) { return (T)(a + b); }); }      // inclusive sums

// ascending unsigned == ascending float, -0 counted as +0
__device__ __forceinline__ uint32_t score_image(float s) {
    const uint32_t u = __float_as_uint(s + 0.0f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

__device__ __forceinline__ float image_score(uint32_t v) { return __uint_as_float((v & 0x80000000u) ? (v & 0x7fffffffu) : ~v); }

// One row in the registers of a wave: the complemented keys and the classes as lane masks.
template <int kSlots>
struct WaveRow {
    WaveKeys<kSlots> w;
    uint64_t m_sel[kSlots], m_far[kSlots], m_forced[kSlots];      // m_far is empty unless the classes rank apart
    int n, n_far;
};
// complemented key of key block kb: (not FAR) << 63 | image << 31 | ~kb (31 bits), the image being the order-preserving
// integer of the score (or the complement of the sample hash); 0 where the class selects nothing
template <int kSlots>
__device__ __forceinline__ void load_wave_row(const uint64_t* __restrict__ class_bits, const float* __restrict__ scores, int64_t row,
                                              int qb, int Sb, const SelectArgs& a, WaveRow<kSlots>& r) {
    const int lane = lane_id();
    const float* srow = scores + row * Sb;
    const uint64_t* cb = class_bits + (int64_t)qb * (kSlots * 3);
    // every load of the row is issued before the first is used: the scores of all kSlots * 64 positions (those past
    // the row's end read its last entry) and the lane masks of the classes
    float sc[kSlots];
    if (a.mode != 3) {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) sc[i] = srow[(uint32_t)min(i * 64 + lane, Sb - 1)];
    } else {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) sc[i] = 0.f;
    }
    const uint64_t ranked_apart = a.two_ratio ? ~0ull : 0ull;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        r.m_sel[i] = cb[i * 3 + 0];
        r.m_far[i] = cb[i * 3 + 1] & ranked_apart;
        r.m_forced[i] = cb[i * 3 + 2];
    }
    r.n = 0;
    r.n_far = 0;
    const uint32_t seed_row = (a.mode == 3) ? fmix32(a.seed ^ fmix32((uint32_t)qb)) : 0u;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        const int kb = i * 64 + lane;
        const uint32_t v = (a.mode == 3) ? ~fmix32(seed_row + (uint32_t)kb) : score_image(sc[i]);
        const bool selectable = __builtin_amdgcn_inverse_ballot_w64(r.m_sel[i]);
        const bool far_key = __builtin_amdgcn_inverse_ballot_w64(r.m_far[i]);
        const uint32_t hi = (v >> 1) | (far_key ? 0u : 0x80000000u), lo = (v << 31) | (0x7fffffffu ^ (uint32_t)kb);
        r.w.c[i] = selectable ? (((uint64_t)hi << 32) | lo) : 0ull;
        r.n += __popcll(r.m_sel[i]);
        r.n_far += __popcll(r.m_far[i]);
    }
}
// The compiler's own v_writelane (it has no builtin), between whose sources and other vector instructions the compiler keeps the wait states
// that the chip asks for; inline assembly it does not look into.
__device__ uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");
// a row's keep words, one per lane (a store for each slot's pair costs three times the instructions), and its count
template <int kSlots, class Kept>
__device__ __forceinline__ void store_keep_words(int64_t row, int Sb, uint32_t* __restrict__ keepbits, int32_t* __restrict__ counts, Kept&& kept_of) {
    static_assert(2 * kSlots <= 64, "a word per lane");
    const int lane = lane_id(), words = (Sb + 31) / 32;
    int kept = 0;
    uint32_t word = 0u;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        const uint64_t m = kept_of(i);                            // (past the row's end: 0)
        kept += __popcll(m);
        word = write_lane((uint32_t)m, 2 * i, word);
        word = write_lane((uint32_t)(m >> 32), 2 * i + 1, word);
    }
    if (lane < words) keepbits[row * words + lane] = word;
    if (lane == 0) counts[row] = kept;
}
// forced blocks, keys that reach c_near, FAR keys that reach c_far
template <int kSlots>
__device__ __forceinline__ void store_wave_row(const WaveRow<kSlots>& r, uint64_t c_near, uint64_t c_far, bool two_ratio, int64_t row,
                                               int Sb, uint32_t* __restrict__ keepbits, int32_t* __restrict__ counts) {
    store_keep_words<kSlots>(row, Sb, keepbits, counts, [&](int i) {
        uint64_t m = r.m_forced[i] | __ballot(r.w.c[i] >= c_near);
        if (two_ratio) m |= __ballot(r.w.c[i] >= c_far) & r.m_far[i];
        return m;
    });
}
__device__ __forceinline__ int bits_of(int Sb) {                        // of a key-block index
    int bits = 0;
    while ((1 << bits) < Sb) ++bits;
    return bits;
}
// The thresholds of the static rules: NEAR keys that reach c_near are kept, FAR keys that reach c_far (rule with two ratios).
// list: 64 words of LDS that belong to this wave.
template <int kSlots>
__device__ __forceinline__ void select_wave_row(const WaveRow<kSlots>& r, int index_bits, const SelectArgs& a, uint64_t* list, uint64_t* c_near,
                                                uint64_t* c_far) {
    WaveThreshold t_near{0u, 0u}, t_far{0u, 0u};
    int k_near = 0, k_far = 0;
    if (r.n > 0) {
        const int n_near = r.n - r.n_far;
        k_near = keep_count(n_near, a.ratio);
        k_far = a.two_ratio ? keep_count(r.n_far, a.ratio_far) : 0;
        if (k_near > 0 && !(k_near <= kShortListMaxK && kth_smallest_wave_short_list<kSlots>(r.w, k_near, index_bits, list, &t_near)))
            t_near = kth_smallest_wave<kSlots>(r.w, k_near, index_bits);
        const int k_all = n_near + k_far;
        if (k_far > 0 && !(k_all <= kShortListMaxK && kth_smallest_wave_short_list<kSlots>(r.w, k_all, index_bits, list, &t_far)))
            t_far = kth_smallest_wave<kSlots>(r.w, k_all, index_bits);
    }
    // a NEAR key's complement has bit 63 set and so has every threshold of the NEAR ranking: no FAR key reaches it;
    // the FAR ranking's threshold is reached by every NEAR key and by the k_far best FAR keys.  With nothing to rank
    // the threshold is beyond every key.
    *c_near = k_near > 0 ? (((uint64_t)t_near.hi << 32) | t_near.lo) : ~0ull;
    *c_far = k_far > 0 ? (((uint64_t)t_far.hi << 32) | t_far.lo) : ~0ull;
}
template <int kSlots>
__global__ __launch_bounds__(kThreads) void k_select_wave(const uint64_t* __restrict__ class_bits,
                                                          const float* __restrict__ scores, int64_t rows_total, int Sb,
                                                          SelectArgs a, uint32_t* __restrict__ keepbits,
                                                          int32_t* __restrict__ counts) {
    __shared__ uint64_t s_list[kWaves][64];                       // a wave's short list of candidate keys
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;   // the same in every lane, and known to be
    if (row >= rows_total) return;
    // (which side of the loads this loop stands on changes how the compiler lays out the rest: 160 masks of 591 rows 107.0 us in front,
    // 110.9 behind; 80 masks of 1024 rows 139 in front, 133 behind)
    constexpr bool kBitsFirst = kSlots < 16;
    const int qb = (int)(row % Sb);
    int index_bits = 0;
    if constexpr (kBitsFirst) index_bits = bits_of(Sb);
    WaveRow<kSlots> r;
    load_wave_row<kSlots>(class_bits, scores, row, qb, Sb, a, r);
    if constexpr (!kBitsFirst) index_bits = bits_of(Sb);
    uint64_t c_near, c_far;
    select_wave_row<kSlots>(r, index_bits, a, s_list[wave], &c_near, &c_far);
    store_wave_row<kSlots>(r, c_near, c_far, a.two_ratio != 0, row, Sb, keepbits, counts);
}

// Cumulative mass for rows of at most 1024 key blocks, one wave per row.  The rule is a sum of fp64 exponentials one by
// one in score order, compared with tau times the whole sum: a serial chain behind a sort, if taken literally (k_select:
// 208 us at 40 x 591 rows; this kernel 23 with scores of a smooth field, more over other distributions; the vector ALU is busy for
// 92 % of the time that a compute unit has work, so what counts is instructions a row: 463, and 538, 29 us, before the keys were
// made without a test each and the keep words stored as one register).  Only the place where the prefix crosses the target is wanted, so it is
// looked for with fixed-point masses, without sorting (mass_crossing), first in 32 and, where those cannot tell, in 64
// bits; a row whose target lies within the error of the 64-bit sums (equal scores that hit it exactly, tau = 1) is decided by
// the literal chain, in this wave.
// LDS per wave: keys[cap] u64 | mass[cap] f64 over bins[256] u64 (the chain comes when the bins are done with), cap a power of two
// >= the largest selectable count of a row.  A quarter more rows in flight than with bins of their own, at 256 keys.
//
// One row in registers: keys as in WaveRow with all blocks in front of FAR ones, made for every position of the row; m_sel says which
// of them count.
template <int kSlots>
struct MassRow {
    uint64_t c[kSlots], m_sel[kSlots], m_forced[kSlots];
    int n;
};
template <int kSlots>
__device__ __forceinline__ void load_mass_row(const uint64_t* __restrict__ class_bits, const float* __restrict__ scores, int64_t row,
                                              int qb, int Sb, MassRow<kSlots>& r) {
    const int lane = lane_id();
    const char* srow = reinterpret_cast<const char*>(scores + row * Sb);
    const uint64_t* cb = class_bits + (int64_t)qb * (kSlots * 3);
    float sc[kSlots];                             // every load before the first is used; past the row's end its last entry
#pragma unroll
    for (int i = 0; i < kSlots; ++i) sc[i] = *reinterpret_cast<const float*>(srow + min((uint32_t)lane * 4u + (uint32_t)i * 256u, (uint32_t)(Sb - 1) * 4u));
    r.n = 0;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        r.m_sel[i] = cb[i * 3 + 0];
        r.m_forced[i] = cb[i * 3 + 2];
        r.n += __popcll(r.m_sel[i]);
    }
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        const uint32_t v = score_image(sc[i]), block = 0x7fffffffu - (uint32_t)(i * 64) - (uint32_t)lane;      // (the complement of its index)
        r.c[i] = ((uint64_t)(0x80000000u | (v >> 1)) << 32) | ((v << 31) | block);
    }
}
template <int kSlots>
__device__ __forceinline__ uint64_t kept_of_mass_row(const MassRow<kSlots>& r, int i, uint64_t threshold) {
    return r.m_forced[i] | (__ballot(r.c[i] >= threshold) & r.m_sel[i]);
}
constexpr int kBins = 256, kMaxTaken = 8;      // keys taken one by one from a bin
__host__ __device__ inline size_t select_mass_lds_bytes(int cap) { return (size_t)cap * 8 + (cap > kBins ? (size_t)cap * 8 : kBins * 8); }

__device__ __forceinline__ uint32_t key_image(uint64_t c) { return (uint32_t)(c >> 31); }
// The rule taken literally by one wave: the n keys (complemented, in LDS, room for a power of two of them) are sorted, the
// masses laid out in that order and added one by one; returns the key that ends the prefix.
__device__ __forceinline__ uint64_t mass_threshold_by_chain(int n, float top, double tau, uint64_t* keys, double* mass) {
    const int lane = lane_id();
    int P = 1;
    while (P < n) P <<= 1;
#pragma unroll 1
    for (int i = n + lane; i < P; i += 64) keys[i] = 0ull;
    wave_lds_fence();
#pragma unroll 1
    for (int k = 2; k <= P; k <<= 1) {
#pragma unroll 1
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll 2
            for (int t = lane; t < P / 2; t += 64) {
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const uint64_t x = keys[i], y = keys[i | j];
                if ((x < y) == ((i & k) == 0)) { keys[i] = y; keys[i | j] = x; }      // descending
            }
            wave_lds_fence();
        }
    }
#pragma unroll 1
    for (int i = lane; i < n; i += 64) mass[i] = exp((double)image_score(key_image(keys[i])) - (double)top);
    wave_lds_fence();
    // one-by-one summation in the total order: the order is part of the definition.  Every lane runs the chain; eight loads
    // are in flight ahead of the dependent additions, and the running sums replace the masses.
    double cum = 0.0;
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        double v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = mass[i + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) { cum = cum + v[e]; v[e] = cum; }
        if (lane == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) mass[i + e] = v[e];
        }
    }
    for (; i < n; ++i) {
        cum = cum + mass[i];
        if (lane == 0) mass[i] = cum;
    }
    wave_lds_fence();
    const double target = tau * cum;
    int k = n;                                              // the first running sum that reaches the target ends the prefix
#pragma unroll 1
    for (int i0 = 0; i0 < n; i0 += 64) {
        const uint64_t at = __ballot(i0 + lane < n && mass[min(i0 + lane, n - 1)] >= target);
        if (at) {
            k = i0 + __ffsll((unsigned long long)at);
            break;
        }
    }
    return keys[max(k, 1) - 1];
}

// The key that ends the prefix, by masses in fixed point (U: 32 or 64 bits; their sums do not depend on an order): the keys are
// dropped into 256 bins of equal width in score (monotone in the score), the bins are scanned, and the keys of the bin in
// which the sum crosses the target are taken from the top.  kLevels > 1: what a bin still holds after that many is binned
// again over its own range, or, where its scores are all the same, divided.  Nothing is decided when that does not reach the
// crossing, or when the target lies within `slack(total)`, the largest error of a prefix, of either side of it.
enum class Crossing { kFound, kTooClose, kTooMany };
template <int kLevels, typename U, class Mass, class Slack>
__device__ __forceinline__ Crossing mass_crossing(int n, float top, float bin_scale, double tau, const uint64_t* keys, U* bins, Mass&& mass_of,
                                              Slack&& slack, uint64_t* ends) {
    const int lane = lane_id();
    uint64_t low = 0ull, last = ~0ull;          // the keys still in question: low <= key < last
    double total = 0.0, target = 0.0;
    U prefix = 0, prev = 0;                     // mass of the keys from `last` up, and before the last of them
    bool crossed = false;
    for (int level = 0; level < kLevels && !crossed; ++level) {
        auto bin_of = [&](uint64_t c) { return (int)fminf((top - image_score(key_image(c))) * bin_scale, 255.0f); };
        auto asked = [&](uint64_t c) { return (kLevels == 1 || c >= low) && c < last; };
#pragma unroll
        for (int e = 0; e < 4; ++e) bins[lane * 4 + e] = 0;
        wave_lds_fence();
#pragma unroll 1
        for (int i = lane; i < n; i += 64)
            if (level == 0 || asked(keys[i])) atomicAdd(&bins[bin_of(keys[i])], mass_of(keys[i]));
        wave_lds_fence();
        const U part[4] = {bins[lane * 4], bins[lane * 4 + 1], bins[lane * 4 + 2], bins[lane * 4 + 3]};
        const U own = part[0] + part[1] + part[2] + part[3];
        const U incl = prefix + wave_prefix(own);
        if (level == 0) {
            total = (double)from_lane(incl, 63);
            target = tau * total;
        }
        const uint64_t reach = __ballot((double)incl >= target);      // (never empty: tau <= 1)
        const int l = reach ? __ffsll((unsigned long long)reach) - 1 : 63;
        U before = incl - own;
        int bin = lane * 4;
        bool found = false;
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (!found) {
                if ((double)(before + part[e]) >= target) found = true;
                else { before += part[e]; ++bin; }
            }
        bin = from_lane(bin, l);
        prefix = prev = from_lane(before, l);
        uint64_t best = 0ull, least = ~0ull;          // of the bin, of what is not taken yet
        for (int taken = 0; taken < kMaxTaken + (kLevels > 1) && !crossed; ++taken) {
            best = 0ull;
            least = ~0ull;
#pragma unroll 1
            for (int i = lane; i < n; i += 64) {
                const uint64_t c = keys[i];
                if (asked(c) && bin_of(c) == bin) {
                    best = c > best ? c : best;
                    if constexpr (kLevels > 1) least = c < least ? c : least;
                }
            }
            best = wave_max(best);
            if (best == 0ull || taken == kMaxTaken) break;
            last = best;
            prev = prefix;
            prefix += mass_of(best);
            crossed = (double)prefix >= target;
        }
        if (kLevels == 1 || crossed || best == 0ull) break;
        least = wave_min(least);
        if (key_image(least) == key_image(best)) {
            // equal masses, in key-block order, which is the order of the packed keys
            const U m = mass_of(best);
            const int j = m ? (int)fmin(ceil((target - (double)prefix) / (double)m), 65536.0) : 0;
            if (j < 1) break;
            int at = 0;
#pragma unroll 1
            for (int i0 = 0; i0 < n; i0 += 64) {
                const uint64_t c = i0 + lane < n ? keys[i0 + lane] : 0ull;
                const uint64_t equal = __ballot(c >= least && c <= best);
                const int nth = j - at;                                   // of this stretch
                at += __popcll(equal);
                if (at < j) continue;
                const uint64_t mine = __ballot(c >= least && c <= best &&
                                               (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(equal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)equal, 0u)) == nth - 1);
                last = from_lane(c, __ffsll((unsigned long long)mine) - 1);
                prev = prefix + (U)(j - 1) * m;
                prefix = prev + m;
                crossed = (double)prefix >= target && (double)prev < target;
                break;
            }
            break;
        }
        low = least;
        last = best + 1ull;
        top = image_score(key_image(best));
        bin_scale = 255.0f / (top - image_score(key_image(least)));
    }
    const double E = slack(total);
    *ends = last;
    if (!crossed) return Crossing::kTooMany;
    return (double)prev + E < tau * (total - E) && (double)prefix - E >= tau * (total + E) ? Crossing::kFound : Crossing::kTooClose;
}

// The threshold of the cumulative-mass rule: every selectable key that reaches it is kept.  `mine`: select_mass_lds_bytes(cap) of LDS
// that belong to this wave.
template <int kSlots, int kLevels>
__device__ __forceinline__ uint64_t select_mass_row(const MassRow<kSlots>& r, const SelectArgs& a, unsigned char* mine, int cap) {
    const int lane = lane_id();
    uint64_t* keys = reinterpret_cast<uint64_t*>(mine);
    double* mass = reinterpret_cast<double*>(mine + (size_t)cap * 8);
    unsigned char* bins = mine + (size_t)cap * 8;
    uint64_t threshold = ~0ull;
    const int n = r.n;
    if (n > 0) {
        int at = 0;
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const int pos = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(r.m_sel[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)r.m_sel[i], 0u));
            if (__builtin_amdgcn_inverse_ballot_w64(r.m_sel[i])) keys[pos] = r.c[i];
            at += __popcll(r.m_sel[i]);
        }
        wave_lds_fence();
        // (the packed keys are read from LDS again by every loop: few iterations, and registers for many waves)
        uint32_t image_max = 0u, image_min = ~0u;
#pragma unroll 1
        for (int i = lane; i < n; i += 64) {
            const uint32_t v = key_image(keys[i]);
            image_max = max(image_max, v);
            image_min = min(image_min, v);
        }
        image_max = wave_max(image_max);
        image_min = wave_min(image_min);
        const float top = image_score(image_max), range = top - image_score(image_min);
        const float bin_scale = (range > 0.f && range < INFINITY) ? 255.0f / range : 0.f;
        const int log_n = 32 - __clz(n);                    // n < 2^log_n: the sums of n masses below fit their types
        // tau = 1 ends the prefix where the running sum stops growing: at the last key when even the smallest mass is above
        // a rounding of the whole sum (at most n)
        const bool all = a.tau >= 1.0 && range < 34.0f - (float)log_n;
        const bool flat = range == 0.f;                     // every mass is 1: the running sum counts, in key-block order
        // (infinities and NaN, or finite scores further apart than a float holds: the chain is the definition)
        Crossing got = (a.tau >= 1.0 || flat || !(range < INFINITY)) ? Crossing::kTooMany : Crossing::kTooClose;
        if (!all && got == Crossing::kTooClose) {
            // 32 bits, exponentials in fp32.  The argument is off by at most 2^-23 |x| (and x e^-x <= 0.37), the
            // instruction by 2^-23 relative, rounding to a unit by one half.
            const float unit = __uint_as_float((uint32_t)(127 + 31 - log_n) << 23);
            got = mass_crossing<kLevels, uint32_t>(
                n, top, bin_scale, a.tau, keys, reinterpret_cast<uint32_t*>(bins),
                [&](uint64_t c) { return (uint32_t)__builtin_rintf(__builtin_amdgcn_exp2f((top - image_score(key_image(c))) * -1.44269504f) * unit); },
                [&](double total) { return total * 0x1p-21 + (double)n + 4.0; }, &threshold);
        }
        if (!all && got == Crossing::kTooClose) {
            // 64 bits, the rule's own exponentials: rounding to a unit, and the chain's own n roundings
            const double unit = __longlong_as_double((long long)(1023 + 62 - log_n) << 52);
            got = mass_crossing<kLevels, unsigned long long>(
                n, top, bin_scale, a.tau, keys, reinterpret_cast<unsigned long long*>(bins),
                [&](uint64_t c) { return (unsigned long long)__builtin_rint(exp((double)image_score(key_image(c)) - (double)top) * unit); },
                [&](double total) { return total * (double)(n + 8) * 0x1p-52 + (double)n + 4.0; }, &threshold);
        }
        if (all) threshold = 1ull;                          // every selectable key's complement is above 0
        else if (flat) threshold = keys[max(1, (int)ceil(a.tau * (double)n)) - 1];      // (packed in that order)
        else if (got != Crossing::kFound) threshold = mass_threshold_by_chain(n, top, a.tau, keys, mass);
    }
    return threshold;
}

// A row that the bins do not decide costs its wave a sort and the chain, 25 us at 1000 keys.  Among many rows that is shared out
// (kLevels = 1); a launch of few rows waits for the slowest, and there the crossing bin is binned again twice (kLevels = 3,
// 28 more registers): one mask of 1013 rows, smooth scores, 45 -> 24 us (34 us with the workgroup-wide sort of k_select), ties
// 45 -> 24..35; 40 masks of 591 rows took 49 us with one level, 59 with three.
template <int kSlots, int kLevels>
__global__ __launch_bounds__(kThreads) void k_select_mass(const uint64_t* __restrict__ class_bits,
                                                          const float* __restrict__ scores, int64_t rows_total, int Sb, int cap,
                                                          SelectArgs a, uint32_t* __restrict__ keepbits, int32_t* __restrict__ counts) {
    extern __shared__ unsigned char smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
    if (row >= rows_total) return;
    MassRow<kSlots> r;
    load_mass_row<kSlots>(class_bits, scores, row, (int)(row % Sb), Sb, r);
    const uint64_t threshold = select_mass_row<kSlots, kLevels>(r, a, smem + (size_t)wave * select_mass_lds_bytes(cap), cap);
    store_keep_words<kSlots>(row, Sb, keepbits, counts, [&](int i) { return kept_of_mass_row(r, i, threshold); });
}

// The whole mask in one launch where it has at most 32 rows of at most 32 key blocks (a row is one lane mask): a workgroup of
// sixteen waves takes a mask, a wave every sixteenth row; the counts of the rows meet in LDS and each wave writes its own out.
// Selection and emission apart are two launches: 11.3 us a call from the host, this 8.3 (1 to 256 masks of 9 to 32 rows); a
// whole call on 256 tokens 27.9 / 25.0.  With 48 rows, three to a wave, the mask alone still gains (11.2 / 8.5), but a call that
// the GPU bounds loses 1.4 us (6144 tokens x 8 heads 85.0 / 86.5), and 40 masks of 64 rows 10.4 / 11.2 by cumulative mass.
// grid: B * masks.  LDS: 16 x select_mass_lds_bytes(cap), or 16 x 64 keys.
constexpr int kShortMask = 32, kShortWaves = 16;
template <bool kMass>
__global__ __launch_bounds__(64 * kShortWaves) void k_mask_short(const uint64_t* __restrict__ class_bits, const float* __restrict__ scores, int Sb,
                                                                 int cap, SelectArgs a, int32_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                                 int64_t capacity, int64_t* __restrict__ nnz) {
    extern __shared__ unsigned char smem[];
    __shared__ int s_count[kShortMask];
    constexpr int kSlots = 2, kOwn = kShortMask / kShortWaves;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t mask_id = blockIdx.x;
    uint64_t kept[kOwn];
    if (threadIdx.x < kShortMask) s_count[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int qb = i * kShortWaves + wave;
        kept[i] = 0ull;
        if (qb >= Sb) continue;                                            // the same in every lane
        if constexpr (kMass) {
            MassRow<kSlots> r;
            load_mass_row<kSlots>(class_bits, scores, mask_id * Sb + qb, qb, Sb, r);
            const uint64_t threshold = select_mass_row<kSlots, 3>(r, a, smem + (size_t)wave * select_mass_lds_bytes(cap), cap);
            kept[i] = kept_of_mass_row(r, 0, threshold);
        } else {
            WaveRow<kSlots> r;
            load_wave_row<kSlots>(class_bits, scores, mask_id * Sb + qb, qb, Sb, a, r);
            uint64_t c_near, c_far;
            select_wave_row<kSlots>(r, bits_of(Sb), a, reinterpret_cast<uint64_t*>(smem) + wave * 64, &c_near, &c_far);
            kept[i] = r.m_forced[0] | __ballot(r.w.c[0] >= c_near);
            if (a.two_ratio) kept[i] |= __ballot(r.w.c[0] >= c_far) & r.m_far[0];
        }
        if (lane == 0) s_count[qb] = __popcll(kept[i]);
    }
    __syncthreads();
    const int own = lane < kShortMask ? s_count[lane] : 0, incl = wave_prefix(own);
    if (wave == 0) {
        int32_t* rp = rowptr + mask_id * (Sb + 1);
        if (lane < Sb) rp[lane] = incl - own;
        if (lane == Sb - 1) {
            rp[Sb] = incl;
            nnz[mask_id] = incl;
        }
    }
    int32_t* out = colidx + mask_id * capacity;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int qb = i * kShortWaves + wave;
        if (qb >= Sb) continue;
        const int64_t p = from_lane(incl - own, qb) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept[i], 0u));
        if (((kept[i] >> lane) & 1ull) && p < capacity) out[p] = lane;
    }
}

// grid: (Sb, masks, B).  A candidate set of the row is identified by the frame f that realises its gap: the key
// blocks whose first frame is f (f after the query block) or whose last frame is f (f before it); they lie in the
// key-block range of frame f, at most `maxlen` blocks.
// LDS: keep[words] u32 | tile[maxlen][Nf] f32.  All threads first scatter the row's selectable scores into the tile,
// position inside the set's range major, frame minor (reads of the row coalesced, the frame arithmetic once per key
// block); a lane then walks "its" frame's column: neighbouring lanes read neighbouring LDS words, and nothing in the
// serial part touches global memory.  Cells that hold no member keep a sentinel (a NaN pattern; scores are finite).
// The host refuses geometries whose tile does not fit the LDS (beyond about a million tokens at block size 32).
// The three passes over a set run in ascending key-block order, one addition at a time, with floating-point
// contraction off: the summation order and the absence of fused multiply-adds are part of the definition the
// results are compared against.  A cell outside the set adds +0.0, which leaves the running sums bit for bit as they
// are (they start at +0.0 and so are never -0.0), so the loops carry no branch.
// The threshold test is the quotient (s - mu) / (sigma + eps) >= tau in IEEE double.  A division costs about ten
// double-precision instructions, so the quotient is first estimated with a reciprocal (relative error <= 2^-52);
// only when the estimate lies within 2^-50 |tau| of tau is the division itself evaluated.
constexpr uint32_t kNoMember = 0x7fc0dead;

template <int kT>
__global__ __launch_bounds__(kT) void k_select_zscore(const uint8_t* __restrict__ class_map,
                                                            const float* __restrict__ scores, int masks, int Sb,
                                                            int maxlen, SelectArgs a, uint32_t* __restrict__ keepbits,
                                                            int32_t* __restrict__ counts) {
#pragma clang fp contract(off)
    extern __shared__ unsigned char smem[];
    const int words = (Sb + 31) / 32;
    uint32_t* keep = reinterpret_cast<uint32_t*>(smem);
    uint32_t* tile = reinterpret_cast<uint32_t*>(smem + (size_t)words * 4);     // [maxlen][Nf], score bits
    __shared__ int s_cnt;
    const int qb = blockIdx.x, m = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int64_t row = ((int64_t)b * masks + m) * Sb + qb;
    const float* srow = scores + row * Sb;
    const uint8_t* crow = class_map + (int64_t)qb * Sb;
    for (int i = tid; i < words; i += kT) keep[i] = 0u;
    if (tid == 0) s_cnt = 0;
    for (int i = tid; i < maxlen * a.Nf; i += kT) tile[i] = kNoMember;
    __syncthreads();
    const int r0 = qb * a.Bs, r1 = min(a.N, r0 + a.Bs);
    const int i0 = r0 / a.Nt, i1 = (r1 - 1) / a.Nt;
    for (int kb = tid; kb < Sb; kb += kT) {
        const int c = crow[kb];
        if (c == 3) atomicOr(&keep[kb >> 5], 1u << (kb & 31));
        if (c == 1 || c == 2) {
            const uint32_t c0 = (uint32_t)kb * (uint32_t)a.Bs;                   // < N <= 2^31 - 1: 32-bit divisions
            const int j0 = (int)(c0 / (uint32_t)a.Nt);
            const int j1 = (int)((min((uint32_t)a.N, c0 + (uint32_t)a.Bs) - 1u) / (uint32_t)a.Nt);
            const int f = j0 > i1 ? j0 : j1;                                     // selectable: j0 > i1 + 1 or j1 < i0 - 1
            const int pos = kb - (int)(((uint32_t)f * (uint32_t)a.Nt) / (uint32_t)a.Bs);
            tile[pos * a.Nf + f] = __float_as_uint(srow[kb]);
        }
    }
    __syncthreads();
    for (int f = tid; f < a.Nf; f += kT) {
        const bool after = f > i1 + 1, before = f < i0 - 1;                      // gaps 0 and 1 are the never-pruned zone
        if (!after && !before) continue;
        const int gap = after ? f - i1 : i0 - f;
        const int64_t f_lo = (int64_t)f * a.Nt, f_hi = f_lo + a.Nt;              // tokens of frame f
        const int kb_lo = (int)(f_lo / a.Bs);
        const int len = min(Sb - 1, (int)((f_hi - 1) / a.Bs)) - kb_lo + 1;
        // cell p of the set: score bits, or kNoMember
        auto cell = [&](int p) -> uint32_t { return tile[p * a.Nf + f]; };
        int n = 0;
        double sum = 0.0;
#pragma unroll 4
        for (int p = 0; p < len; ++p) {
            const uint32_t v = cell(p);
            const bool in = v != kNoMember;
            sum = sum + (in ? (double)__uint_as_float(v) : 0.0);
            n += in ? 1 : 0;
        }
        if (n == 0) continue;
        const double mu = sum / (double)n;
        double ssq = 0.0;
#pragma unroll 4
        for (int p = 0; p < len; ++p) {
            const uint32_t v = cell(p);
            const double dlt = (double)__uint_as_float(v) - mu;
            const double sq = dlt * dlt;
            ssq = ssq + (v != kNoMember ? sq : 0.0);
        }
        const double denom = sqrt(ssq / (double)n) + 1e-6;
        const double rcp = 1.0 / denom;
        // every member of the set has the same smallest frame distance (the gap), hence the same decay state
        const double tau = ((a.near_mask[gap >> 6] >> (gap & 63)) & 1ull) ? a.tau_near : a.tau_far;
        // estimates outside [tau_lo, tau_hi] decide by themselves; an infinite tau never needs the division
        const double slack = fabs(tau) != INFINITY ? 8.9e-16 * fabs(tau) + 1e-290 : 0.0;
        const double tau_lo = tau - slack, tau_hi = tau + slack;
        bool any = false;
        int best_p = -1;
        float best_s = 0.f;
#pragma unroll 4
        for (int p = 0; p < len; ++p) {
            const uint32_t v = cell(p);
            if (v == kNoMember) continue;
            const float x = __uint_as_float(v);
            const double dev = (double)x - mu;
            const double est = dev * rcp;
            bool pass = est >= tau;
            if (est >= tau_lo && est <= tau_hi && slack != 0.0) pass = dev / denom >= tau;
            if (pass) { any = true; atomicOr(&keep[(kb_lo + p) >> 5], 1u << ((kb_lo + p) & 31)); }
            if (best_p < 0 || x > best_s) { best_p = p; best_s = x; }
        }
        if (!any) atomicOr(&keep[(kb_lo + best_p) >> 5], 1u << ((kb_lo + best_p) & 31));
    }
    __syncthreads();
    store_row<kT>(keep, words, row, keepbits, counts, &s_cnt);
}

// grid: (Sb, masks, B)
// rowptr of every mask where the rows do not add up the earlier counts themselves (launch_emit): the exclusive prefix of its
// rows' kept counts, one workgroup per mask.  grid: (masks, B).
__global__ __launch_bounds__(kThreads) void k_row_offsets(const int32_t* __restrict__ counts, int masks, int Sb, int shared,
                                                          int32_t* __restrict__ rowptr, int64_t* __restrict__ nnz) {
    __shared__ long long s_wave[kWaves];
    const int m = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t mask_id = (int64_t)b * masks + m;
    const int64_t src = shared ? 0 : mask_id * Sb;
    int32_t* rp = rowptr + mask_id * (Sb + 1);
    long long running = 0;
    for (int base = 0; base < Sb; base += kThreads) {
        const int i = base + tid;
        const long long c = (i < Sb) ? counts[src + i] : 0;
        long long incl = c;
        for (int o = 1; o < 64; o <<= 1) {
            const long long t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        long long wave_base = 0, total = 0;
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) wave_base += s_wave[w];
            total += s_wave[w];
        }
        if (i < Sb) rp[i] = (int32_t)(running + wave_base + incl - c);
        running += total;
        __syncthreads();
    }
    if (tid == 0) {
        rp[Sb] = (int32_t)running;
        nnz[mask_id] = running;
    }
}

// One workgroup per row: the set bits of its keep bitmap, ascending, written from the row's offset on.
__global__ __launch_bounds__(kThreads) void k_emit(const uint32_t* __restrict__ keepbits, int masks, int Sb, int shared,
                                                   const int32_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                   int64_t capacity) {
    __shared__ int s_wave[kWaves];
    const int qb = blockIdx.x, m = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int64_t mask_id = (int64_t)b * masks + m;
    const int64_t src = shared ? 0 : mask_id * Sb;      // shared: one selection (Sb rows) serves every (b, m)
    const int64_t row = src + qb;
    const int words = (Sb + 31) / 32;
    const long long off0 = rowptr[mask_id * (Sb + 1) + qb];      // negative only if the mask outgrew 32-bit offsets
    int32_t* out = colidx + mask_id * capacity;
    long long base = off0;
    for (int w0 = 0; w0 < words; w0 += kThreads) {
        const int wi = w0 + tid;
        const uint32_t wv = (wi < words) ? keepbits[row * words + wi] : 0u;
        const int c = __popc(wv);
        // exclusive prefix of c over the workgroup
        int incl = c;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int wave_base = 0, total = 0;
        for (int i = 0; i < kWaves; ++i) {
            if (i < wave) wave_base += s_wave[i];
            total += s_wave[i];
        }
        long long pos = base + wave_base + incl - c;
        uint32_t bits = wv;
        while (bits) {
            const int bit = __ffs(bits) - 1;
            bits &= bits - 1;
            if (pos >= 0 && pos < capacity) out[pos] = wi * 32 + bit;
            ++pos;
        }
        base += total;
        __syncthreads();
    }
}

}  // namespace

// register slots of the selection kernel for a row of Sb key blocks (0: too long for it)
int wave_select_slots(int Sb) {
    const int need = (Sb + 63) / 64;
    for (int s : {2, 4, 8, 12, 16})
        if (need <= s) return s;
    return 0;
}
static_assert(kWaveSelectMaxSlots == 16, "the largest instantiation");

hipError_t launch_class_map(const Geometry& g, const FrameTab& tab, uint8_t* class_map, uint64_t* class_bits,
                            int32_t* row_sel, unsigned long long* totals, hipStream_t s) {
    hipLaunchKernelGGL(k_class_map, dim3(g.Sb), dim3(kThreads), 0, s, g, tab, class_map, row_sel, totals);
    if (class_bits)
        hipLaunchKernelGGL(k_class_bits, dim3((g.Sb + kWaves - 1) / kWaves), dim3(kThreads), 0, s, class_map, g.Sb,
                           wave_select_slots(g.Sb), class_bits);
    return hipGetLastError();
}

hipError_t launch_select(const uint8_t* class_map, const uint64_t* class_bits, const float* scores, int B, int masks,
                         int Sb, const SelectArgs& a, uint32_t* keepbits, int32_t* counts, hipStream_t s) {
    // One wave per row pays when there are more rows than workgroups the chip holds at once (per-head masks), and while
    // a row's keys fit 16 register pairs per lane: measured 15 - 35 % faster than a workgroup per row there, slower
    // beyond 1024 key blocks (registers, one wave per SIMD) and on the few hundred rows of a single fused mask.
    const int64_t rows_total = (int64_t)B * masks * Sb;
    if ((a.mode == 0 || a.mode == 3) && class_bits && Sb <= kWaveSelectMaxBlocks && rows_total >= kWaveSelectMinRows) {
        // few rows: one per workgroup, so that they spread over as many CUs as there are rows
        const int waves = rows_total >= kWaveSelectPackRows ? kWaves : 1;
        const dim3 grid((unsigned)((rows_total + waves - 1) / waves)), block(64 * waves);
        const int slots = wave_select_slots(Sb);
#define DR_SELECT_WAVE(S) \
    hipLaunchKernelGGL(k_select_wave<S>, grid, block, 0, s, class_bits, scores, rows_total, Sb, a, keepbits, counts)
        if (slots == 2) DR_SELECT_WAVE(2);
        else if (slots == 4) DR_SELECT_WAVE(4);
        else if (slots == 8) DR_SELECT_WAVE(8);
        else if (slots == 12) DR_SELECT_WAVE(12);
        else DR_SELECT_WAVE(16);
#undef DR_SELECT_WAVE
        return hipGetLastError();
    }
    // Cumulative mass, one wave per row as well (the prefix's end is found without sorting).
    if (a.mode == 1 && class_bits && Sb <= kWaveSelectMaxBlocks) {
        const int waves = rows_total >= kWaveSelectPackRows ? kWaves : 1;
        const dim3 grid((unsigned)((rows_total + waves - 1) / waves)), block(64 * waves);
        const int cap = (a.sort_cap + 1) & ~1, slots = wave_select_slots(Sb);      // (16-byte aligned bins)
        const size_t lds = select_mass_lds_bytes(cap) * waves;
        auto launch = [&](auto kern) -> hipError_t {
            if (lds > 64 * 1024) {
                hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(kern, grid, block, lds, s, class_bits, scores, rows_total, Sb, cap, a, keepbits, counts);
            return hipGetLastError();
        };
#define DR_SELECT_MASS(SLOTS) launch(waves > 1 ? k_select_mass<SLOTS, 1> : k_select_mass<SLOTS, 3>)
        if (slots == 2) return DR_SELECT_MASS(2);
        if (slots == 4) return DR_SELECT_MASS(4);
        if (slots == 8) return DR_SELECT_MASS(8);
        if (slots == 12) return DR_SELECT_MASS(12);
        return DR_SELECT_MASS(16);
#undef DR_SELECT_MASS
    }
    const size_t words = (Sb + 31) / 32;
    const size_t lds = (size_t)a.sort_cap * (a.mode == 1 ? 16 : 8) + words * 4;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_select),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_select, dim3(Sb, masks, B), dim3(kThreads), lds, s, class_map, scores, masks, Sb, a,
                       keepbits, counts);
    return hipGetLastError();
}

bool mask_short_supported(int mode, int B, int masks, int Sb) {
    return (mode == 0 || mode == 1) && Sb <= kShortMask && (int64_t)B * masks <= 256;
}
hipError_t launch_mask_short(const uint64_t* class_bits, const float* scores, int B, int masks, int Sb, const SelectArgs& a, int32_t* rowptr,
                             int32_t* colidx, int64_t capacity, int64_t* nnz, hipStream_t s) {
    const int cap = (a.sort_cap + 1) & ~1;      // (16-byte aligned bins)
    const size_t lds = a.mode == 1 ? select_mass_lds_bytes(cap) * kShortWaves : (size_t)kShortWaves * 64 * 8;
    hipLaunchKernelGGL(a.mode == 1 ? k_mask_short<true> : k_mask_short<false>, dim3((unsigned)(B * masks)), dim3(64 * kShortWaves), lds, s, class_bits,
                       scores, Sb, cap, a, rowptr, colidx, capacity, nnz);
    return hipGetLastError();
}

hipError_t launch_select_zscore(const uint8_t* class_map, const float* scores, int B, int masks, int Sb,
                                const SelectArgs& a, uint32_t* keepbits, int32_t* counts, hipStream_t s) {
    const size_t lds = select_zscore_lds_bytes(Sb, a.Nt, a.Nf, a.Bs);
    if (lds > kSelectZscoreMaxLds) return hipErrorInvalidValue;      // the host layer checks this before calling
    // In the serial part as many lanes work as there are frames, so where many rows wait one wave per row keeps four times as
    // many of them in flight, if their tiles let them: whole calls, four waves a row / one, 40 masks of 591 rows 131 / 88 us, 12 of
    // 370 28.6 / 22.3, 8 of 700 (4 frames) 164 / 105, 3 of 929 26.6 / 22.4, 2 of 2000 (tiles of 5.5 KB) 58.4 / 56.5.
    const int64_t rows_total = (int64_t)B * masks * Sb;
    const bool one_wave = rows_total >= kWaveSelectPackRows && lds <= 8 * 1024;
    auto kern = one_wave ? k_select_zscore<64> : k_select_zscore<kThreads>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int maxlen = (a.Nt + a.Bs - 1) / a.Bs + 1;          // key blocks that can touch one frame
    hipLaunchKernelGGL(kern, dim3(Sb, masks, B), dim3(one_wave ? 64 : kThreads), lds, s, class_map, scores, masks, Sb, maxlen,
                       a, keepbits, counts);
    return hipGetLastError();
}

// Column lists of rows of at most 2048 key blocks (64 bitmap words).  A lane loads one bitmap word; the wave then walks the row 64
// key blocks at a time: the two words of that stretch are read back as a wave-uniform lane mask, a lane whose bit is set stores
// its key block at the running offset plus the number of set bits below it (v_mbcnt), so that each store instruction writes
// one contiguous run.
__device__ __forceinline__ void emit_row(uint32_t wv, int Sb, long long pos, int32_t* __restrict__ out, int64_t capacity) {
    const int lane = lane_id(), stretches = (Sb + 63) / 64;
    char* at = reinterpret_cast<char*>(out + pos);                          // (the same in every lane; places of the row are 32-bit offsets)
    const int64_t left = capacity - pos;
    const uint32_t room = left <= 0 ? 0u : left < 0x7fffffff ? (uint32_t)left : 0x7fffffffu;
    uint32_t done = 0u;
    for (int i = 0; i < stretches; ++i) {                                  // wave-uniform
        const uint32_t lo = __builtin_amdgcn_readlane(wv, 2 * i), hi = __builtin_amdgcn_readlane(wv, 2 * i + 1);
        const uint64_t m = ((uint64_t)hi << 32) | lo;
        const uint32_t place = (uint32_t)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, done));
        if (__builtin_amdgcn_inverse_ballot_w64(m) && place < room) *reinterpret_cast<int32_t*>(at + place * 4u) = i * 64 + lane;
        done += (uint32_t)__popcll(m);
    }
}

// One wave per row and workgroup: calls of few rows, which spread over as many CUs as there are rows.  The wave adds up the
// counts of the mask's earlier rows itself (at most 32 coalesced reads per lane out of L2).  grid: B * masks * Sb.
__global__ __launch_bounds__(64) void k_emit_wave(const uint32_t* __restrict__ keepbits, const int32_t* __restrict__ counts, int Sb,
                                                  int shared, int32_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                  int64_t capacity, int64_t* __restrict__ nnz) {
    const int lane = lane_id();
    const int64_t r = blockIdx.x, mask_id = r / Sb;                        // (mask_id, qb) flattened
    const int qb = (int)(r - mask_id * Sb);
    const int64_t src = shared ? 0 : mask_id * Sb;                         // shared: one selection serves every (b, m)
    const int words = (Sb + 31) / 32;
    const uint32_t wv = (lane < words) ? keepbits[(src + qb) * words + lane] : 0u;
    int before = 0;                                                        // (at most 2048 rows of 2048 blocks: 32 bits hold it)
    int32_t* rp = rowptr + mask_id * (Sb + 1);
#pragma unroll 4
    for (int i = lane; i < qb; i += 64) before += counts[src + i];
    before = from_lane(wave_prefix(before), 63);
    if (lane == 0) {
        rp[qb] = before;
        if (qb == Sb - 1) {
            const int all = before + counts[src + qb];
            rp[Sb] = all;
            nnz[mask_id] = all;
        }
    }
    emit_row(wv, Sb, before, colidx + mask_id * capacity, capacity);
}

// kRows rows of one mask per workgroup, whose bitmaps are on their way while the workgroup adds up the counts of the mask's earlier
// rows, once for all of them.  (Each wave for itself: 13 us of launch at 40 masks of 591 rows where four rows take 11.7 and eight 10.6;
// 8 masks of 2000 rows, whole call, 148 -> 144.)  Eight where many rows wait, four where more workgroups count for more: whole
// calls, four / eight / sixteen, 3716 rows 13.0 / 13.6 / 15.5 us, 4440 11.5 / 11.8 / 12.6, 7608 17.6 / 17.2 / 17.7, 23 640 34.3 / 33.2 / 32.8
// and 36.6 / 35.1 / 35.2, uniform rule at 35 460 16.4 / 14.7 / 14.2.
// grid: B * masks * ceil(Sb / kRows).
constexpr int64_t kEmitEightRows = 6000;
template <int kEmitRows>
__global__ __launch_bounds__(kThreads) void k_emit_rows(const uint32_t* __restrict__ keepbits, const int32_t* __restrict__ counts, int Sb,
                                                        int shared, int32_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                        int64_t capacity, int64_t* __restrict__ nnz) {
    __shared__ int s_part[kWaves];
    constexpr int kOwn = kEmitRows / kWaves;
    const int tiles = (Sb + kEmitRows - 1) / kEmitRows;
    const int64_t mask_id = blockIdx.x / tiles;
    const int q0 = (int)(blockIdx.x - mask_id * tiles) * kEmitRows;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t src = shared ? 0 : mask_id * Sb;
    const int words = (Sb + 31) / 32;
    uint32_t wv[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int qb = q0 + wave * kOwn + i;
        wv[i] = (lane < words && qb < Sb) ? keepbits[(src + qb) * words + lane] : 0u;
    }
    const int own = (lane < kEmitRows && q0 + lane < Sb) ? counts[src + q0 + lane] : 0;
    int before = 0;                                                        // (at most 2048 rows of 2048 blocks: 32 bits hold it)
    for (int i0 = 0; i0 < q0; i0 += 4 * kThreads) {                        // (once, or twice: q0 < 2048)
        int c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = counts[src + min(i0 + e * kThreads + tid, q0 - 1)];
#pragma unroll
        for (int e = 0; e < 4; ++e) before += i0 + e * kThreads + tid < q0 ? c[e] : 0;
    }
    before = wave_prefix(before);
    if (lane == 63) s_part[wave] = before;
    __syncthreads();
    before = s_part[0] + s_part[1] + s_part[2] + s_part[3];
    const int incl = before + wave_prefix(own);                            // lane r: with the counts of rows q0 .. q0 + r
    int32_t* rp = rowptr + mask_id * (Sb + 1);
    if (wave == 0 && lane < kEmitRows && q0 + lane < Sb) {
        rp[q0 + lane] = incl - own;
        if (q0 + lane == Sb - 1) {
            rp[Sb] = incl;
            nnz[mask_id] = incl;
        }
    }
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int r = wave * kOwn + i;
        if (q0 + r < Sb) emit_row(wv[i], Sb, from_lane(incl - own, r), colidx + mask_id * capacity, capacity);
    }
}
static_assert(8 * kThreads >= 64 * 32, "the earlier rows of a mask");

// The same with the offsets made by k_row_offsets before: a wave writes its row without waiting for any other.  (The row is worked out
// in vector registers: the same in scalar ones puts argument loads behind the row's and takes 18.5 us a call where this takes 15.5,
// 2000 masks of 40 rows.)  grid: ceil(B * masks * Sb / 4).
__global__ __launch_bounds__(kThreads) void k_emit_rows_at(const uint32_t* __restrict__ keepbits, uint32_t rows_total, int Sb, int shared,
                                                           const int32_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                           int64_t capacity) {
    const int lane = lane_id();
    const uint32_t r = blockIdx.x * kWaves + (threadIdx.x >> 6);           // (mask_id, qb) flattened
    if (r >= rows_total) return;
    const uint32_t mask_id = r / (uint32_t)Sb;
    const int qb = (int)(r - mask_id * (uint32_t)Sb);
    const int64_t src = shared ? 0 : (int64_t)mask_id * Sb;
    const int words = (Sb + 31) / 32;
    const uint32_t wv = (lane < words) ? keepbits[(src + qb) * words + lane] : 0u;
    const int before = rowptr[(int64_t)mask_id * (Sb + 1) + qb];
    emit_row(wv, Sb, from_lane(before, 0), colidx + (int64_t)__builtin_amdgcn_readfirstlane(mask_id) * capacity, capacity);
}

hipError_t launch_emit(const uint32_t* keepbits, const int32_t* counts, int B, int masks, int Sb, bool shared,
                       int32_t* rowptr, int32_t* colidx, int64_t capacity, int64_t* nnz, hipStream_t s) {
    const int64_t rows_total = (int64_t)B * masks * Sb;
    // A launch of its own for the offsets costs 2 to 5 us, the more the longer the rows (a workgroup walks the counts of a mask); made
    // in the emission's launch they cost each workgroup a round of reads and a barrier, of which long rows hide more.  Whole calls of
    // the uniform rule, offsets in the emission's launch / apart, rows of 40 key blocks: 20 000 rows 6.5 / 8.4 us, 30 000 8.7 / 8.5,
    // 80 000 19.7 / 15.7; of 300: 30 000 12.4 / 12.5, 80 000 26.8 / 23.6, 240 000 71 / 57; of 591: 40 000 20.1 / 20.9, 60 000 28.3 / 27.7,
    // 160 000 67 / 60; of 1024: 60 000 36.3 / 37.2, 100 000 57.4 / 55.8; of 2040: 50 000 50 / 54, 118 000 113 / 115.
    const int64_t line = 20000 + 55 * (int64_t)Sb;
    const bool apart = Sb > 64 * 32 || rows_total >= (line > 30000 ? line : 30000);
    if (apart) hipLaunchKernelGGL(k_row_offsets, dim3(masks, B), dim3(kThreads), 0, s, counts, masks, Sb, shared ? 1 : 0, rowptr, nnz);
    if (Sb > 64 * 32) {
        hipLaunchKernelGGL(k_emit, dim3(Sb, masks, B), dim3(kThreads), 0, s, keepbits, masks, Sb, shared ? 1 : 0, rowptr,
                           colidx, capacity);
    } else if (apart) {
        hipLaunchKernelGGL(k_emit_rows_at, dim3((unsigned)((rows_total + kWaves - 1) / kWaves)), dim3(kThreads), 0, s, keepbits, (uint32_t)rows_total,
                           Sb, shared ? 1 : 0, rowptr, colidx, capacity);
    } else if (rows_total >= kWaveSelectPackRows) {
        const int per = rows_total >= kEmitEightRows ? 8 : 4;
        hipLaunchKernelGGL(per == 8 ? k_emit_rows<8> : k_emit_rows<4>, dim3((unsigned)((int64_t)B * masks * ((Sb + per - 1) / per))), dim3(kThreads), 0, s,
                           keepbits, counts, Sb, shared ? 1 : 0, rowptr, colidx, capacity, nnz);
    } else {
        hipLaunchKernelGGL(k_emit_wave, dim3((unsigned)rows_total), dim3(64), 0, s, keepbits, counts, Sb, shared ? 1 : 0, rowptr, colidx, capacity, nnz);
    }
    return hipGetLastError();
}

}  // namespace dr
