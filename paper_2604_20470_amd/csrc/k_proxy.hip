// Objective of the paper's offline parameter search on its proxy task (App. C, Eq. 22) as a device reduction:
//   nmse = mean over (b, h) of ||A_dense - A_sparse||_F^2 / ||A_dense||_F^2,
//   loss = nmse + alpha * max(0, target - sparsity),  sparsity = 1 - mean(nnz) / Sb^2.
// Two launches: per (b, h) and slice, fp64 partial sums in a fixed order; then one workgroup folds the slices in
// order and forms the three outputs.  No atomics: the result is the same bits on every run.
// The objective alone needs neither matrix: k_proxy_rows forms the same sums from Q, K and the mask.
#include "dr_internal.h"

namespace dr {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ void block_sum2(double& a, double& b, double* sh) {
    const int tid = threadIdx.x;
    sh[tid] = a;
    sh[kThreads + tid] = b;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (tid < s) {
            sh[tid] += sh[tid + s];
            sh[kThreads + tid] += sh[kThreads + tid + s];
        }
        __syncthreads();
    }
    a = sh[0];
    b = sh[kThreads];
}

// (a norm that is not a number, from features that are not, stays one: it must not look like a perfect reconstruction)
__device__ __forceinline__ double ratio_of(double num, double den) { return den == 0.0 ? 0.0 : num / den; }

__device__ __forceinline__ void store_objective(double ratio_sum, double nnz_sum, int BH, int n_masks, int Sb, double target, double alpha,
                                                double* __restrict__ out) {
    const double nmse = ratio_sum / (double)BH;
    const double sparsity = 1.0 - nnz_sum / (double)n_masks / ((double)Sb * (double)Sb);
    const double short_of = target - sparsity;
    out[0] = nmse + alpha * (short_of > 0.0 ? short_of : 0.0);
    out[1] = nmse;
    out[2] = sparsity;
}

// grid (kProxySlices, B * H): slice s of head bh covers elements [s * per, (s + 1) * per) of its N x N matrices.
__global__ __launch_bounds__(kThreads) void k_proxy_partial(const float* __restrict__ ad, const float* __restrict__ as,
                                                            long long nn, double* __restrict__ partial) {
    __shared__ double sh[2 * kThreads];
    const int bh = blockIdx.y, slice = blockIdx.x;
    const long long per = (nn + kProxySlices - 1) / kProxySlices;
    const long long lo = (long long)slice * per, hi = min(nn, lo + per);
    const float* pd = ad + (long long)bh * nn;
    const float* ps = as + (long long)bh * nn;
    double num = 0.0, den = 0.0;
    for (long long i = lo + threadIdx.x; i < hi; i += kThreads) {
        const double d = (double)pd[i], e = d - (double)ps[i];
        num += e * e;
        den += d * d;
    }
    block_sum2(num, den, sh);
    if (threadIdx.x == 0) {
        partial[((long long)bh * kProxySlices + slice) * 2 + 0] = num;
        partial[((long long)bh * kProxySlices + slice) * 2 + 1] = den;
    }
}

__global__ __launch_bounds__(kThreads) void k_proxy_final(const double* __restrict__ partial, int BH,
                                                          const int64_t* __restrict__ nnz, int n_masks, int Sb,
                                                          double target, double alpha, double* __restrict__ out) {
    __shared__ double sh[2 * kThreads];
    double ratio_sum = 0.0, nnz_sum = 0.0;
    for (int bh = threadIdx.x; bh < BH; bh += kThreads) {
        double num = 0.0, den = 0.0;
        for (int s = 0; s < kProxySlices; ++s) {
            num += partial[((long long)bh * kProxySlices + s) * 2 + 0];
            den += partial[((long long)bh * kProxySlices + s) * 2 + 1];
        }
        ratio_sum += ratio_of(num, den);
    }
    for (int m = threadIdx.x; m < n_masks; m += kThreads) nnz_sum += (double)nnz[m];
    block_sum2(ratio_sum, nnz_sum, sh);
    if (threadIdx.x == 0) store_objective(ratio_sum, nnz_sum, BH, n_masks, Sb, target, alpha, out);
}

// The same sums without the matrices.  In a row of A_dense and A_sparse (both softmaxes of the same logits s, one over all
// keys, one over the kept ones) let l and E be the sums of e^s and of e^2s over the kept (k) and the pruned (u) keys:
//   ||a_dense||^2 = (E_k + E_u) / (l_k + l_u)^2,   ||a_dense - a_sparse||^2 = (E_u + l_u^2 E_k / l_k^2) / (l_k + l_u)^2,
// all terms positive, so nothing cancels where the two rows are nearly alike.  Logits and exponentials are fp32; every sum is fp64,
// taken online against its own moving reference, a whole power of two, so that moving it rounds nothing.
// One pass over the logits, which the fp32 matrix instruction forms (fp32 products and sums): what bounds it is that
// instruction, 1.1 GFLOP at 2048 tokens x 2 heads of 64 channels.  A workgroup owns 16 queries, so that 2048 tokens x 2 heads
// are 256 of them; its eight wavefronts take every eighth group of 32 keys, straight from memory to registers (a lane
// holds four consecutive channels c of its row and feeds one to each of four instructions: the order of the contraction
// is permuted alike for both operands), the next group on its way meanwhile.  22 us at that size, a third of it the matrix
// instructions; the two matrices read off the attention kernel with one-hot values and their difference took 2.2 ms.
// The quotient of the norms against 64 bits, over 24 cases of drifting features (256 to 1120 tokens, half of the blocks kept): off by
// 3.0e-8 of its value rms, 6.5e-8 at most (8.2e-8 and 2.7e-7 from the matrices, whose fp32 entries cancel where the two are alike).
// grid: (ceil(N / 16), H, B).  LDS: bitmap of the query block's kept key blocks.  partial: [B * H][gridDim.x][2].
constexpr int kRowWaves = 8, kRowTile = 16;
typedef float v4f __attribute__((ext_vector_type(4)));

struct RowSums {
    float m;            // reference (log2 units, a whole number, or -inf before the first key)
    double l, e;        // sum of 2^(x - m), sum of its squares
    // the sums against a reference not below this one (both -inf: they are 0; infinite logits have made them NaN already)
    __device__ __forceinline__ void move(float ref) {
        const int by = (int)fmaxf(m - ref, -4096.f);
        l = __builtin_ldexp(l, by);
        e = __builtin_ldexp(e, 2 * by);
        m = ref;
    }
    __device__ __forceinline__ void merge(RowSums o) {
        const float top = fmaxf(m, o.m);
        move(top);
        o.move(top);
        l += o.l;
        e += o.e;
    }
};

template <int D>
__global__ __launch_bounds__(64 * kRowWaves) void k_proxy_rows(const float* __restrict__ Q, const float* __restrict__ K, TensorDesc td,
                                                               const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                               int64_t colidx_stride, int mask_heads, int Bs, int Sb,
                                                               double* __restrict__ partial) {
    constexpr int kVec = D / 16;                // 16-byte pieces of a row per lane
    constexpr float kScaleLog2 = (float)(1.4426950408889634 / (D == 128 ? 11.313708498984760 : 8.0));
    extern __shared__ uint32_t s_kept[];
    __shared__ RowSums s_part[kRowWaves][2][kRowTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, quarter = lane >> 4;
    const int q0 = blockIdx.x * kRowTile, h = blockIdx.y, b = blockIdx.z, qb = q0 / Bs, N = td.N;
    const int64_t head = (int64_t)b * td.stride_b + (int64_t)h * td.stride_h;
    v4f qf[kVec];
#pragma unroll
    for (int j = 0; j < kVec; ++j)
        qf[j] = *reinterpret_cast<const v4f*>(Q + head + (int64_t)min(q0 + r16, N - 1) * td.stride_n + 16 * j + 4 * quarter);
    const int groups = (N + 31) / 32;
    v4f kf[2][kVec];
    auto load = [&](int group) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < kVec; ++j)
                kf[t][j] = *reinterpret_cast<const v4f*>(K + head + (int64_t)min(group * 32 + t * 16 + r16, N - 1) * td.stride_n + 16 * j + 4 * quarter);
    };
    if (wave < groups) load(wave);
    const int words = (Sb + 31) / 32;
    for (int i = tid; i < words; i += 64 * kRowWaves) s_kept[i] = 0u;
    __syncthreads();
    {
        // as the attention kernels read a mask: row range clipped to the colidx array, indices clamped
        const int64_t mask = (int64_t)b * mask_heads + (mask_heads == 1 ? 0 : h);
        const int32_t* rp = rowptr + mask * (Sb + 1);
        const int64_t beg = min(max((int64_t)rp[qb], (int64_t)0), colidx_stride), end = min(max((int64_t)rp[qb + 1], beg), colidx_stride);
        for (int64_t i = beg + tid; i < end; i += 64 * kRowWaves) {
            const int kb = min(max(colidx[mask * colidx_stride + i], 0), Sb - 1);
            atomicOr(&s_kept[kb >> 5], 1u << (kb & 31));
        }
    }
    __syncthreads();
    RowSums kept = {-INFINITY, 0.0, 0.0}, pruned = kept;      // of query r16, over this lane's keys
    for (int group = wave; group < groups; group += kRowWaves) {
        v4f k[2][kVec];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < kVec; ++j) k[t][j] = kf[t][j];
        load(min(group + kRowWaves, groups - 1));
        __builtin_amdgcn_sched_barrier(0);      // (the loads stay ahead of the products)
        v4f part[2][4];                         // four sums a logit: a quarter of the roundings in a row, and independent instructions
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) part[t][c] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < kVec; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int t = 0; t < 2; ++t) part[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[t][j][c], qf[j][c], part[t][c], 0, 0, 0);
        v4f s[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) s[t] = (part[t][0] + part[t][1]) + (part[t][2] + part[t][3]);
        // element i of s[t]: key group * 32 + t * 16 + 4 * quarter + i, query r16
        if (group * 32 + 32 > N) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (group * 32 + t * 16 + 4 * quarter + i >= N) s[t][i] = -INFINITY;
        }
        auto add = [&](RowSums& st) {
            float mx = s[0][0];
#pragma unroll
            for (int i = 1; i < 8; ++i) mx = fmaxf(mx, s[i >> 2][i & 3]);
            const float top = fmaxf(st.m, ceilf(mx * kScaleLog2)), ref = top == -INFINITY ? 0.f : top;
            st.move(top);
            // The product rounds once, with the subtraction.  Where logits are so large that a reference can be off the product it is the
            // rounding of by more than an exponent holds, it rounds before: the difference to the highest is then 0.
            const bool far = fabsf(ref) >= 0x1p28f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma clang fp contract(off)
                const float x = s[i >> 2][i & 3], by = far ? x * kScaleLog2 - ref : __builtin_fmaf(x, kScaleLog2, -ref);
                const double p = (double)__builtin_amdgcn_exp2f(by);
                st.l += p;
                st.e = __builtin_fma(p, p, st.e);
            }
        };
        const int kb = group * 32 / Bs;         // (a key block holds whole groups)
        if (__builtin_amdgcn_readfirstlane(s_kept[kb >> 5] >> (kb & 31)) & 1u) add(kept);
        else add(pruned);
    }
    for (int off = 16; off < 64; off <<= 1) {
        kept.merge({__shfl_xor(kept.m, off), __shfl_xor(kept.l, off), __shfl_xor(kept.e, off)});
        pruned.merge({__shfl_xor(pruned.m, off), __shfl_xor(pruned.l, off), __shfl_xor(pruned.e, off)});
    }
    if (quarter == 0) {
        s_part[wave][0][r16] = kept;
        s_part[wave][1][r16] = pruned;
    }
    __syncthreads();
    if (tid >= 2 * kRowTile) return;
    RowSums own = s_part[0][quarter][r16];      // quarter 0: kept keys, 1: pruned ones
    for (int w = 1; w < kRowWaves; ++w) own.merge(s_part[w][quarter][r16]);
    RowSums u = {__shfl_xor(own.m, 16), __shfl_xor(own.l, 16), __shfl_xor(own.e, 16)};
    double num = 0.0, den = 0.0;
    if (quarter == 0 && q0 + r16 < N) {
        const double of_kept = own.l == 0.0 ? 0.0 : own.e / (own.l * own.l);      // (a row that keeps nothing is 0)
        const float top = fmaxf(own.m, u.m);
        own.move(top);
        u.move(top);
        const double all = own.l + u.l;
        num = (u.e + u.l * u.l * of_kept) / (all * all);
        den = (own.e + u.e) / (all * all);
    }
    for (int off = 1; off < 16; off <<= 1) {
        num += __shfl_xor(num, off);
        den += __shfl_xor(den, off);
    }
    if (tid == 0) {
        double* out = partial + (((int64_t)b * td.H + h) * gridDim.x + blockIdx.x) * 2;
        out[0] = num;
        out[1] = den;
    }
}

// The partial sums of every (b, h), `parts` of them, folded in a fixed order, a wavefront each in turn; then the three outputs.
__global__ __launch_bounds__(kThreads) void k_proxy_fold(const double* __restrict__ partial, int BH, int parts,
                                                         const int64_t* __restrict__ nnz, int n_masks, int Sb,
                                                         double target, double alpha, double* __restrict__ out) {
    __shared__ double sh[2 * kThreads];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double ratio_sum = 0.0, nnz_sum = 0.0;
    for (int bh = wave; bh < BH; bh += kThreads / 64) {
        double num = 0.0, den = 0.0;
#pragma unroll 4
        for (int s = lane; s < parts; s += 64) {
            num += partial[((int64_t)bh * parts + s) * 2 + 0];
            den += partial[((int64_t)bh * parts + s) * 2 + 1];
        }
        for (int off = 32; off > 0; off >>= 1) {
            num += __shfl_xor(num, off);
            den += __shfl_xor(den, off);
        }
        if (lane == 0) ratio_sum += ratio_of(num, den);
    }
    for (int m = threadIdx.x; m < n_masks; m += kThreads) nnz_sum += (double)nnz[m];
    block_sum2(ratio_sum, nnz_sum, sh);
    if (threadIdx.x == 0) store_objective(ratio_sum, nnz_sum, BH, n_masks, Sb, target, alpha, out);
}

}  // namespace

hipError_t launch_proxy_objective(const float* Q, const float* K, const TensorDesc& td, const int32_t* rowptr, const int32_t* colidx,
                                  int64_t colidx_stride, int mask_heads, int Bs, int Sb, const int64_t* nnz, double target,
                                  double alpha, double* partial, double* out, hipStream_t s) {
    const int tiles = proxy_row_tiles(td.N);
    const size_t lds = (size_t)((Sb + 31) / 32) * 4;
    hipLaunchKernelGGL(td.d == 64 ? k_proxy_rows<64> : k_proxy_rows<128>, dim3(tiles, td.H, td.B), dim3(64 * kRowWaves), lds, s, Q, K, td,
                       rowptr, colidx, colidx_stride, mask_heads, Bs, Sb, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_proxy_fold, dim3(1), dim3(kThreads), 0, s, partial, td.B * td.H, tiles, nnz, td.B * mask_heads, Sb, target, alpha, out);
    return hipGetLastError();
}

hipError_t launch_proxy_loss(const float* A_dense, const float* A_sparse, int BH, int N, const int64_t* nnz, int n_masks,
                             int Sb, double target, double alpha, double* partial, double* out, hipStream_t s) {
    const long long nn = (long long)N * N;
    hipLaunchKernelGGL(k_proxy_partial, dim3(kProxySlices, BH), dim3(kThreads), 0, s, A_dense, A_sparse, nn, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_proxy_final, dim3(1), dim3(kThreads), 0, s, partial, BH, nnz, n_masks, Sb, target, alpha, out);
    return hipGetLastError();
}

}  // namespace dr
