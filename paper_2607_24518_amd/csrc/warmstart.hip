// Learned warm start (an addition to the paper's method): a Gaussian sketch
// Y = S Omega of width 64, canonical per-row coordinates (whitening of Y^T Y
// and successive-projection anchors), an MLP 64 -> 256 -> 256 -> k with
// GELU and a softplus output, and its training with the permutation-invariant
// Gram loss ||A A^T - B B^T||_F^2 and AdamW.  This file holds the kernels; the
// orchestration is in runtime.hip.
#include "common.h"

namespace symnmf {

// Omega_ij = sqrt(-2 ln(1-u)) cos(2 pi v) (Box & Muller 1958), u and v the
// 53-bit uniforms of SplitMix64 outputs 2e and 2e+1 of key seed, e = i*w + j.
__global__ void omega_kernel(uint64_t seed, int64_t n, int64_t rows_alloc, int w, float* __restrict__ out) {
    const int64_t total = rows_alloc * w;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        if (e >= n * w) { out[e] = 0.0f; continue; }
        const double u = (double)(splitmix64(seed, 2 * (uint64_t)e) >> 11) * (1.0 / 9007199254740992.0);
        const double v = (double)(splitmix64(seed, 2 * (uint64_t)e + 1) >> 11) * (1.0 / 9007199254740992.0);
        out[e] = (float)(sqrt(-2.0 * log(1.0 - u)) * cos(6.283185307179586 * v));
    }
}

hipError_t launch_omega(uint64_t seed, int64_t n, int64_t rows_alloc, int w, float* out, hipStream_t stream) {
    int64_t blocks = (rows_alloc * w + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(omega_kernel, dim3(blocks), dim3(256), 0, stream, seed, n, rows_alloc, w, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small dense GEMM, FP32 accumulation: C (M x N) = op(A) op(B) + bias, then an
// epilogue.  A: TA = 0 -> M x K row-major, TA = 1 -> K x M.  B: TB = 0 -> N x K
// row-major (used transposed), TB = 1 -> K x N.  B may hold bf16 values (the
// network weights at inference).  64 x 64 output tile, 16 reduction indices at
// a time; each of the four waves computes a 32 x 32 quarter as 2 x 2 blocks of
// v_mfma_f32_16x16x4_f32 (FP32 products and accumulation: the bf16 weights are
// widened exactly).  blockIdx.z splits K into ranges of kchunk: with more than
// one range every range writes its own partial C + z M N (no bias, no
// epilogue), summed in order by the kernel that applies the gradient.
// EPI: 0 none, 1 GELU x Phi(x) (Phi from erfc), 2 softplus, 3 residual output
// max(aux + x, 0), 4 GELU backward x (Phi(z) + z phi(z)) with z = aux, and the
// FP64 column sums of the result over the 64 rows in part.  Z (optional)
// receives the value before the epilogue.
// The matrices are small and read once: bound by latency, so the next 16
// indices are in flight in registers, 16 bytes a load, while the current ones
// are multiplied from one of two LDS buffers; with 21 KB of LDS up to seven
// work-groups share a CU (two buffers of 32 indices allow four and were 7 % of
// a training step slower).
// An operand whose rows hold the reduction index is kept row by row, 20 floats
// apart, a lane reading four consecutive indices 4 g .. 4 g + 3 at once, MFMA e
// reducing over the indices 4 g + e; one stored by reduction index is kept that
// way, 68 floats apart (4 rows are 16 banks): both without bank conflicts.
// m = 20000 rows, us before (4-byte loads, no overlap, the activation's
// backward in a launch of its own, weight gradients on 256 work-groups) and
// now: forward through a 256 x 256 layer 62 -> 43, backward through it 72 -> 46,
// the three weight gradients 290 -> 70.
// ---------------------------------------------------------------------------
constexpr int GK = 16;                            // reduction indices of a slab
constexpr int GLR = GK + 4, GLK = 64 + 4;         // LDS row strides: rows of reduction indices, of columns
constexpr int GSIDE = 64 * GLR > GK * GLK ? 64 * GLR : GK * GLK;
constexpr int GEMM_WGS = 512;                     // split weight gradients up to this many work-groups

// 16 (8) bytes of the alignment of their entries
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t ushort4u __attribute__((ext_vector_type(4), aligned(2)));

__device__ inline float normal_cdf_f(float x) { return 0.5f * erfcf(-x * 0.70710678118654752f); }

// four consecutive entries of p, those at lim or beyond as zeros
template <typename T>
__device__ inline floatx4 gemm_load4(const T* p, int64_t lim) {
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    if (lim >= 4) {
        if constexpr (sizeof(T) == 2) {
            const ushort4u u = *(const ushort4u*)p;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = bf16_bits_to_f32(u[e]);
        } else {
            v = *(const float4u*)p;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < lim) {
                if constexpr (sizeof(T) == 2) v[e] = bf16_bits_to_f32(p[e]);
                else v[e] = p[e];
            }
    }
    return v;
}

template <int TA, int TB, typename BT, int EPI>
__global__ __launch_bounds__(256) void gemm_kernel(const float* __restrict__ A, const BT* __restrict__ B,
                                                   const float* __restrict__ bias, float* __restrict__ C,
                                                   float* __restrict__ Z, const float* __restrict__ aux, int64_t ldaux,
                                                   double* __restrict__ part, int64_t M, int64_t N, int64_t K,
                                                   int64_t kchunk) {
    __shared__ __align__(16) float As[2][GSIDE];
    __shared__ __align__(16) float Bs[2][GSIDE];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int rb = 32 * (wv >> 1), cb = 32 * (wv & 1);   // this wave's quarter of the tile
    const int li = lane & 15, lk = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
    const int64_t kb = (int64_t)blockIdx.z * kchunk;
    const int64_t ke = kb + kchunk < K ? kb + kchunk : K;
    floatx4 acc[2][2];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = floatx4{0.f, 0.f, 0.f, 0.f};
    // a thread's vectors of a slab: rows t / RV + q RS, indices 4 (t % RV) ..,
    // or reduction indices t / 16 + 16 q, columns 4 (t % 16) ..
    constexpr int NQ = GK / 16, RV = GK / 4, RS = 256 / RV;
    floatx4 ra[NQ], rbv[NQ];
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int64_t kr = k0 + (t >> 4) + 16 * q, kc = k0 + 4 * (t % RV);
            const int64_t ar = m0 + t / RV + RS * q, ac = m0 + 4 * (t & 15);
            const int64_t br = n0 + t / RV + RS * q, bc = n0 + 4 * (t & 15);
            if (TA) ra[q] = gemm_load4(A + kr * M + ac, kr < ke ? M - ac : 0);
            else ra[q] = gemm_load4(A + ar * K + kc, ar < M ? ke - kc : 0);
            if (TB) rbv[q] = gemm_load4(B + kr * N + bc, kr < ke ? N - bc : 0);
            else rbv[q] = gemm_load4(B + br * K + kc, br < N ? ke - kc : 0);
        }
    };
    load(kb);
    int buf = 0;
    for (int64_t k0 = kb; k0 < ke; k0 += GK, buf ^= 1) {
        const int row = t / RV, idx = 4 * (t % RV), kr = t >> 4, col = 4 * (t & 15);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            *(floatx4*)&As[buf][TA ? (kr + 16 * q) * GLK + col : (row + RS * q) * GLR + idx] = ra[q];
            *(floatx4*)&Bs[buf][TB ? (kr + 16 * q) * GLK + col : (row + RS * q) * GLR + idx] = rbv[q];
        }
        __syncthreads();
        if (k0 + GK < ke) load(k0 + GK);
#pragma unroll
        for (int s = 0; s < GK / 16; ++s) {
            const int kk = 16 * s + 4 * lk;
            floatx4 av[2], bv[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = rb + 16 * h + li, c = cb + 16 * h + li;
                if (TA) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) av[h][e] = As[buf][(kk + e) * GLK + r];
                } else {
                    av[h] = *(const floatx4*)&As[buf][r * GLR + kk];
                }
                if (TB) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) bv[h][e] = Bs[buf][(kk + e) * GLK + c];
                } else {
                    bv[h] = *(const floatx4*)&Bs[buf][c * GLR + kk];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int bj = 0; bj < 2; ++bj)
                        acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[bi][e], bv[bj][e], acc[bi][bj], 0, 0, 0);
        }
    }
    const bool split = gridDim.z > 1;
    float* Cz = C + (split ? (int64_t)blockIdx.z * M * N : 0);
    double sum[2] = {0.0, 0.0};
    // output: lane (j, q) holds rows 4 q + v, v < 4, of column j of each block
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t m = m0 + rb + 16 * bi + 4 * lk + v, nn = n0 + cb + 16 * bj + li;
            if (m >= M || nn >= N) continue;
            float v_ = acc[bi][bj][v];
            if (split) { Cz[m * N + nn] = v_; continue; }
            if (bias) v_ += bias[nn];
            if (Z) Z[m * N + nn] = v_;
            if (EPI == 1) v_ = v_ * normal_cdf_f(v_);
            else if (EPI == 2) v_ = fmaxf(v_, 0.0f) + log1pf(expf(-fabsf(v_)));
            else if (EPI == 3) {
                v_ = aux[m * ldaux + nn] + v_;
                v_ = v_ > 0.0f ? v_ : 0.0f;
            } else if (EPI == 4) {
                const float z = aux[m * ldaux + nn];
                v_ = v_ * (normal_cdf_f(z) + z * expf(-0.5f * z * z) * 0.3989422804014327f);
                sum[bj] += (double)v_;
            }
            Cz[m * N + nn] = v_;
        }
    if constexpr (EPI == 4) {
        __shared__ double half[2][64];
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
            sum[bj] += __shfl_xor(sum[bj], 16, 64);
            sum[bj] += __shfl_xor(sum[bj], 32, 64);
            if (lk == 0) half[wv >> 1][cb + 16 * bj + li] = sum[bj];
        }
        __syncthreads();
        if (t < 64 && n0 + t < N) part[(int64_t)blockIdx.y * N + n0 + t] = half[0][t] + half[1][t];
    }
}

// K ranges of a weight gradient (m x n, contraction over K rows): enough to
// give every CU two work-groups where the output has few tiles, none shorter
// than 256 rows
int64_t gemm_max_splits(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((N + 63) / 64) * ((M + 63) / 64);
    if (tiles >= GEMM_WGS || K < 512) return 1;
    return std::max<int64_t>(1, std::min<int64_t>(GEMM_WGS / tiles, K / 256));
}
int64_t gemm_splits(int64_t M, int64_t N, int64_t K) {
    const int64_t splits = gemm_max_splits(M, N, K);
    const int64_t kchunk = ((K + splits - 1) / splits + 15) / 16 * 16;
    return (K + kchunk - 1) / kchunk;
}
int64_t gemm_row_blocks(int64_t M) { return (M + 63) / 64; }

hipError_t launch_gemm(int ta, int tb, int b_bf16, int epi, const float* A, const void* B, const float* bias, float* C,
                       float* Z, int64_t M, int64_t N, int64_t K, int64_t splits, hipStream_t stream, const float* aux,
                       int64_t ldaux, double* part) {
    if (M < 1 || N < 1 || K < 1 || splits < 1 || (splits > 1 && (epi != 0 || bias || Z))) return hipErrorInvalidValue;
    if ((epi >= 3) != (aux != nullptr) || (aux && ldaux < N) || (epi == 4) != (part != nullptr)) return hipErrorInvalidValue;
    const int64_t kchunk = ((K + splits - 1) / splits + 15) / 16 * 16;
    if ((K + kchunk - 1) / kchunk != splits) return hipErrorInvalidValue;
    dim3 grid((N + 63) / 64, (M + 63) / 64, splits), block(256);
#define G(TA, TB, BT, E)                                                                                     \
    hipLaunchKernelGGL((gemm_kernel<TA, TB, BT, E>), grid, block, 0, stream, A, (const BT*)B, bias, C, Z, aux, ldaux, \
                       part, M, N, K, kchunk)
    if (ta == 0 && tb == 0) {
        if (b_bf16) {
            if (epi == 1) G(0, 0, uint16_t, 1);
            else if (epi == 2) G(0, 0, uint16_t, 2);
            else if (epi == 3) G(0, 0, uint16_t, 3);
            else return hipErrorInvalidValue;
        } else {
            if (epi == 1) G(0, 0, float, 1);
            else if (epi == 2) G(0, 0, float, 2);
            else if (epi == 3) G(0, 0, float, 3);
            else return hipErrorInvalidValue;
        }
    } else if (b_bf16) {
        return hipErrorInvalidValue;
    } else if (ta == 0 && tb == 1 && epi == 4) {
        G(0, 1, float, 4);
    } else if (ta == 1 && tb == 1 && epi == 0) {
        G(1, 1, float, 0);
    } else {
        return hipErrorInvalidValue;
    }
#undef G
    return hipGetLastError();
}

// Gradient of every parameter from its partials, then AdamW (the first nw
// entries, the weights, get decoupled weight decay).  Weight entries are the
// sums of the split-K partials in split order, one thread each; a bias entry
// is the FP64 sum of its row-block partials, one wave each, in a fixed order.
// Nothing is written unless coef[3] (the loss kernel's status) is 0.
__global__ __launch_bounds__(256) void grad_adamw_kernel(GradParts gp, const double* __restrict__ coef,
                                                         float* __restrict__ P, float* __restrict__ G,
                                                         float* __restrict__ Mm, float* __restrict__ V, float lr,
                                                         float b1, float b2, float eps, float wd, float c1, float c2) {
    if (coef[3] != 0.0) return;
    const int64_t nw = gp.wsize[0] + gp.wsize[1] + gp.wsize[2];
    const int64_t wblocks = (nw + 255) / 256;
    int64_t i;
    float g;
    bool mine;
    if ((int64_t)blockIdx.x < wblocks) {
        i = (int64_t)blockIdx.x * 256 + threadIdx.x;
        mine = i < nw;
        if (!mine) return;
        int l = 0;
        int64_t e = i;
        while (e >= gp.wsize[l]) e -= gp.wsize[l++];
        g = 0.0f;
#pragma unroll 8
        for (int z = 0; z < gp.splits[l]; ++z) g += gp.wpart[l][z * gp.wsize[l] + e];
    } else {
        int64_t e = ((int64_t)blockIdx.x - wblocks) * 4 + (threadIdx.x >> 6);
        i = nw + e;
        if (e >= gp.bsize[0] + gp.bsize[1] + gp.bsize[2]) return;
        int l = 0;
        while (e >= gp.bsize[l]) e -= gp.bsize[l++];
        double s = 0.0;
        for (int64_t q = threadIdx.x & 63; q < gp.bblocks[l]; q += 64) s += gp.bpart[l][q * gp.bsize[l] + e];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        g = (float)s;
        if ((threadIdx.x & 63) != 0) return;
    }
    G[i] = g;
    const float mi = b1 * Mm[i] + (1.0f - b1) * g;
    const float vi = b2 * V[i] + (1.0f - b2) * g * g;
    Mm[i] = mi;
    V[i] = vi;
    float p = P[i];
    if (i < nw) p -= lr * wd * p;
    p -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    P[i] = p;
}

hipError_t launch_grad_adamw(const GradParts& gp, const double* coef, float* P, float* G, float* M, float* V, float lr,
                             float b1, float b2, float eps, float wd, int64_t t, hipStream_t stream) {
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    const int64_t nw = gp.wsize[0] + gp.wsize[1] + gp.wsize[2], nb = gp.bsize[0] + gp.bsize[1] + gp.bsize[2];
    hipLaunchKernelGGL(grad_adamw_kernel, dim3((nw + 255) / 256 + (nb + 3) / 4), dim3(256), 0, stream, gp, coef, P, G, M,
                       V, lr, b1, b2, eps, wd, c1, c2);
    return hipGetLastError();
}

__global__ void to_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t m) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = f32_to_bf16_bits(x[i]);
}

hipError_t launch_to_bf16(const float* x, uint16_t* y, int64_t m, hipStream_t stream) {
    int64_t blocks = (m + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks), dim3(256), 0, stream, x, y, m);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Successive projection (Gillis & Vavasis 2014) on the rows of R (m x k, FP64,
// stored by columns): argmax of the residual row norms (lowest index on ties),
// then every row is projected off the chosen row's direction.  One launch per
// pick: every work-group finds pick s - 1 from the block maxima of the launch
// before, projects its rows and leaves their block maximum for the next launch
// (two buffers in turn).  The picked row itself is read by all work-groups of
// its launch, so its owner clears it one launch later and counts its norm as 0
// meanwhile.  At k = 16 and 32, the ranks of most solves, a thread has its whole
// row in registers, its loads issued together (at 64 the addresses and the row
// no longer fit).  Four launches per pick over row-major rows (a serial scan of
// the block maxima among them) took 32.3 us a pick at m = 20000, k = 32, reading
// the row twice, eight entries at a time, 11.6 us; this takes 8.6 us.
// ---------------------------------------------------------------------------
__device__ inline void spa_better(double& v, int64_t& i, double ov, int64_t oi) {
    if (ov > v || (ov == v && oi < i)) {
        v = ov;
        i = oi;
    }
}

// argmax over the work-group, valid in every thread
__device__ inline void spa_block_argmax(double& v, int64_t& i, double* sv, int64_t* si) {
    for (int off = 32; off > 0; off >>= 1) spa_better(v, i, __shfl_xor(v, off, 64), __shfl_xor(i, off, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        sv[threadIdx.x >> 6] = v;
        si[threadIdx.x >> 6] = i;
    }
    __syncthreads();
    v = sv[0];
    i = si[0];
    for (int q = 1; q < 4; ++q) spa_better(v, i, sv[q], si[q]);
}

template <int KX>   // k, or 0 for any k
__global__ __launch_bounds__(256) void spa_step_kernel(double* __restrict__ R, int64_t m, int k, int step,
                                                       const double* __restrict__ bval_in,
                                                       const int64_t* __restrict__ bidx_in, int nb,
                                                       double* __restrict__ bval_out, int64_t* __restrict__ bidx_out,
                                                       int64_t* __restrict__ pick) {
    __shared__ double u[KMAX];
    __shared__ double sv[4];
    __shared__ int64_t si[4];
    const int t = threadIdx.x;
    int64_t p = -1, prev = -1;
    if (step > 0) {
        double v = -1.0;
        int64_t i = INT64_MAX;
        for (int b = t; b < nb; b += 256) spa_better(v, i, bval_in[b], bidx_in[b]);
        spa_block_argmax(v, i, sv, si);
        p = i;
        if (step > 1) prev = pick[step - 2];
        if (blockIdx.x == 0 && t == 0) pick[step - 1] = p;
        if (step == k) return;                              // the last launch only picks
        if (t < 64) {
            const double x = t < k ? R[t * m + p] : 0.0;
            double s = 0.0;
            for (int c = 0; c < k; ++c) {
                const double y = __shfl(x, c, 64);
                s += y * y;
            }
            const double nrm = sqrt(s);
            if (t < k) u[t] = nrm > 0.0 ? x / nrm : 0.0;
        }
        __syncthreads();
    }
    double best = -1.0;
    int64_t bi = 0;
    for (int64_t i = blockIdx.x * (int64_t)256 + t; i < m; i += (int64_t)gridDim.x * 256) {
        double s = 0.0;
        if (i == p) {
            // read by every work-group of this launch: left alone
        } else if (i == prev) {
            for (int c = 0; c < k; ++c) R[c * m + i] = 0.0;
        } else if (KX > 0) {
            double x[KX > 0 ? KX : 1];
            double* e = R + i;
#pragma unroll
            for (int c = 0; c < KX; ++c, e += m) x[c] = *e;
            if (step > 0) {
                double d = 0.0;
#pragma unroll
                for (int c = 0; c < KX; ++c) d += x[c] * u[c];
                e = R + i;
#pragma unroll
                for (int c = 0; c < KX; ++c, e += m) {
                    const double r = x[c] - d * u[c];
                    *e = r;
                    s += r * r;
                }
            } else {
#pragma unroll
                for (int c = 0; c < KX; ++c) s += x[c] * x[c];
            }
        } else if (step > 0) {
            double d = 0.0;
#pragma unroll 8
            for (int c = 0; c < k; ++c) d += R[c * m + i] * u[c];
#pragma unroll 8
            for (int c = 0; c < k; ++c) {
                const double r = R[c * m + i] - d * u[c];
                R[c * m + i] = r;
                s += r * r;
            }
        } else {
#pragma unroll 8
            for (int c = 0; c < k; ++c) s += R[c * m + i] * R[c * m + i];
        }
        if (s > best) { best = s; bi = i; }
    }
    spa_block_argmax(best, bi, sv, si);
    if (t == 0) {
        bval_out[blockIdx.x] = best;
        bidx_out[blockIdx.x] = bi;
    }
}

// bval / bidx: two buffers of nb entries each
hipError_t launch_spa(double* R, int64_t m, int64_t k, double* bval, int64_t* bidx, int nb, int64_t* pick,
                      hipStream_t stream) {
    for (int s = 0; s <= k; ++s) {
        const int in = (s + 1) & 1, out = s & 1;
        const dim3 grid(s == k ? 1 : nb), block(256);
#define SPA(KX)                                                                                                   \
    hipLaunchKernelGGL(spa_step_kernel<KX>, grid, block, 0, stream, R, m, (int)k, s, (const double*)bval + in * nb, \
                       (const int64_t*)bidx + in * nb, nb, bval + out * nb, bidx + out * nb, pick)
        if (k == 16) SPA(16);
        else if (k == 32) SPA(32);
        else SPA(0);
#undef SPA
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP64 products of two row-major FP32 matrices over m rows, kx, ky <= 64:
// X^T Y (NP = 1), or X^T X, X^T Y and Y^T Y at once (NP = 3, kx = ky), on the
// FP64 matrix cores.  A work-group stages XTY_ROWS rows, 64 at a time, in LDS
// (rows 80 floats apart: the four rows of an operand read fall on disjoint
// banks); a wave forms the 16 columns of X (and of Y) that are its own against
// all columns, four rows to an MFMA, the operands widened exactly.  The blocks'
// partials are then summed in a fixed order by four phases per entry (one
// thread per entry walked all of them).  The three products of a training step
// at m = 20000, k = 64, 0.5 GFLOP: 99 + 207 us in six launches of vector code
// with two 4-byte LDS reads per FMA, 52 + 6 us in two with a 4 x 4 block in
// registers, 24 + 6 us now.
// ---------------------------------------------------------------------------
constexpr int XTY_ROWS = 128;
constexpr int XTY_LD = KMAX + 16;
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <int NP>
__global__ __launch_bounds__(256) void xty_slab_kernel(const float* __restrict__ X, int64_t ldx, int kx,
                                                       const float* __restrict__ Y, int64_t ldy, int ky, int64_t m,
                                                       double* __restrict__ part) {
    constexpr int NB = KMAX / 16;
    __shared__ float xs[64 * XTY_LD];
    __shared__ float ys[64 * XTY_LD];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, li = lane & 15, lk = lane >> 4;
    doublex4 acc[NP][NB];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[p][n] = doublex4{0.0, 0.0, 0.0, 0.0};
    // a thread's 16 entries of each matrix, both halves' asked for ahead
    float rx[16], ry[16];
    auto load = [&](int half) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int64_t r = (int64_t)blockIdx.x * XTY_ROWS + 64 * half + 4 * q + wv;
            rx[q] = r < m && lane < kx ? X[r * ldx + lane] : 0.0f;
            ry[q] = r < m && lane < ky ? Y[r * ldy + lane] : 0.0f;
        }
    };
    load(0);
#pragma unroll 1
    for (int half = 0; half < XTY_ROWS / 64; ++half) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            xs[(4 * q + wv) * XTY_LD + lane] = rx[q];
            ys[(4 * q + wv) * XTY_LD + lane] = ry[q];
        }
        __syncthreads();
        if (half + 1 < XTY_ROWS / 64) load(half + 1);
        if (16 * wv < kx) {
#pragma unroll 4
            for (int s = 0; s < 16; ++s) {
                const float* x = xs + (4 * s + lk) * XTY_LD + li;
                const float* y = ys + (4 * s + lk) * XTY_LD + li;
                const double xa = (double)x[16 * wv], ya = (double)y[16 * wv];
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    if (16 * n >= ky) break;
                    const double yb = (double)y[16 * n];
                    if (NP == 3) {
                        const double xb = (double)x[16 * n];
                        acc[0][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, xb, acc[0][n], 0, 0, 0);
                        acc[NP == 3 ? 1 : 0][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb, acc[NP == 3 ? 1 : 0][n], 0, 0, 0);
                        acc[NP == 3 ? 2 : 0][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(ya, yb, acc[NP == 3 ? 2 : 0][n], 0, 0, 0);
                    } else {
                        acc[0][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb, acc[0][n], 0, 0, 0);
                    }
                }
            }
        }
    }
    // D of the FP64 form: lane (j, q) holds rows 4 v + q of column j
    const int kk = kx * ky;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int a = 16 * wv + 4 * v + lk, c = 16 * n + li;
                if (a < kx && c < ky) part[((int64_t)blockIdx.x * NP + p) * kk + a * ky + c] = acc[p][n][v];
            }
}

// out[e] = sum over the slabs, 64 entries per work-group, four phases each
__global__ __launch_bounds__(256) void sum_slabs_kernel(const double* __restrict__ part, int64_t slabs, int entries,
                                                        double* __restrict__ out) {
    __shared__ double red[4][64];
    const int lc = threadIdx.x & 63, ph = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lc;
    double s = 0.0;
    if (e < entries) {
#pragma unroll 8
        for (int64_t b = ph; b < slabs; b += 4) s += part[b * entries + e];
    }
    red[ph][lc] = s;
    __syncthreads();
    if (ph == 0 && e < entries) out[e] = red[0][lc] + red[1][lc] + red[2][lc] + red[3][lc];
}

int64_t xty_work_doubles(int64_t m, int64_t kx, int64_t ky) { return ((m + XTY_ROWS - 1) / XTY_ROWS) * kx * ky; }

hipError_t launch_xty(const float* X, int64_t ldx, int64_t kx, const float* Y, int64_t ldy, int64_t ky, int64_t m,
                      double* work, double* out, hipStream_t stream) {
    if (kx < 1 || ky < 1 || kx > KMAX || ky > KMAX || m < 1) return hipErrorInvalidValue;
    const int64_t slabs = (m + XTY_ROWS - 1) / XTY_ROWS;
    hipLaunchKernelGGL(xty_slab_kernel<1>, dim3(slabs), dim3(256), 0, stream, X, ldx, (int)kx, Y, ldy, (int)ky, m, work);
    const int entries = (int)(kx * ky);
    hipLaunchKernelGGL(sum_slabs_kernel, dim3((entries + 63) / 64), dim3(256), 0, stream, (const double*)work, slabs,
                       entries, out);
    return hipGetLastError();
}

// out = [A^T A, A^T B, B^T B], k x k each; work: 3 xty_work_doubles(m, k, k)
hipError_t launch_gram3(const float* A, const float* B, int64_t k, int64_t m, double* work, double* out,
                        hipStream_t stream) {
    if (k < 1 || k > KMAX || m < 1) return hipErrorInvalidValue;
    const int64_t slabs = (m + XTY_ROWS - 1) / XTY_ROWS;
    hipLaunchKernelGGL(xty_slab_kernel<3>, dim3(slabs), dim3(256), 0, stream, A, k, (int)k, B, k, (int)k, m, work);
    const int entries = (int)(3 * k * k);
    hipLaunchKernelGGL(sum_slabs_kernel, dim3((entries + 63) / 64), dim3(256), 0, stream, (const double*)work, slabs,
                       entries, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Symmetric eigen-decomposition of a w x w FP64 matrix (w <= 64) in one
// work-group: cyclic two-sided Jacobi rotations (Golub & Van Loan, Matrix
// Computations, symmetric Schur decomposition of 2 x 2 blocks) in the
// round-robin parallel order, w/2 disjoint rotations at a time.  Then the k
// largest eigenvalues (descending, lower index first on ties) and
// M = V_k diag(lambda)^-1/2 (w x k).  status[0] = 1 when a selected
// eigenvalue is not positive and finite, 2 when the sweeps do not converge.
// A serial chain of about 600 rounds: bound by the latency of a round.  With 32
// pairs a thread owns the 2 x 2 block of two pairs, so J^T A J is one read and
// one write per entry and a round has two barriers (rotations; update of A), A
// and V both in LDS; V, which no rotation depends on, is updated by the other
// waves while one wave computes the next round's rotations (a chain of three
// divisions and two square roots).  Updating rows and columns in turn with V
// in global memory and four barriers a round, the norm and the selection on one
// thread, took 5.13 ms at w = 64; V in the phase of A 1.07 ms; this takes
// 0.75 ms.
// ---------------------------------------------------------------------------
constexpr int JT = 1024;

__global__ __launch_bounds__(JT) void jacobi_topk_kernel(const double* __restrict__ G, int w, int k,
                                                         double* __restrict__ Mout, double* __restrict__ lam_out,
                                                         int32_t* __restrict__ status) {
    __shared__ double A[KMAX][KMAX + 1];
    __shared__ double V[KMAX][KMAX + 1];
    __shared__ int order[KMAX];
    __shared__ int rotated, bad;
    __shared__ uint8_t dead[KMAX + 1];       // columns of a sketch with a NaN in them
    __shared__ double red[JT / 64];
    __shared__ double2 rot[2][KMAX / 2];     // (cos, sin) of every pair, of this round and the one before
    __shared__ int2 pair[2][KMAX / 2];
    const int t = threadIdx.x;
    const int wp = w + (w & 1);    // even player count; index w (odd w) is a bye: a zero row and column
    const int half = wp / 2;
    // A NaN in column p of the sketch makes row and column p of G NaN: they take
    // no part in any rotation, as if they were zero, and the column's eigenvector
    // is its own; the others are those of the rest of G.
    if (t <= w) dead[t] = t < w && !(G[t * w + t] == G[t * w + t]);
    __syncthreads();
    double fro = 0.0;
    for (int e = t; e < wp * wp; e += JT) {
        const int i = e / wp, j = e - i * wp;
        const double a = i < w && j < w && !dead[i] && !dead[j] ? 0.5 * (G[i * w + j] + G[j * w + i]) : 0.0;
        A[i][j] = a;
        V[i][j] = i == j ? 1.0 : 0.0;
        fro += a * a;
    }
    // a pair is rotated when |a_pq| > max(1e-14 sqrt(|a_pp a_qq|), 1e-15 ||G||_F)
    // (the relative criterion of Demmel & Veselic 1992, with an absolute floor
    // so that rounding noise inside a null space of a semidefinite G does not
    // keep the sweeps going); converged after a sweep with no rotation
    for (int off = 32; off > 0; off >>= 1) fro += __shfl_xor(fro, off, 64);
    if ((t & 63) == 0) red[t >> 6] = fro;
    if (t < KMAX) order[t] = 0;
    if (t == 0) bad = 0;
    __syncthreads();
    fro = 0.0;
    for (int q = 0; q < JT / 64; ++q) fro += red[q];
    const double floor_abs = 1e-15 * sqrt(fro);
    const int bi = t / half, bj = t - bi * half;           // the thread's block of A
    int sweep = 0, round = 0;
    // V <- V J with the rotations of a round, by threads first, first + 1, ...
    auto rotate_v = [&](int cur, int first) {
        if (t < first) return;
        int row = (t - first) % w, pr = (t - first) / w;
        const int drow = (JT - first) % w, dpr = (JT - first) / w;
        while (pr < half) {
            const double2 cs = rot[cur][pr];
            if (cs.y != 0.0) {
                const int2 pq = pair[cur][pr];
                const double vp = V[row][pq.x], vq = V[row][pq.y];
                V[row][pq.x] = cs.x * vp - cs.y * vq;
                V[row][pq.y] = cs.y * vp + cs.x * vq;
            }
            row += drow;
            pr += dpr;
            if (row >= w) {
                row -= w;
                ++pr;
            }
        }
    };
    for (; sweep < 60; ++sweep) {
        if (t == 0) rotated = 0;
        __syncthreads();
        for (int r = 0; r < wp - 1; ++r, ++round) {
            // pair i of round r: (wp-1, r) for i = 0, else ((r+i) mod (wp-1), (r-i) mod (wp-1));
            // every rotation is computed from the block before any row is changed
            const int cur = round & 1;
            if (t < half) {
                int p = r + t, q = r - t;
                if (p >= wp - 1) p -= wp - 1;
                if (q < 0) q += wp - 1;
                if (t == 0) p = wp - 1;
                if (p > q) { const int tmp = p; p = q; q = tmp; }
                double c = 1.0, sn = 0.0;
                const double apq = A[p][q], app = A[p][p], aqq = A[q][q];
                if (fabs(apq) > fmax(1e-14 * sqrt(fabs(app * aqq)), floor_abs)) {
                    rotated = 1;
                    const double tau = (aqq - app) / (2.0 * apq);
                    const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                    c = 1.0 / sqrt(1.0 + tt * tt);
                    sn = tt * c;
                }
                rot[cur][t] = double2{c, sn};
                pair[cur][t] = int2{p, q};
            } else if (round > 0) {
                rotate_v(cur ^ 1, 64);                     // of the round before
            }
            __syncthreads();
            // A <- J^T A J by 2 x 2 blocks
            if (bi < half) {
                const double2 ri = rot[cur][bi], rj = rot[cur][bj];
                const double ci = ri.x, si = ri.y, cj = rj.x, sj = rj.y;
                if (si != 0.0 || sj != 0.0) {
                    const int2 i = pair[cur][bi], j = pair[cur][bj];
                    const double a = A[i.x][j.x], b = A[i.x][j.y], c = A[i.y][j.x], d = A[i.y][j.y];
                    const double ra = ci * a - si * c, rb = ci * b - si * d;
                    const double rc = si * a + ci * c, rd = si * b + ci * d;
                    A[i.x][j.x] = cj * ra - sj * rb;
                    A[i.x][j.y] = sj * ra + cj * rb;
                    A[i.y][j.x] = cj * rc - sj * rd;
                    A[i.y][j.y] = sj * rc + cj * rd;
                }
            }
            __syncthreads();
        }
        const int any = rotated;
        __syncthreads();
        if (!any) break;
    }
    if (round > 0) rotate_v((round - 1) & 1, 0);
    __syncthreads();
    // place of every eigenvalue in descending order, lower index first on ties;
    // a dead column comes once all columns before it have been taken
    auto place = [&](int i) {
        int rank = 0;
        for (int j = 0; j < w; ++j) rank += !dead[j] && (A[j][j] > A[i][i] || (A[j][j] == A[i][i] && j < i)) ? 1 : 0;
        return rank;
    };
    if (t < w && !dead[t]) {
        const double l = A[t][t];
        const int rank = place(t);
        if (rank < k) order[rank] = t;
        if (!(l == l) || (rank < k && (!(l > 0.0) || !isfinite(l)))) bad = 1;
    } else if (t < w) {
        int at = 0;
        for (int j = 0; j < t && !dead[j]; ++j) at = max(at, place(j) + 1);
        if (at < k) bad = 1;
    }
    __syncthreads();
    if (t < k) lam_out[t] = A[order[t]][order[t]];
    if (t == 0) status[0] = bad ? 1 : (sweep >= 60 ? 2 : 0);
    for (int e = t; e < w * k; e += JT) {
        const int i = e / k, c = e - i * k;
        const double l = A[order[c]][order[c]];
        Mout[e] = l > 0.0 ? V[i][order[c]] / sqrt(l) : 0.0;
    }
}

hipError_t launch_jacobi_topk(const double* G, int64_t w, int64_t k, double* M, double* lam, int32_t* status,
                              hipStream_t stream) {
    if (w < 1 || w > KMAX || k < 1 || k > w) return hipErrorInvalidValue;
    hipLaunchKernelGGL(jacobi_topk_kernel, dim3(1), dim3(JT), 0, stream, G, (int)w, (int)k, M, lam, status);
    return hipGetLastError();
}

// Y (m x w, FP32) W (w x k, FP64) with FP64 sums: to FP64 by columns (k columns
// of m, the order the anchor search reads), or to FP32 rows of ldo columns, zero
// past k.  A work-group takes 64 rows, a wave 16 columns of them at a time: the
// rows sit in LDS with an odd stride, a lane owns a row and W's entries are the
// same for the whole wave.
template <typename OUT>
__global__ __launch_bounds__(256) void project_rows_kernel(const float* __restrict__ Y, int64_t m, int w,
                                                           const double* __restrict__ W, int k, int ldo,
                                                           OUT* __restrict__ out) {
    __shared__ double Ws[KMAX * KMAX];
    __shared__ float Ys[64][KMAX + 1];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    for (int e = t; e < w * k; e += 256) Ws[e] = W[e];
    for (int f = t; f < 64 * w; f += 256) {
        const int r = f / w, c = f - r * w;
        Ys[r][c] = r0 + r < m ? Y[(r0 + r) * w + c] : 0.0f;
    }
    __syncthreads();
    float res[KMAX / 4];                                    // FP32 form: this lane's row, columns 16 wv ..
#pragma unroll
    for (int q = 0; q < KMAX / 4; ++q) {
        const int c = (KMAX / 4) * wv + q;
        double s = 0.0;
        if (c < k)
            for (int l = 0; l < w; ++l) s += (double)Ys[lane][l] * Ws[l * k + c];
        if (sizeof(OUT) == 8) {
            if (c < k && r0 + lane < m) out[c * m + r0 + lane] = (OUT)s;
        } else {
            res[q] = (float)s;
        }
    }
    if (sizeof(OUT) == 8) return;
    // turn the rows through LDS for a coalesced store
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KMAX / 4; ++q) Ys[lane][(KMAX / 4) * wv + q] = res[q];
    __syncthreads();
    for (int f = t; f < 64 * ldo; f += 256) {
        const int r = f / ldo, c = f - r * ldo;
        if (r0 + r < m) out[(r0 + r) * ldo + c] = (OUT)Ys[r][c];
    }
}

hipError_t launch_project_rows(const float* Y, int64_t m, int64_t w, const double* W, int64_t k, int64_t ldo,
                               int out_f64, void* out, hipStream_t stream) {
    if (w > KMAX || k > KMAX || ldo < k || ldo > KMAX) return hipErrorInvalidValue;
    const dim3 grid((m + 63) / 64), block(256);
    if (out_f64)
        hipLaunchKernelGGL(project_rows_kernel<double>, grid, block, 0, stream, Y, m, (int)w, W, (int)k, (int)ldo,
                           (double*)out);
    else
        hipLaunchKernelGGL(project_rows_kernel<float>, grid, block, 0, stream, Y, m, (int)w, W, (int)k, (int)ldo,
                           (float*)out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Anchor basis in one work-group: A = Y[anchors] M (k x k, FP64), LU with
// partial pivoting, then W = M A^-1 (w x k) by solving A^T w_l = m_l for every
// row l of M.  C = Y W then equals Z A^-1 with Z = Y M.  status[0] = 0, or 3
// when a pivot is below 1e-13 times the largest entry of A.
// ---------------------------------------------------------------------------
// A serial chain of 3 k short stages: the pivot is found by one wave, the solves
// update all rows of M at once, column by column (the subtractions of a row keep
// their order).  Pivots and row solves on single threads, the latter with their
// vector in scratch memory, took 163 us at w = 64, k = 32; this takes 94 us.
__global__ __launch_bounds__(256) void anchor_solve_kernel(const float* __restrict__ Y, int w,
                                                           const double* __restrict__ M, int k,
                                                           const int64_t* __restrict__ anchors, double* __restrict__ W,
                                                           int32_t* __restrict__ status) {
    __shared__ double LU[KMAX][KMAX + 1];
    __shared__ double X[KMAX][KMAX + 1];
    __shared__ int perm[KMAX];
    __shared__ double wmax[4];
    __shared__ int piv, singular;
    const int t = threadIdx.x;
    if (t == 0) singular = 0;
    double mx = 0.0;
    for (int e = t; e < k * k; e += 256) {
        const int j = e / k, c = e - j * k;
        const int64_t row = anchors[j];
        double s = 0.0;
#pragma unroll 8
        for (int l = 0; l < w; ++l) s += (double)Y[row * w + l] * M[l * k + c];
        LU[j][c] = s;
        mx = fmax(mx, fabs(s));
    }
    for (int e = t; e < w * k; e += 256) X[e / k][e % k] = M[e];
    if (t < k) perm[t] = t;
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
    if ((t & 63) == 0) wmax[t >> 6] = mx;
    __syncthreads();
    const double amax = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
    for (int j = 0; j < k; ++j) {
        if (t < 64) {
            // largest |entry| of the column at or below the diagonal, the first on ties
            double v = t >= j && t < k ? fabs(LU[t][j]) : -1.0;
            int i = t >= j && t < k ? t : KMAX;
            for (int off = 32; off > 0; off >>= 1) {
                const double ov = __shfl_xor(v, off, 64);
                const int oi = __shfl_xor(i, off, 64);
                if (ov > v || (ov == v && oi < i)) {
                    v = ov;
                    i = oi;
                }
            }
            if (t == 0) {
                piv = i < k ? i : j;                       // a column of NaNs: no exchange, singular
                if (!(v > 1e-13 * amax)) singular = 1;
            }
        }
        __syncthreads();
        const int p = piv;
        if (p != j) {
            for (int c = t; c < k; c += 256) {
                const double tmp = LU[j][c];
                LU[j][c] = LU[p][c];
                LU[p][c] = tmp;
            }
            if (t == 0) { const int tp = perm[j]; perm[j] = perm[p]; perm[p] = tp; }
        }
        __syncthreads();
        const double d = LU[j][j];
        for (int i = j + 1 + t; i < k; i += 256) LU[i][j] = d != 0.0 ? LU[i][j] / d : 0.0;
        __syncthreads();
        for (int e = t; e < (k - j - 1) * (k - j - 1); e += 256) {
            const int i = j + 1 + e / (k - j - 1), c = j + 1 + e % (k - j - 1);
            LU[i][c] -= LU[i][j] * LU[j][c];
        }
        __syncthreads();
    }
    // P A = L U  =>  A^T = U^T L^T P.  For row l of M: U^T y = m (forward),
    // L^T x = y (backward, unit diagonal), w = P^T x, i.e. w[perm[i]] = x[i].
    for (int j = 0; j < k; ++j) {
        const double d = LU[j][j];
        for (int l = t; l < w; l += 256) X[l][j] = d != 0.0 ? X[l][j] / d : 0.0;
        __syncthreads();
        for (int e = t; e < w * (k - j - 1); e += 256) {
            const int l = e % w, i = j + 1 + e / w;
            X[l][i] -= LU[j][i] * X[l][j];
        }
        __syncthreads();
    }
    for (int j = k - 1; j > 0; --j) {
        for (int e = t; e < w * j; e += 256) {
            const int l = e % w, i = e / w;
            X[l][i] -= LU[j][i] * X[l][j];
        }
        __syncthreads();
    }
    for (int e = t; e < w * k; e += 256) W[(e / k) * k + perm[e % k]] = X[e / k][e % k];
    if (t == 0) status[0] = singular ? 3 : 0;
}

hipError_t launch_anchor_solve(const float* Y, int64_t w, const double* M, int64_t k, const int64_t* anchors,
                               double* W, int32_t* status, hipStream_t stream) {
    if (w > KMAX || k > KMAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(anchor_solve_kernel, dim3(1), dim3(256), 0, stream, Y, (int)w, M, (int)k, anchors, W, status);
    return hipGetLastError();
}

// Loss and its gradient's coefficients from gram3 = [A^T A, A^T B, B^T B]
// (one work-group): coef = {L, ca, cb, status}, the gradient being
// dA = ca A (A^T A) - cb B (B^T A).  With a, b, c the squared norms of the
// three products, kind 0: L = (a - 2 b + c) / c, ca = cb = 4 / c; kind 1:
// L = 1 - b^2 / (a c), cb = 4 b / (a c), ca = cb b / a.  status 1: c is zero or
// not finite; 2 (kind 1): a is zero; 3: L is not finite.  On the device so
// that a training step waits for the host once, at its end.
__global__ __launch_bounds__(256) void loss_coef_kernel(const double* __restrict__ gram3, int kk, int kind,
                                                        double* __restrict__ coef) {
    __shared__ double red[3][4];
    const int t = threadIdx.x;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        double s = 0.0;
#pragma unroll 4
        for (int e = t; e < kk; e += 256) {
            const double v = gram3[p * kk + e];
            s += v * v;
        }
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if ((t & 63) == 0) red[p][t >> 6] = s;
    }
    __syncthreads();
    if (t != 0) return;
    const double a = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    const double b = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    const double c = red[2][0] + red[2][1] + red[2][2] + red[2][3];
    double L = 0.0, ca = 0.0, cb = 0.0, status = 0.0;
    if (!(c > 0.0) || !isfinite(c)) {
        status = 1.0;
    } else if (kind == 0) {
        L = (a - 2.0 * b + c) / c;
        ca = cb = 4.0 / c;
    } else if (!(a > 0.0)) {
        status = 2.0;
    } else {
        L = 1.0 - b * b / (a * c);
        cb = 4.0 * b / (a * c);
        ca = cb * b / a;
    }
    if (status == 0.0 && !isfinite(L)) status = 3.0;
    coef[0] = L;
    coef[1] = ca;
    coef[2] = cb;
    coef[3] = status;
}

hipError_t launch_loss_coef(const double* gram3, int64_t k, int kind, double* coef, hipStream_t stream) {
    hipLaunchKernelGGL(loss_coef_kernel, dim3(1), dim3(256), 0, stream, gram3, (int)(k * k), kind, coef);
    return hipGetLastError();
}

// Backward of the Gram loss through the network's output, 64 rows per
// work-group: dA = ca A (A^T A) - cb B (B^T A) on the FP32 matrix cores (both
// Gram losses have this form), dZ = dA f'(Z) with f the residual output
// max(X + z, 0) or softplus, and the FP64 column sums of dZ (the last layer's
// bias gradient).  Rows and the k x k products sit in LDS, zero-padded to a
// multiple of 16 columns; an operand read of four consecutive reduction
// indices feeds four MFMAs.  m = 20000, k = 64: 61 us in two launches (scalar
// dot products, then the activation) before, 25 us now.
template <int KP, bool RES>
__global__ __launch_bounds__(256) void loss_backward_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                            const double* __restrict__ gram3,
                                                            const double* __restrict__ coef,
                                                            const float* __restrict__ X, int64_t ldx,
                                                            const float* __restrict__ Zpre, int k, int64_t m,
                                                            float* __restrict__ dZ, double* __restrict__ part) {
    constexpr int LD = KP + 4, NB = KP / 16;
    __shared__ __align__(16) float As[64 * LD], Bs[64 * LD];
    __shared__ float Ps[KP * LD], Qs[KP * LD];
    __shared__ double red[4][KP];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * 64;
    for (int f = t; f < 64 * KP; f += 256) {
        const int r = f / KP, c = f - r * KP;
        const bool in = r0 + r < m && c < k;
        As[r * LD + c] = in ? A[(r0 + r) * k + c] : 0.0f;
        Bs[r * LD + c] = in ? B[(r0 + r) * k + c] : 0.0f;
    }
    for (int f = t; f < KP * KP; f += 256) {
        const int j = f / KP, c = f - j * KP;
        const bool in = j < k && c < k;
        Ps[j * LD + c] = in ? (float)gram3[j * k + c] : 0.0f;
        Qs[c * LD + j] = in ? (float)gram3[k * k + j * k + c] : 0.0f;   // Q[c][j] = (A^T B)_jc
    }
    __syncthreads();
    floatx4 ga[NB], gb[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) ga[n] = gb[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NB; ++s) {
        const floatx4 av = *(const floatx4*)&As[(16 * wv + lr) * LD + 16 * s + 4 * lg];
        const floatx4 bv = *(const floatx4*)&Bs[(16 * wv + lr) * LD + 16 * s + 4 * lg];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const int o = (16 * s + 4 * lg + e) * LD + 16 * n + lr;
                ga[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], Ps[o], ga[n], 0, 0, 0);
                gb[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[e], Qs[o], gb[n], 0, 0, 0);
            }
    }
    const float ca = (float)coef[1], cb = (float)coef[2];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int c = 16 * n + lr;
        double s = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t r = r0 + 16 * wv + 4 * lg + v;
            if (r < m && c < k) {
                const float dA = ca * ga[n][v] - cb * gb[n][v];
                const float z = Zpre[r * k + c];
                const float d = RES ? (X[r * ldx + c] + z > 0.0f ? dA : 0.0f) : dA * (0.5f * (1.0f + tanhf(0.5f * z)));
                dZ[r * k + c] = d;
                s += (double)d;
            }
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (lg == 0) red[wv][c] = s;
    }
    __syncthreads();
    for (int c = t; c < k; c += 256) part[blockIdx.x * (int64_t)k + c] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
}

int64_t loss_backward_blocks(int64_t m) { return (m + 63) / 64; }

hipError_t launch_loss_backward(const float* A, const float* B, const double* gram3, const double* coef, const float* X,
                                int64_t ldx, const float* Z, int residual, int64_t k, int64_t m, float* dZ, double* part,
                                hipStream_t stream) {
    if (k < 1 || k > KMAX || m < 1) return hipErrorInvalidValue;
    const dim3 grid(loss_backward_blocks(m)), block(256);
#define LB(KP)                                                                                                    \
    do {                                                                                                          \
        if (residual)                                                                                             \
            hipLaunchKernelGGL((loss_backward_kernel<KP, true>), grid, block, 0, stream, A, B, gram3, coef, X, ldx, Z, \
                               (int)k, m, dZ, part);                                                              \
        else                                                                                                      \
            hipLaunchKernelGGL((loss_backward_kernel<KP, false>), grid, block, 0, stream, A, B, gram3, coef, X, ldx, Z, \
                               (int)k, m, dZ, part);                                                              \
    } while (0)
    if (k <= 16) LB(16); else if (k <= 32) LB(32); else LB(64);
#undef LB
    return hipGetLastError();
}

// out (m x k) = max(X[:, :k], 0) for X (m x w)
__global__ void clip_cols_kernel(const float* __restrict__ X, int64_t m, int w, int k, float* __restrict__ out) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m * k; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / k;
        const int c = (int)(e - i * k);
        out[e] = fmaxf(X[i * w + c], 0.0f);
    }
}

hipError_t launch_clip_cols(const float* X, int64_t m, int64_t w, int64_t k, float* out, hipStream_t stream) {
    int64_t blocks = (m * k + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(clip_cols_kernel, dim3(blocks), dim3(256), 0, stream, X, m, (int)w, (int)k, out);
    return hipGetLastError();
}

__global__ void scale_kernel(float* __restrict__ x, int64_t m, float a) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x)
        x[e] *= a;
}

hipError_t launch_scale(float* x, int64_t m, float a, hipStream_t stream) {
    int64_t blocks = (m + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(scale_kernel, dim3(blocks), dim3(256), 0, stream, x, m, a);
    return hipGetLastError();
}

// ||M_A^T (A^T B) M_B||_F^2 for k x k FP64 matrices (one work-group); with
// M_X^T (X^T X) M_X = I this is ||Q_A^T Q_B||_F^2 of orthonormal bases of the
// column spans of A and B.
__global__ __launch_bounds__(256) void span_overlap_kernel(const double* __restrict__ MA,
                                                           const double* __restrict__ AtB,
                                                           const double* __restrict__ MB, int k,
                                                           double* __restrict__ out) {
    __shared__ double T[KMAX * KMAX];
    __shared__ double red[4];
    for (int e = threadIdx.x; e < k * k; e += 256) {
        const int i = e / k, j = e - i * k;
        double s = 0.0;
        for (int l = 0; l < k; ++l) s += AtB[i * k + l] * MB[l * k + j];
        T[e] = s;   // (A^T B M_B)_ij
    }
    __syncthreads();
    double acc = 0.0;
    for (int e = threadIdx.x; e < k * k; e += 256) {
        const int i = e / k, j = e - i * k;
        double q = 0.0;
        for (int l = 0; l < k; ++l) q += MA[l * k + i] * T[l * k + j];
        acc += q * q;
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = red[0] + red[1] + red[2] + red[3];
}

hipError_t launch_span_overlap(const double* MA, const double* AtB, const double* MB, int64_t k, double* out,
                               hipStream_t stream) {
    if (k < 1 || k > KMAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(span_overlap_kernel, dim3(1), dim3(256), 0, stream, MA, AtB, MB, (int)k, out);
    return hipGetLastError();
}

}  // namespace symnmf
