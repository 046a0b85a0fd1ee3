// Fused gradient + optimiser update of one iteration, and the FP64 reductions
// behind the objective and the stop rule.
//
// For every row tile of the panel the update kernel
//   * sums the S.H partials of the tile (stream kernel output) - or, for a
//     row the step did not sample, takes the snapshot gradient mu,
//   * forms g = c_g (H (Gram_eff) - S H) with the k x k Gram in LDS
//     (paper: grad f = 4 (H (H^T H) - S H), H (H^T H) formed right to left;
//     block steps: c_g = 2 with the block Gram, appendix Block-SVRG),
//   * applies the AdaGrad / RMSprop rule in projected or softplus form
//     (appendix family 3; eq. logspace_grad for softplus),
//   * writes H_{t+1} and accumulates in FP64 the per-tile partials of
//     tr(H_t^T S H_t), ||grad_proj||^2 (eq. proj_grad) and Gram(H_{t+1}).
// The finalize kernel reduces the tile partials in a fixed order.
#include "admm_inverse.h"
#include "image.h"

namespace symnmf {

template <typename T> __device__ inline T dev_sqrt(T x);
template <> __device__ inline float dev_sqrt<float>(float x) { return __builtin_sqrtf(x); }
template <> __device__ inline double dev_sqrt<double>(double x) { return __builtin_sqrt(x); }

// softplus(x) = max(x, 0) + log1p(exp(-|x|)); sigmoid(x) = 1 / (1 + exp(-x))
__device__ inline float softplus_f(float x) { return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x))); }
__device__ inline double softplus_f(double x) { return fmax(x, 0.0) + log1p(exp(-fabs(x))); }
__device__ inline float sigmoid_f(float x) { return 0.5f * (1.0f + tanhf(0.5f * x)); }
__device__ inline double sigmoid_f(double x) { return 0.5 * (1.0 + tanh(0.5 * x)); }

// tr, kkt and the non-finite count of a work-group of UT threads at once
__device__ inline void block_sum3(double& tr, double& kkt, double& bad, double (*sh)[3]) {
    const int t = threadIdx.x;
    for (int off = 32; off > 0; off >>= 1) {
        tr += __shfl_down(tr, off, 64);
        kkt += __shfl_down(kkt, off, 64);
        bad += __shfl_down(bad, off, 64);
    }
    if ((t & 63) == 0) {
        sh[t >> 6][0] = tr;
        sh[t >> 6][1] = kkt;
        sh[t >> 6][2] = bad;
    }
    __syncthreads();
    tr = kkt = bad = 0.0;
    if (t == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
            tr += sh[i][0];
            kkt += sh[i][1];
            bad += sh[i][2];
        }
}

__device__ inline double block_sum(double v, double* sh) {
    const int t = threadIdx.x;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __syncthreads();
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (t == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
    __syncthreads();
    return s;   // valid in thread 0
}

// Threads of the update work-group (one row slice of SR rows).  A slice is a
// chain of short phases (loads, H (H^T H), the rule, the Gram), each bound by
// the latency of LDS reads when a SIMD has one wave of it: with 256 threads the
// phases of a 64-column slice took 4.9, 8.8, 5.4 and 10 us of 31.  us a step
// with 256 threads and now, FP32 S: MU k = 64 n = 512 48.5 / 33.8, n = 4100 80 / 65;
// MU k = 32 n = 4100 38.5 / 36.5; ADMM k = 64 n = 512 70 / 54, n = 4100 121 / 104,
// k = 32 n = 512 29.2 / 24.9, k = 16 n = 512 18.7 / 17.9.  The row share of n = 10^6,
// k = 64: 62 / 37 us in the kernel; n = 10^5, k = 32, FP8 S, AdaGrad, where the
// slices fill the card: 49.5 / 57.4 of 1615.
template <typename HT, int KB>
constexpr int update_threads() {
    return sizeof(HT) == 8 ? 256 : (KB == 64 ? 1024 : 512);
}

// RULE: the update rule (SYMNMF_ADAM stands for NADAM too), SP: its softplus form.
// Both are fixed at compile time: with every rule in one kernel a slice of
// 64 x 32 took 18.5 us at n = 4100 (68 work-groups, so the time of one; 16.1 us
// now), most of it code and registers of the other rules.
template <typename HT, int KB, int RULE, bool SP>
__global__ __launch_bounds__((update_threads<HT, KB>()), sizeof(HT) == 8 ? 1 : (KB == 64 ? 4 : 5)) void update_kernel(UpdateArgs a, PlanView p) {
    constexpr int UT = update_threads<HT, KB>();
    __shared__ __align__(32) HT Hs[SR * KB];
    __shared__ __align__(32) HT Hns[SR * KB];
    __shared__ HT Gs[KB * KB];
    __shared__ double red[UT / 64][3];
    const int t = threadIdx.x;
    const int64_t slice = blockIdx.x;
    const int64_t tile = slice / SUBT;
    const int r0 = (int)(slice % SUBT) * SR;           // first tile row of the slice
    const int k = (int)a.k;
    const int32_t act = p.full ? (int32_t)tile : p.tile_active[tile];
    const int cls = (act >= 0 && !p.full) ? p.active_class[act] : 0;
    const HT* gram = (const HT*)a.gram_eff + (int64_t)cls * k * k;
    constexpr int NJ = SR * KB / UT;
    const int c = t % KB, rb = t / KB;
    int64_t w_lo, w_hi, slot_base, slot_mul;
    partial_slots(p, act, w_lo, w_hi, slot_base, slot_mul);
    const HT* part = (const HT*)a.part;
    HT* G = (HT*)a.G;
    HT* M = (HT*)a.M;
    HT* Th = (HT*)a.Theta;
    HT* Mu = (HT*)a.Mu;
    HT* Go = (HT*)a.Gout;
    HT* Hn = (HT*)a.Hn;
    const HT eta = (HT)a.eta, eps = (HT)a.eps, alpha = (HT)a.alpha, mom = (HT)a.mu, cg = (HT)a.cgrad;
    const int64_t g0 = a.row0 + tile * TR + r0;       // global row of slice row 0
    const HT* Ht = (const HT*)a.H;
    // What a thread needs from memory is asked for before the first barrier, so
    // that a slice waits for memory once: the Gram and H into LDS, the S.H
    // partials and the accumulator of its own elements into registers.
    // The partials are summed over the writing work-groups in increasing order,
    // the loads of all elements of one work-group issued together (a row of the
    // n = 10^6 share has ten partials: one after another they are ten dependent
    // load latencies per element).
    constexpr int NG = (KB * KB + UT - 1) / UT;
    HT shv[NJ], gv[NJ], hl[NJ], gl[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int e = t + UT * q, i = e / KB, j = e % KB;
        gl[q] = i < k && j < k ? gram[i * k + j] : (HT)0;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rb + j * (UT / KB);
        const int64_t prow = tile * TR + r0 + r;
        hl[j] = c < k ? Ht[(g0 + r) * k + c] : (HT)0;
        gv[j] = prow < a.rows && c < k && RULE != SYMNMF_MU ? G[prow * k + c] : (HT)0;
        shv[j] = 0;
    }
    if (act >= 0 && c < k) {
        for (int64_t w = w_lo; w <= w_hi; ++w) {
            const HT* pw = part + ((slot_mul * w + slot_base) * TR + r0 + rb) * a.kp + c;
#pragma unroll
            for (int j = 0; j < NJ; ++j) shv[j] += pw[j * (UT / KB) * a.kp];
        }
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
        if (t + UT * q < KB * KB) Gs[t + UT * q] = gl[q];
#pragma unroll
    for (int j = 0; j < NJ; ++j) Hs[t + UT * j] = hl[j];
    __syncthreads();
    // Elements f = t + UT j of the slice in rows of KB columns (those past k are
    // zero and have no storage): a thread's elements share the column
    // c = t % KB, as UT is a multiple of KB, so every Gram entry of H (H^T H) is
    // read from LDS once for all of them and the H rows in 4-wide vectors.
    typedef HT hvec4 __attribute__((ext_vector_type(4)));
    HT hgv[NJ];
    if (act >= 0) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) hgv[j] = 0;
#pragma unroll 2
        for (int b = 0; b < KB; b += 4) {
            const HT g0 = Gs[b * KB + c], g1 = Gs[(b + 1) * KB + c], g2 = Gs[(b + 2) * KB + c],
                     g3 = Gs[(b + 3) * KB + c];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const hvec4 hv = *(const hvec4*)&Hs[(rb + j * (UT / KB)) * KB + b];
                HT v = hgv[j];
                v += hv[0] * g0;
                v += hv[1] * g1;
                v += hv[2] * g2;
                v += hv[3] * g3;
                hgv[j] = v;
            }
        }
    }
    double tr = 0.0, kkt = 0.0;
    int bad = 0;
    // the element of slice row r and this thread's column, with its S.H sum,
    // H (H^T H) entry and accumulator
    auto element = [&](int r, HT sh_in, HT hg_in, HT acc_in) {
        const int64_t prow = tile * TR + r0 + r;
        HT hn = 0;
        if (prow < a.rows && c < k) {
            const HT h = Hs[r * KB + c];
            const int64_t idx = prow * k + c;
            HT g, sh = 0, hg = 0;
            if (act >= 0) {
                sh = sh_in;
                if (a.fp8) {   // codes carry S * scale off the diagonal; S_ii is kept exactly
                    // and enters with the weight the plan gives column i of this row:
                    // 1 on full and row-sampled steps; on a block step 0 for rows in I
                    // only or J only (their own block is not among the streamed
                    // chunks) and 2 for rows in both sets
                    const HT dw = (p.full || !a.block_step) ? (HT)1 : (cls == 2 ? (HT)2 : (HT)0);
                    sh = sh / (HT)a.panel_scale[(uint32_t)prow / (uint32_t)a.panel_rows] + dw * (HT)a.diag[prow] * h;
                }
                hg = hg_in;
                g = cg * (hg - sh);
                tr += (double)h * (double)sh;
            } else {
                g = Mu[idx];
            }
            const HT pg = SP ? g : (h > (HT)0 ? g : (g < (HT)0 ? g : (HT)0));
            kkt += (double)pg * (double)pg;
            if (!(g == g) || g - g != (HT)0) ++bad;
            if (a.store_mu) Mu[idx] = g;
            if (Go) Go[idx] = g;
            if (RULE == SYMNMF_ADAM || RULE == SYMNMF_ADAN) {
                // family 3, Adam-type rules on x = Theta (softplus) or H (projected)
                const HT x = SP ? Th[idx] : h;
                const HT gx = SP ? g * sigmoid_f(x) : g;
                const HT b1 = (HT)a.beta1, b2 = (HT)a.beta2;
                const HT m = b1 * M[idx] + ((HT)1 - b1) * gx;
                M[idx] = m;
                HT step;
                if (RULE == SYMNMF_ADAN) {
                    const HT b3 = (HT)a.beta3;
                    HT* D = (HT*)a.D;
                    HT* Gp = (HT*)a.Gp;
                    const HT diff = a.first ? (HT)0 : gx - Gp[idx];
                    const HT d = b2 * D[idx] + ((HT)1 - b2) * diff;
                    const HT u = gx + b2 * diff;
                    const HT nv = b3 * acc_in + ((HT)1 - b3) * u * u;
                    D[idx] = d;
                    G[idx] = nv;
                    Gp[idx] = gx;
                    step = (m / (HT)a.bc1 + b2 * d / (HT)a.bc2) / (dev_sqrt(nv / (HT)a.bc3) + eps);
                } else {
                    const HT v = b2 * acc_in + ((HT)1 - b2) * gx * gx;
                    G[idx] = v;
                    HT mh = m / (HT)a.bc1;
                    if (a.method == SYMNMF_NADAM) mh = b1 * mh + ((HT)1 - b1) * gx / (HT)a.bc1;
                    step = mh / (dev_sqrt(v / (HT)a.bc2) + eps);
                }
                const HT xn = x - eta * step;
                if (SP) {
                    Th[idx] = xn;
                    hn = softplus_f(xn);
                } else {
                    hn = xn > (HT)0 ? xn : (HT)0;
                }
            } else if (RULE == SYMNMF_MU) {
                // family 1: dampened multiplicative update, H stays >= 0
                hn = (HT)0.5 * h * ((HT)1 + sh / (hg + eps));
            } else if (SP) {
                HT th = Th[idx];
                const HT gt = g * sigmoid_f(th);
                if (RULE == SYMNMF_RMSPROP) {
                    const HT v = alpha * acc_in + ((HT)1 - alpha) * gt * gt;
                    const HT m = mom * M[idx] + eta * gt / (dev_sqrt(v) + eps);
                    G[idx] = v;
                    M[idx] = m;
                    th -= m;
                } else {
                    const HT acc = acc_in + gt * gt;
                    G[idx] = acc;
                    th -= eta * gt / (dev_sqrt(acc) + eps);
                }
                Th[idx] = th;
                hn = softplus_f(th);
            } else if (RULE == SYMNMF_RMSPROP) {
                const HT v = alpha * acc_in + ((HT)1 - alpha) * g * g;
                const HT m = mom * M[idx] + eta * g / (dev_sqrt(v) + eps);
                G[idx] = v;
                M[idx] = m;
                hn = h - m;
                hn = hn > (HT)0 ? hn : (HT)0;
            } else {
                const HT acc = acc_in + g * g;
                G[idx] = acc;
                hn = h - eta * g / (dev_sqrt(acc) + eps);
                hn = hn > (HT)0 ? hn : (HT)0;
            }
            Hn[(g0 + r) * k + c] = hn;
        }
        Hns[r * KB + c] = hn;
    };
    // compile-time j, so the precomputed sums stay in registers
#pragma unroll
    for (int j = 0; j < NJ; ++j) element(rb + j * (UT / KB), shv[j], hgv[j], gv[j]);
    __syncthreads();
    if constexpr (sizeof(HT) == 4)
        if (a.img1 && g0 < a.n_chunks * KC)
            write_image_slice<KB, UT>(a.img_kind, Hns, Hs, (int)min(a.rows - tile * TR - r0, (int64_t)SR), g0, a.img1, a.img2);
    double* tg = a.tile_gram + slice * (int64_t)k * k;
    if (KB >= 32) {
        // each thread: entries (ia0 + q, ib), q < NQ, consecutive ia read as
        // aligned vectors; the same FP64 sums over the slice rows
        constexpr int NQ = KB >= 32 ? (KB * KB) / UT : 4;
        constexpr int VQ = NQ < 4 ? NQ : 4;
        static_assert(NQ % VQ == 0, "vector reads of the Gram rows");
        typedef HT hvecq __attribute__((ext_vector_type(VQ)));
        const int ib = t % KB, ia0 = (t / KB) * NQ;
        double sq[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) sq[q] = 0.0;
#pragma unroll 4
        for (int r = 0; r < SR; ++r) {
            const double hb = (double)Hns[r * KB + ib];
#pragma unroll
            for (int q = 0; q < NQ; q += VQ) {
                const hvecq hv = *(const hvecq*)&Hns[r * KB + ia0 + q];
#pragma unroll
                for (int e = 0; e < VQ; ++e) sq[q + e] += (double)hv[e] * hb;
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (ia0 + q < k && ib < k) tg[(ia0 + q) * k + ib] = sq[q];
    } else {
        for (int e = t; e < k * k; e += UT) {
            const int ia = e / k, ib = e - ia * k;
            double s = 0.0;
#pragma unroll 8
            for (int r = 0; r < SR; ++r) s += (double)Hns[r * KB + ia] * (double)Hns[r * KB + ib];
            tg[e] = s;
        }
    }
    double nbad = (double)bad;
    block_sum3(tr, kkt, nbad, red);
    if (t == 0) {
        a.tile_tr[slice] = tr;
        a.tile_kkt[slice] = kkt;
        a.tile_bad[slice] = (int32_t)nbad;
    }
}

template <typename HT, int RULE, bool SP>
static hipError_t launch_rule(const UpdateArgs& a, const PlanView& p, hipStream_t stream) {
    const dim3 grid(a.rows_pad / TR * SUBT);
    constexpr bool F64 = sizeof(HT) == 8;
#define UPDATE(KB) \
    hipLaunchKernelGGL((update_kernel<HT, KB, RULE, SP>), grid, dim3((update_threads<HT, KB>())), 0, stream, a, p)
    if (F64 && a.k <= 8) UPDATE(F64 ? 8 : 16);
    else if (a.k <= 16) UPDATE(16);
    else if (a.k <= 32) UPDATE(32);
    else if (!F64) UPDATE(F64 ? 32 : 64);
#undef UPDATE
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename HT>
static hipError_t launch_update_t(const UpdateArgs& a, const PlanView& p, hipStream_t stream) {
#define RULE(R) return a.softplus ? launch_rule<HT, R, true>(a, p, stream) : launch_rule<HT, R, false>(a, p, stream)
    switch (a.method) {
        case SYMNMF_ADAGRAD: RULE(SYMNMF_ADAGRAD);
        case SYMNMF_RMSPROP: RULE(SYMNMF_RMSPROP);
        case SYMNMF_ADAM:
        case SYMNMF_NADAM: RULE(SYMNMF_ADAM);
        case SYMNMF_ADAN: RULE(SYMNMF_ADAN);
        case SYMNMF_MU:
            if (!a.softplus) return launch_rule<HT, SYMNMF_MU, false>(a, p, stream);
    }
#undef RULE
    return hipErrorInvalidValue;
}

hipError_t launch_update(const UpdateArgs& a, int h_f64, const PlanView& p, hipStream_t stream) {
    return h_f64 ? launch_update_t<double>(a, p, stream) : launch_update_t<float>(a, p, stream);
}

// ---------------------------------------------------------------------------
// ADMM (appendix family 6).  Per step: the inverse of M = 2 W^T W + rho I (k x k,
// FP64 Gauss-Jordan in place in one work-group; M is symmetric positive
// definite, so no pivoting), then one fused pass over the rows of the panel that sums the
// S.W partials and, per row,
//   * records the statistics of W_t: tr partial W . SW, the projected gradient
//     of g = 4 (W (W^T W) - S W) (the stop rule is taken on W),
//   * a = 2 SW + rho (W - U) and H = a M^-1 (eq. admm_H),
//   * W_{t+1} = [H + U]_+ (eq. admm_W), U <- U + H - W_{t+1} (eq. admm_U),
//   * the FP64 Gram partials of W_{t+1}.
// ---------------------------------------------------------------------------
template <typename HT, int BS>
__global__ __launch_bounds__(256) void admm_minv_kernel(const double* __restrict__ gram, int k, double rho,
                                                        HT* __restrict__ minv) {
    __shared__ double rc[4 * KMAX];
    admm_inverse<HT, BS>(gram, k, rho, minv, rc);
}

template <typename HT>
static void launch_minv(const double* gram, int k, double rho, HT* minv, hipStream_t stream) {
    if (k <= 16) hipLaunchKernelGGL((admm_minv_kernel<HT, 1>), dim3(1), dim3(256), 0, stream, gram, k, rho, minv);
    else if (k <= 32) hipLaunchKernelGGL((admm_minv_kernel<HT, 2>), dim3(1), dim3(256), 0, stream, gram, k, rho, minv);
    else hipLaunchKernelGGL((admm_minv_kernel<HT, 4>), dim3(1), dim3(256), 0, stream, gram, k, rho, minv);
}

template <typename HT, int KB>
__global__ __launch_bounds__((update_threads<HT, KB>()), sizeof(HT) == 4 ? 4 : 1) void admm_update_kernel(UpdateArgs a, PlanView p) {
    constexpr int UT = update_threads<HT, KB>();
    __shared__ __align__(32) HT Ws[SR * KB];
    __shared__ __align__(32) HT Wns[SR * KB];
    __shared__ __align__(32) HT As[SR * KB];
    __shared__ HT Gs[KB * KB];
    __shared__ HT Ms[KB * KB];
    __shared__ double red[UT / 64][3];
    const int t = threadIdx.x;
    const int64_t slice = blockIdx.x;
    const int64_t tile = slice / SUBT;
    const int r0 = (int)(slice % SUBT) * SR;
    const int k = (int)a.k;
    const int32_t act = (int32_t)tile;                  // full steps only
    const HT* gram = (const HT*)a.gram_eff;
    const HT* minv = (const HT*)a.minv;
    // Elements f = t + UT j in rows of KB columns (zero past k), sharing the
    // column cc = t % KB, as in the update kernel: the Gram and M^-1 entries of
    // the column are read from LDS once for all rows (rows in 4-wide vectors),
    // and everything from memory, the S.W partials and the dual among it, is
    // asked for before the first barrier.
    constexpr int NJ = SR * KB / UT;
    typedef HT hvec4 __attribute__((ext_vector_type(4)));
    const int cc = t % KB, rb = t / KB;
    const int64_t g0 = a.row0 + tile * TR + r0;
    const HT* Wt = (const HT*)a.H;
    int64_t w_lo, w_hi, slot_base, slot_mul;
    partial_slots(p, act, w_lo, w_hi, slot_base, slot_mul);
    const HT* part = (const HT*)a.part;
    HT* Ud = (HT*)a.M;
    HT* Go = (HT*)a.Gout;
    HT* Wn = (HT*)a.Hn;
    const HT rho = (HT)a.rho;
    constexpr int NG = (KB * KB + UT - 1) / UT;
    HT swv[NJ], wgv[NJ], uv[NJ], wl[NJ], gl[NG], ml[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int e = t + UT * q, i = e / KB, j = e % KB;
        const bool in = i < k && j < k;
        gl[q] = in ? gram[i * k + j] : (HT)0;
        ml[q] = in ? minv[i * k + j] : (HT)0;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rb + j * (UT / KB);
        const int64_t prow = tile * TR + r0 + r;
        wl[j] = cc < k ? Wt[(g0 + r) * k + cc] : (HT)0;
        uv[j] = prow < a.rows && cc < k ? Ud[prow * k + cc] : (HT)0;
        swv[j] = wgv[j] = 0;
    }
    if (cc < k) {
        for (int64_t w = w_lo; w <= w_hi; ++w) {
            const HT* pw = part + ((slot_mul * w + slot_base) * TR + r0 + rb) * a.kp + cc;
#pragma unroll
            for (int j = 0; j < NJ; ++j) swv[j] += pw[j * (UT / KB) * a.kp];
        }
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
        if (t + UT * q < KB * KB) {
            Gs[t + UT * q] = gl[q];
            Ms[t + UT * q] = ml[q];
        }
#pragma unroll
    for (int j = 0; j < NJ; ++j) Ws[t + UT * j] = wl[j];
    __syncthreads();
#pragma unroll 2
    for (int b = 0; b < KB; b += 4) {
        const HT g0 = Gs[b * KB + cc], g1 = Gs[(b + 1) * KB + cc], g2 = Gs[(b + 2) * KB + cc],
                 g3 = Gs[(b + 3) * KB + cc];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const hvec4 wv = *(const hvec4*)&Ws[(rb + j * (UT / KB)) * KB + b];
            HT v = wgv[j];
            v += wv[0] * g0;
            v += wv[1] * g1;
            v += wv[2] * g2;
            v += wv[3] * g3;
            wgv[j] = v;
        }
    }
    double tr = 0.0, kkt = 0.0;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rb + j * (UT / KB);
        const int64_t prow = tile * TR + r0 + r;
        HT av = 0;
        if (prow < a.rows && cc < k) {
            const HT w = Ws[r * KB + cc];
            const int64_t idx = prow * k + cc;
            HT sw = swv[j];
            if (a.fp8) sw = sw / (HT)a.panel_scale[(uint32_t)prow / (uint32_t)a.panel_rows] + (HT)a.diag[prow] * w;
            const HT g = (HT)4 * (wgv[j] - sw);
            tr += (double)w * (double)sw;
            const HT pg = w > (HT)0 ? g : (g < (HT)0 ? g : (HT)0);
            kkt += (double)pg * (double)pg;
            if (!(g == g) || g - g != (HT)0) ++bad;
            if (Go) Go[idx] = g;
            av = __builtin_elementwise_fma((HT)2, sw, rho * (w - uv[j]));   // one rounding order: ADMM's dual keeps it
        }
        As[r * KB + cc] = av;
    }
    __syncthreads();
    HT hv[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) hv[j] = 0;
#pragma unroll 2
    for (int b = 0; b < KB; b += 4) {
        const HT m0 = Ms[b * KB + cc], m1 = Ms[(b + 1) * KB + cc], m2 = Ms[(b + 2) * KB + cc],
                 m3 = Ms[(b + 3) * KB + cc];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const hvec4 av4 = *(const hvec4*)&As[(rb + j * (UT / KB)) * KB + b];
            HT v = hv[j];
            v += av4[0] * m0;
            v += av4[1] * m1;
            v += av4[2] * m2;
            v += av4[3] * m3;
            hv[j] = v;
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rb + j * (UT / KB);
        const int64_t prow = tile * TR + r0 + r;
        HT wn = 0;
        if (prow < a.rows && cc < k) {
            const int64_t idx = prow * k + cc;
            const HT h = hv[j], u = uv[j];
            wn = h + u > (HT)0 ? h + u : (HT)0;
            Ud[idx] = u + h - wn;
            Wn[(g0 + r) * k + cc] = wn;
        }
        Wns[r * KB + cc] = wn;
    }
    __syncthreads();
    if constexpr (sizeof(HT) == 4)
        if (a.img1 && g0 < a.n_chunks * KC)
            write_image_slice<KB, UT>(a.img_kind, Wns, Ws, (int)min(a.rows - tile * TR - r0, (int64_t)SR), g0, a.img1, a.img2);
    double* tg = a.tile_gram + slice * (int64_t)k * k;
    if (KB >= 32) {
        // entries (ia0 + q, ib), q < NQ, as in the update kernel: the same FP64
        // sums over the slice rows, consecutive ia read as vectors
        constexpr int NQ = KB >= 32 ? (KB * KB) / UT : 4;
        constexpr int VQ = NQ < 4 ? NQ : 4;
        static_assert(NQ % VQ == 0, "vector reads of the Gram rows");
        typedef HT hvecq __attribute__((ext_vector_type(VQ)));
        const int ib = t % KB, ia0 = (t / KB) * NQ;
        double sq[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) sq[q] = 0.0;
#pragma unroll 4
        for (int r = 0; r < SR; ++r) {
            const double hb = (double)Wns[r * KB + ib];
#pragma unroll
            for (int q = 0; q < NQ; q += VQ) {
                const hvecq wv = *(const hvecq*)&Wns[r * KB + ia0 + q];
#pragma unroll
                for (int e = 0; e < VQ; ++e) sq[q + e] += (double)wv[e] * hb;
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (ia0 + q < k && ib < k) tg[(ia0 + q) * k + ib] = sq[q];
    } else {
        for (int e = t; e < k * k; e += UT) {
            const int ia = e / k, ib = e - ia * k;
            double s = 0.0;
#pragma unroll 8
            for (int r = 0; r < SR; ++r) s += (double)Wns[r * KB + ia] * (double)Wns[r * KB + ib];
            tg[e] = s;
        }
    }
    double nbad = (double)bad;
    block_sum3(tr, kkt, nbad, red);
    if (t == 0) {
        a.tile_tr[slice] = tr;
        a.tile_kkt[slice] = kkt;
        a.tile_bad[slice] = (int32_t)nbad;
    }
}

hipError_t launch_admm(const UpdateArgs& a, const double* gram64, int h_f64, const PlanView& p, hipStream_t stream) {
    if (!p.full || a.k > KMAX || (h_f64 && a.k > 32)) return hipErrorInvalidValue;
    if (!gram64) {
        // the stream's launch formed the inverse
    } else if (h_f64) launch_minv(gram64, (int)a.k, a.rho, (double*)a.minv, stream);
    else launch_minv(gram64, (int)a.k, a.rho, (float*)a.minv, stream);
    const int64_t tiles = a.rows_pad / TR;
    const dim3 grid(tiles * SUBT);
#define UPDATE(HT, KB) \
    hipLaunchKernelGGL((admm_update_kernel<HT, KB>), grid, dim3((update_threads<HT, KB>())), 0, stream, a, p)
    if (h_f64) {
        if (a.k <= 8) UPDATE(double, 8);
        else if (a.k <= 16) UPDATE(double, 16);
        else UPDATE(double, 32);
    } else {
        if (a.k <= 16) UPDATE(float, 16);
        else if (a.k <= 32) UPDATE(float, 32);
        else UPDATE(float, 64);
    }
#undef UPDATE
    return hipGetLastError();
}

// Per-tile FP64 Gram partials of H rows [row0 + tile*TR, +TR) (rows >= row0+rows are zero).
template <typename HT>
__global__ __launch_bounds__(256) void tile_gram_kernel(const HT* __restrict__ H, int64_t row0, int64_t rows,
                                                        int k, double* __restrict__ out) {
    const int64_t slice = blockIdx.x;
    const int t = threadIdx.x;
    double* dst = out + slice * (int64_t)k * k;
    for (int e = t; e < k * k; e += 256) {
        const int ia = e / k, ib = e - ia * k;
        double s = 0.0;
        for (int r = 0; r < SR; ++r) {
            const int64_t prow = slice * SR + r;
            if (prow < rows) s += (double)H[(row0 + prow) * k + ia] * (double)H[(row0 + prow) * k + ib];
        }
        dst[e] = s;
    }
}

hipError_t launch_tile_gram(const void* H, int h_f64, int64_t row0, int64_t rows, int64_t tiles, int64_t k,
                            double* tile_gram, hipStream_t stream) {
    if (h_f64)
        hipLaunchKernelGGL(tile_gram_kernel<double>, dim3(tiles * SUBT), dim3(256), 0, stream, (const double*)H,
                           row0, rows, (int)k, tile_gram);
    else
        hipLaunchKernelGGL(tile_gram_kernel<float>, dim3(tiles * SUBT), dim3(256), 0, stream, (const float*)H,
                           row0, rows, (int)k, tile_gram);
    return hipGetLastError();
}

// FP64 Gram of the rows of [0, n) outside [skip_lo, skip_hi): one work-group per
// entry, fixed order.  (For a row panel: the rows that stay fixed.)
template <typename HT>
__global__ __launch_bounds__(256) void gram_rows_kernel(const HT* __restrict__ H, int64_t n, int64_t skip_lo,
                                                        int64_t skip_hi, int k, double* __restrict__ out) {
    __shared__ double red[8];
    const int e = blockIdx.x;
    const int ia = e / k, ib = e - ia * k;
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += 256)
        if (r < skip_lo || r >= skip_hi) s += (double)H[r * k + ia] * (double)H[r * k + ib];
    s = block_sum(s, red);
    if (threadIdx.x == 0) out[e] = s;
}

hipError_t launch_gram_rows(const void* H, int h_f64, int64_t n, int64_t skip_lo, int64_t skip_hi, int64_t k,
                            double* out, hipStream_t stream) {
    if (h_f64)
        hipLaunchKernelGGL(gram_rows_kernel<double>, dim3(k * k), dim3(256), 0, stream, (const double*)H, n, skip_lo,
                           skip_hi, (int)k, out);
    else
        hipLaunchKernelGGL(gram_rows_kernel<float>, dim3(k * k), dim3(256), 0, stream, (const float*)H, n, skip_lo,
                           skip_hi, (int)k, out);
    return hipGetLastError();
}

template <typename HT>
__global__ __launch_bounds__(256) void finalize_kernel(int64_t tiles, int k, const double* __restrict__ tile_gram,
                                                       const double* __restrict__ tile_tr,
                                                       const double* __restrict__ tile_kkt,
                                                       const int32_t* __restrict__ tile_bad,
                                                       const double* __restrict__ gram_fixed,
                                                       const double* __restrict__ gram_cur,
                                                       double* __restrict__ gram_next, HT* __restrict__ gram_eff,
                                                       double* __restrict__ stats) {
    __shared__ double red[8];
    const int kk = k * k;
    const int ngram = (kk + 3) / 4;          // one wave per Gram entry
    const int t = threadIdx.x;
    if ((int)blockIdx.x < ngram) {
        const int e = blockIdx.x * 4 + (t >> 6);
        const int lane = t & 63;
        if (e >= kk) return;
        // lane l sums tiles l, l+64, ...; then a fixed-order butterfly
        double s = 0.0;
        for (int64_t i = lane; i < tiles; i += 64) s += tile_gram[i * kk + e];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if (lane == 0) {
            if (gram_fixed) s += gram_fixed[e];
            gram_next[e] = s;
            gram_eff[e] = (HT)s;
            gram_eff[kk + e] = (HT)s;
            gram_eff[2 * kk + e] = (HT)s;
        }
        return;
    }
    double tr = 0.0, kkt = 0.0, bad = 0.0, gn = 0.0;
    for (int64_t i = t; i < tiles; i += 256) {
        tr += tile_tr[i];
        kkt += tile_kkt[i];
        bad += (double)tile_bad[i];
    }
    if (gram_cur)
        for (int e = t; e < kk; e += 256) gn += gram_cur[e] * gram_cur[e];
    tr = block_sum(tr, red);
    kkt = block_sum(kkt, red);
    bad = block_sum(bad, red);
    gn = block_sum(gn, red);
    if (t == 0) {
        stats[0] = tr;
        stats[1] = kkt;
        stats[2] = bad;
        stats[3] = gn;
    }
}

hipError_t launch_finalize(int64_t tiles, int64_t k, const double* tile_gram, const double* tile_tr,
                           const double* tile_kkt, const int32_t* tile_bad, const double* gram_fixed,
                           const double* gram_cur64, double* gram_next64, void* gram_eff, int h_f64,
                           double* stats, hipStream_t stream) {
    const int ngram = (int)((k * k + 3) / 4);
    dim3 grid(ngram + 1), block(256);
    if (h_f64)
        hipLaunchKernelGGL(finalize_kernel<double>, grid, block, 0, stream, tiles, (int)k, tile_gram, tile_tr,
                           tile_kkt, tile_bad, gram_fixed, gram_cur64, gram_next64, (double*)gram_eff, stats);
    else
        hipLaunchKernelGGL(finalize_kernel<float>, grid, block, 0, stream, tiles, (int)k, tile_gram, tile_tr,
                           tile_kkt, tile_bad, gram_fixed, gram_cur64, gram_next64, (float*)gram_eff, stats);
    return hipGetLastError();
}

// Block step: Gram_J, Gram_I and their sum from the slice partials of H_t.  A
// work-group sums GS_E consecutive entries, 64 phases over the slices each (one
// thread per entry walked the sampled tiles' slices one after another, I and J
// in turn: 40 us at n = 20000, k = 32; this takes 7.5 us).
constexpr int GS_E = 16, GS_P = 64;

template <typename HT>
__global__ __launch_bounds__(GS_E * GS_P) void gram_select_kernel(int k, const double* __restrict__ tile_gram,
                                                                 PlanView p, HT* __restrict__ out) {
    __shared__ double red[2][GS_P][GS_E + 1];
    const int kk = k * k, le = threadIdx.x % GS_E, ph = threadIdx.x / GS_E;
    const int e = blockIdx.x * GS_E + le;
    double gi = 0.0, gj = 0.0;
    if (e < kk) {
#pragma unroll 4
        for (int s = ph; s < p.n_tiles * SUBT; s += GS_P) {
            const int32_t act = p.tile_active[s / SUBT];
            const int32_t cls = act >= 0 ? p.active_class[act] : -1;   // 0: rows in I only, 1: in J only, 2: in both
            const double g = cls >= 0 ? tile_gram[(int64_t)s * kk + e] : 0.0;
            gi += cls == 0 || cls == 2 ? g : 0.0;
            gj += cls == 1 || cls == 2 ? g : 0.0;
        }
    }
    red[0][ph][le] = gi;
    red[1][ph][le] = gj;
    __syncthreads();
    for (int h = GS_P / 2; h > 0; h >>= 1) {
        if (ph < h) {
            red[0][ph][le] += red[0][ph + h][le];
            red[1][ph][le] += red[1][ph + h][le];
        }
        __syncthreads();
    }
    if (ph == 0 && e < kk) {
        gi = red[0][0][le];
        gj = red[1][0][le];
        out[e] = (HT)gj;
        out[kk + e] = (HT)gi;
        out[2 * kk + e] = (HT)(gi + gj);
    }
}

hipError_t launch_gram_select(int64_t k, const double* tile_gram, const PlanView& plan, void* gram_eff, int h_f64,
                              hipStream_t stream) {
    dim3 grid((k * k + GS_E - 1) / GS_E), block(GS_E * GS_P);
    if (h_f64)
        hipLaunchKernelGGL(gram_select_kernel<double>, grid, block, 0, stream, (int)k, tile_gram, plan, (double*)gram_eff);
    else
        hipLaunchKernelGGL(gram_select_kernel<float>, grid, block, 0, stream, (int)k, tile_gram, plan, (float*)gram_eff);
    return hipGetLastError();
}

// H0_ij = u_ij * scale, u_ij the 24-bit uniform of counter i*k + j.
__global__ void init_h_kernel(float* __restrict__ H, int64_t count, uint64_t seed, float scale) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        H[i] = (float)uniform24(seed, (uint64_t)i) * scale;
}

hipError_t launch_init_H(float* H, int64_t n, int64_t k, uint64_t seed, float scale, hipStream_t stream) {
    const int64_t count = n * k;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(init_h_kernel, dim3(blocks), dim3(256), 0, stream, H, count, seed, scale);
    return hipGetLastError();
}

// Zero fill of `bytes` bytes at any alignment: 16-byte vector stores over the
// aligned middle, single bytes for the unaligned ends.  Used instead of a
// memset node so that work a caller records into a HIP graph replays the
// clear as a kernel.
__global__ void zero_kernel(unsigned char* __restrict__ p, int64_t bytes) {
    const int64_t mis = (int64_t)((16 - ((uintptr_t)p & 15)) & 15);
    const int64_t head = mis < bytes ? mis : bytes;
    const int64_t nvec = (bytes - head) / 16;
    const int64_t tail0 = head + nvec * 16;
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    u32x4* v = (u32x4*)(p + head);
    for (int64_t i = i0; i < nvec; i += stride) v[i] = u32x4{0u, 0u, 0u, 0u};
    if (i0 < head) p[i0] = 0;
    if (i0 < bytes - tail0) p[tail0 + i0] = 0;
}

hipError_t launch_zero(void* p, int64_t bytes, hipStream_t stream) {
    if (bytes <= 0) return hipSuccess;
    if (!p) return hipErrorInvalidValue;
    int64_t blocks = (bytes / 16 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(256), 0, stream, (unsigned char*)p, bytes);
    return hipGetLastError();
}

template <typename A, typename B>
__global__ void copy_kernel(const A* __restrict__ s, B* __restrict__ d, int64_t m) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = (B)s[i];
}

hipError_t launch_copy_h(const void* src, int src_f64, void* dst, int dst_f64, int64_t count, hipStream_t stream) {
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) return hipSuccess;
    if (src_f64 && dst_f64)
        hipLaunchKernelGGL((copy_kernel<double, double>), dim3(blocks), dim3(256), 0, stream, (const double*)src, (double*)dst, count);
    else if (src_f64)
        hipLaunchKernelGGL((copy_kernel<double, float>), dim3(blocks), dim3(256), 0, stream, (const double*)src, (float*)dst, count);
    else if (dst_f64)
        hipLaunchKernelGGL((copy_kernel<float, double>), dim3(blocks), dim3(256), 0, stream, (const float*)src, (double*)dst, count);
    else
        hipLaunchKernelGGL((copy_kernel<float, float>), dim3(blocks), dim3(256), 0, stream, (const float*)src, (float*)dst, count);
    return hipGetLastError();
}

// Theta0 = softplus^-1(max(H0, 1e-12)); H0 <- softplus(Theta0).
template <typename HT>
__global__ void softplus_init_kernel(HT* __restrict__ H, HT* __restrict__ Th, int64_t m) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        double h = (double)H[i];
        h = h > 1e-12 ? h : 1e-12;
        const double th = h > 20.0 ? h + log(-expm1(-h)) : log(expm1(h));
        Th[i] = (HT)th;
        H[i] = softplus_f((HT)th);
    }
}

hipError_t launch_softplus_init(void* H, void* Theta, int h_f64, int64_t count, hipStream_t stream) {
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) return hipSuccess;
    if (h_f64)
        hipLaunchKernelGGL(softplus_init_kernel<double>, dim3(blocks), dim3(256), 0, stream, (double*)H, (double*)Theta, count);
    else
        hipLaunchKernelGGL(softplus_init_kernel<float>, dim3(blocks), dim3(256), 0, stream, (float*)H, (float*)Theta, count);
    return hipGetLastError();
}

// FP64 sum of m values (single work-group, fixed order).
template <typename T>
__global__ __launch_bounds__(1024) void sum_kernel(const T* __restrict__ x, int64_t m, double* out) {
    __shared__ double red[16];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < m; i += 1024) s += (double)x[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = 0.0;
        for (int i = 0; i < 16; ++i) r += red[i];
        *out = r;
    }
}

hipError_t launch_sum(const void* x, int x_f64, int64_t m, double* out, hipStream_t stream) {
    if (x_f64) hipLaunchKernelGGL(sum_kernel<double>, dim3(1), dim3(1024), 0, stream, (const double*)x, m, out);
    else hipLaunchKernelGGL(sum_kernel<float>, dim3(1), dim3(1024), 0, stream, (const float*)x, m, out);
    return hipGetLastError();
}

// Piecewise reset: G_i <- max(c g_i^2, c median(g^2)).
template <typename HT>
__global__ void piecewise_kernel(HT* __restrict__ G, const HT* __restrict__ g, int64_t m, double c,
                                 const double* __restrict__ med) {
    const HT floor_v = (HT)(c * (double)med[0]);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const HT v = (HT)c * g[i] * g[i];
        G[i] = v > floor_v ? v : floor_v;
    }
}

// Objective pass (FP64 S.H partials of a full plan): per slice of SR rows the
// partial of sum_r h_r . (S H)_r and the FP64 Gram of the slice's H rows, a 4 x 4
// block of it per thread from rows in LDS (threads left over at small k take
// rows of their own; their sums are added in a fixed order).  One work-group per
// 256 rows with an entry of the Gram per thread, read from memory, took 711 us
// at n = 20000, k = 64; with the partials of an element one after another 44 us;
// this takes 30 us.
template <typename HT>
__global__ __launch_bounds__(256) void objective_tiles_kernel(UpdateArgs a, PlanView p) {
    constexpr int LD = KMAX + 2;
    __shared__ __align__(16) double Hs[SR * LD];
    static_assert(sizeof(Hs) >= 256 * 16 * sizeof(double), "the reduction reuses the row buffer");
    __shared__ double red[8];
    typedef double dvec2 __attribute__((ext_vector_type(2)));
    const int t = threadIdx.x;
    const int64_t slice = blockIdx.x, tile = slice / SUBT;
    const int r0 = (int)(slice % SUBT) * SR;
    const int k = (int)a.k;
    const int64_t g0 = a.row0 + tile * TR + r0;
    const HT* H = (const HT*)a.H;
    const double* part = (const double*)a.part;
    const int kr = (k + 3) / 4 * 4;
    for (int f = t; f < SR * kr; f += 256) {
        const int r = f / kr, c = f - r * kr;
        const bool in = c < k && tile * TR + r0 + r < a.rows;
        Hs[r * LD + c] = in ? (double)H[(g0 + r) * k + c] : 0.0;
    }
    __syncthreads();
    const int64_t U = (int64_t)p.n_tiles * p.n_chunks;
    const int64_t Pe = U < p.P ? U : p.P;
    const int64_t w_lo = wg_owner(tile * p.n_chunks, U, Pe);
    const int64_t w_hi = wg_owner((tile + 1) * p.n_chunks - 1, U, Pe);
    double tr = 0.0;
    constexpr int NE = 8;                                  // elements of a thread whose loads are in flight together
    for (int f0 = t; f0 < SR * k; f0 += 256 * NE) {
        int r[NE], c[NE];
        double sh[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int f = min(f0 + 256 * e, SR * k - 1);
            r[e] = f / k;
            c[e] = f - r[e] * k;
            sh[e] = 0.0;
        }
#pragma unroll 2
        for (int64_t w = w_lo; w <= w_hi; ++w) {
            const double* pw = part + ((w + tile) * TR + r0) * a.kp;
#pragma unroll
            for (int e = 0; e < NE; ++e) sh[e] += pw[r[e] * a.kp + c[e]];
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int64_t prow = tile * TR + r0 + r[e];
            if (f0 + 256 * e >= SR * k || prow >= a.rows) continue;
            const double h = Hs[r[e] * LD + c[e]];
            double v = sh[e];
            if (a.fp8) v = v / (double)a.panel_scale[(uint32_t)prow / (uint32_t)a.panel_rows] + (double)a.diag[prow] * h;
            tr += h * v;
        }
    }
    const int nk = kr / 4, nt = nk * nk, groups = 256 / nt;
    const int grp = t / nt, blk = t - grp * nt;
    const int ca = 4 * (blk / nk), cb = 4 * (blk % nk);
    double acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0;
    if (grp < groups)
        for (int r = grp; r < SR; r += groups) {
            const dvec2 a0 = *(const dvec2*)&Hs[r * LD + ca], a1 = *(const dvec2*)&Hs[r * LD + ca + 2];
            const dvec2 b0 = *(const dvec2*)&Hs[r * LD + cb], b1 = *(const dvec2*)&Hs[r * LD + cb + 2];
            const double av[4] = {a0[0], a0[1], a1[0], a1[1]}, bv[4] = {b0[0], b0[1], b1[0], b1[1]};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[4 * i + j] += av[i] * bv[j];
        }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) Hs[e * 256 + t] = acc[e];
    __syncthreads();
    double* tg = a.tile_gram + slice * (int64_t)k * k;
    for (int e = t; e < k * k; e += 256) {
        const int i = e / k, j = e - i * k;
        const int src = (4 * (i & 3) + (j & 3)) * 256 + (i >> 2) * nk + (j >> 2);
        double s = 0.0;
        for (int g = 0; g < groups; ++g) s += Hs[src + g * nt];
        tg[e] = s;
    }
    const double str = block_sum(tr, red);
    if (t == 0) {
        a.tile_tr[slice] = str;
        a.tile_kkt[slice] = 0.0;
        a.tile_bad[slice] = 0;
    }
}

hipError_t launch_objective_tiles(const UpdateArgs& a, int h_f64, const PlanView& p, hipStream_t stream) {
    const dim3 grid(a.rows_pad / TR * SUBT), block(256);
    if (h_f64) hipLaunchKernelGGL(objective_tiles_kernel<double>, grid, block, 0, stream, a, p);
    else hipLaunchKernelGGL(objective_tiles_kernel<float>, grid, block, 0, stream, a, p);
    return hipGetLastError();
}

hipError_t launch_piecewise_apply(void* G, const void* g, int h_f64, int64_t m, double c, const double* med,
                                  hipStream_t stream) {
    int64_t blocks = (m + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (h_f64)
        hipLaunchKernelGGL(piecewise_kernel<double>, dim3(blocks), dim3(256), 0, stream, (double*)G, (const double*)g, m, c, med);
    else
        hipLaunchKernelGGL(piecewise_kernel<float>, dim3(blocks), dim3(256), 0, stream, (float*)G, (const float*)g, m, c, med);
    return hipGetLastError();
}

}  // namespace symnmf
