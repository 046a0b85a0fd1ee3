// S.H row-panel stream: the dominant O(n^2 k) product of every iteration
// (paper section "Computational Methodology": S x H dominates each step).
//
// Work split: see PlanView in common.h.  Each persistent work-group walks its
// unit range; per unit (256-row tile x 256-column chunk) it streams the tile of
// S from HBM straight into MFMA A-operand registers - the tiled storage puts
// every wave's 64 rows of the tile in one contiguous run - while the H rows of
// the chunk sit in LDS in B-operand order.  Once per step a prep kernel writes
// H as "images", one per chunk, already in that LDS order (and, for BF16/FP8
// S, already split into bf16 planes), so staging a chunk is a plain 16-byte
// copy; the image of the next unit is fetched during the current unit and S
// loads run three sub-steps ahead across unit boundaries, so the S stream never
// drains.  Each wave owns 64 rows (4 MFMA row groups) so every B fragment read
// from LDS feeds 4 MFMAs.
//
// MFMA operand layouts used (CDNA3/CDNA4, 64-lane wave, lane l, r = l%16,
// g = l/16):
//   v_mfma_f32_16x16x4_f32 : A[r][g], B[g][r], D[4g+v][r] (v = 0..3)
//   v_mfma_f32_16x16x32_bf16: A[r][8g..8g+7], B[8g..8g+7][r], D as above
// The reduction index of one MFMA may be any permutation of the columns as
// long as A and B agree; each kernel uses the one in which a lane's 16 bytes
// of S are consecutive columns.
#include <algorithm>
#include <type_traits>

#include "admm_inverse.h"
#include "image.h"

namespace symnmf {

__device__ inline void plan_bounds(const PlanView& p, int64_t& U, int32_t& na) {
    if (p.full) {
        na = p.tall ? (int32_t)tall_pairs(p.n_tiles) : p.n_tiles;
        U = (int64_t)na * p.n_chunks;
    } else {
        na = p.hdr[0];
        U = (int64_t)(uint32_t)p.hdr[1] | ((int64_t)p.hdr[2] << 32);
    }
}
__device__ inline int64_t unit_off(const PlanView& p, int32_t a) {
    return p.full ? (int64_t)a * p.n_chunks : (int64_t)p.unit_offset[a];
}
__device__ inline int32_t find_active(const PlanView& p, int64_t u, int32_t na) {
    if (p.full) return (int32_t)(u / p.n_chunks);
    int lo = 0, hi = na - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if ((int64_t)p.unit_offset[mid] <= u) lo = mid; else hi = mid - 1;
    }
    return lo;
}
__device__ inline void unit_chunk(const PlanView& p, int32_t a, int64_t j, int32_t& chunk, float& w) {
    if (p.full) { chunk = (int32_t)j; w = 1.0f; return; }
    int c = p.active_class[a];
    chunk = p.class_chunks[c * p.n_chunks + j];
    w = (float)p.class_weight[c * p.n_chunks + j];
}
__device__ inline int32_t tile_of(const PlanView& p, int32_t a) { return p.full ? a : p.active_tile[a]; }

// unit u -> (active tile, chunk, weight), a = active tile holding u or a hint below it
__device__ inline void unit_decode(const PlanView& p, int64_t u, int32_t& a, int32_t& chunk, float& w) {
    while (u >= unit_off(p, a + 1)) ++a;
    unit_chunk(p, a, u - unit_off(p, a), chunk, w);
}

// ---------------------------------------------------------------------------
// Generic kernel: any storage type, FP64 H and accumulation, k <= KB.
// One thread per row of the tile.  Used for FP64 H: parity runs at ranks other
// than 16 and 32, and the objective of an FP64 factor.
// ---------------------------------------------------------------------------
template <typename ST>
__device__ inline int64_t s_index(int64_t r, int64_t c, int64_t ld, int64_t n_chunks) {
    if (sizeof(ST) == 8) return r * ld + c;
    return tiled_offset(r, c, n_chunks, (int)(16 / sizeof(ST)));
}

template <typename ST, int KB>
__global__ __launch_bounds__(256) void stream_generic(const ST* __restrict__ S, int64_t ld,
                                                      const double* __restrict__ H, int k,
                                                      double* __restrict__ part, PlanView p) {
    constexpr int SUB = 32;
    __shared__ double Hs[SUB * KB];
    int64_t U; int32_t na;
    plan_bounds(p, U, na);
    if (U == 0) return;
    const int64_t Pe = U < p.P ? U : p.P;
    const int64_t w = blockIdx.x;
    if (w >= Pe) return;
    int64_t u = wg_start(w, U, Pe);
    const int64_t u1 = wg_start(w + 1, U, Pe);
    int32_t a = find_active(p, u, na);
    const int t = threadIdx.x;
    while (u < u1) {
        const int64_t abase = unit_off(p, a);
        const int64_t run_end = min(u1, unit_off(p, a + 1));
        const int64_t tile = tile_of(p, a);
        double acc[KB];
#pragma unroll
        for (int c = 0; c < KB; ++c) acc[c] = 0;
        const int64_t row = tile * TR + t;
        for (; u < run_end; ++u) {
            int32_t chunk; float wt;
            unit_chunk(p, a, u - abase, chunk, wt);
            for (int sub = 0; sub < KC; sub += SUB) {
                __syncthreads();
                for (int f = t; f < SUB * k; f += 256) {
                    int kk = f / k, c = f - kk * k;
                    Hs[kk * KB + c] = H[((int64_t)chunk * KC + sub + kk) * k + c] * (double)wt;
                }
                __syncthreads();
                const int64_t col0 = (int64_t)chunk * KC + sub;
                for (int kk = 0; kk < SUB; ++kk) {
                    const double s = load_as_f64(S + s_index<ST>(row, col0 + kk, ld, p.n_chunks));
#pragma unroll
                    for (int c = 0; c < KB; ++c)
                        if (c < k) acc[c] += s * Hs[kk * KB + c];
                }
            }
        }
        double* dst = part + ((w + a) * TR + t) * (int64_t)k;
#pragma unroll
        for (int c = 0; c < KB; ++c)
            if (c < k) dst[c] = acc[c];
        ++a;
    }
}

// ---------------------------------------------------------------------------
// FP64 storage (row-major, leading dimension ld), FP64 H and FP64 accumulation
// on the FP64 matrix cores, k = 16 NT.  v_mfma_f64_16x16x4_f64 (lane l,
// r = l % 16, g = l / 16): A[r][g], B[g][r], D[4v+g][r] (v = 0..3: the four
// output rows of a lane are interleaved, unlike the FP32 16x16x4 form).  A wave
// owns 64 rows of the tile (4 row groups of 16); per sub-step of 8 columns a
// lane loads 16 bytes (2 doubles) of its row in each row group, and the two
// MFMAs of an element e reduce over the columns 2g + e of the sub-step, with
// the matching H rows read from the chunk staged in LDS (scaled by the unit's
// weight).  S loads run one sub-step pair ahead.  Units and partials follow
// the plan as in stream_generic.
// ---------------------------------------------------------------------------
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <int NT>
__global__ __launch_bounds__(256, 2) void stream_f64_mfma(const double* __restrict__ S, int64_t ld,
                                                          const double* __restrict__ H,
                                                          double* __restrict__ part, PlanView p) {
    constexpr int K = 16 * NT;
    constexpr int SS = KC / 8;                             // sub-steps of 8 columns per unit
    __shared__ double Hs[KC * K];
    int64_t U; int32_t na;
    plan_bounds(p, U, na);
    if (U == 0) return;
    const int64_t Pe = U < p.P ? U : p.P;
    const int64_t w = blockIdx.x;
    if (w >= Pe) return;
    int64_t u = wg_start(w, U, Pe);
    const int64_t u1 = wg_start(w + 1, U, Pe);
    int32_t a = find_active(p, u, na);
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;
    while (u < u1) {
        const int64_t abase = unit_off(p, a);
        const int64_t run_end = min(u1, unit_off(p, a + 1));
        const int64_t tile = tile_of(p, a);
        doublex4 acc[4][NT];
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = doublex4{0.0, 0.0, 0.0, 0.0};
        const double* rowp[4];
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
            rowp[rg] = S + (tile * TR + 64 * wv + 16 * rg + lr) * ld + 2 * lg;
        for (; u < run_end; ++u) {
            int32_t chunk; float wt;
            unit_chunk(p, a, u - abase, chunk, wt);
            __syncthreads();
            const double* hsrc = H + (int64_t)chunk * KC * K;
            for (int f = t; f < KC * K; f += 256) Hs[f] = hsrc[f] * (double)wt;
            __syncthreads();
            const int64_t col0 = (int64_t)chunk * KC;
            doublex2 cur[2][4], nxt[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) cur[q][rg] = *(const doublex2*)(rowp[rg] + col0 + 8 * q);
            for (int s = 0; s < SS; s += 2) {
                if (s + 2 < SS) {
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg)
                            nxt[q][rg] = *(const doublex2*)(rowp[rg] + col0 + 8 * (s + 2 + q));
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int kk = 8 * (s + q) + 2 * lg + e;
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const double b = Hs[kk * K + 16 * nt + lr];
#pragma unroll
                            for (int rg = 0; rg < 4; ++rg)
                                acc[rg][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[q][rg][e], b, acc[rg][nt],
                                                                                   0, 0, 0);
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) cur[q][rg] = nxt[q][rg];
            }
        }
        double* dst = part + (w + a) * (int64_t)TR * K;
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    dst[(64 * wv + 16 * rg + 4 * v + lg) * K + 16 * nt + lr] = acc[rg][nt][v];
        ++a;
    }
}

// ---------------------------------------------------------------------------
// The objective of an FP32 H at ranks other than 16 and 32: FP64 products and
// FP64 sums on the FP64 matrix cores, from tiled FP32 / BF16 / FP8 S (full
// plans).  Both operands are widened exactly and a product of two FP32 numbers
// is exact in FP64, so the result differs from the thread-per-row form's in the
// order of its FP64 sums only.  (FP32 sums within a chunk were no substitute:
// they put f 1e-9 to 2e-8 of ||S||^2 off at n = 700 to 10000, these 1e-14, and
// f cancels as E gets small.)
// Bound by the FP64 matrix cores: n = 20000, k = 64, FP32 S takes 1.0 ms for the
// whole call (0.7 at the rate of a large FP64 product), 10.5 with a thread per
// row; k = 17 0.55, k = 1 0.33.  A lane's 16 bytes of S are E consecutive
// columns of its row; MFMA e of a sub-step reduces over the columns E g + e of
// the four lane groups g.  H stays FP32 in LDS, rows E apart on disjoint banks
// (LD), so two work-groups share a CU; k is padded to a multiple of 16 there,
// and the partial rows have k entries.
// ---------------------------------------------------------------------------
template <int KIND, int NT>
__global__ __launch_bounds__(256, 2) void stream_f64_tiled(const void* __restrict__ Sv, const float* __restrict__ H,
                                                           int k, double* __restrict__ part, PlanView p) {
    constexpr int K = 16 * NT, E = KIND == 0 ? 4 : (KIND == 1 ? 8 : 16), EB = 16 / E;
    constexpr int NS = KC / (4 * E), LD = K + 16 / E;
    __shared__ float Hs[KC * LD];
    const int64_t U = (int64_t)p.n_tiles * p.n_chunks, Pe = U < p.P ? U : p.P;
    const int64_t w = blockIdx.x;
    if (w >= Pe) return;
    int64_t u = wg_start(w, U, Pe);
    const int64_t u1 = wg_start(w + 1, U, Pe);
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;
    while (u < u1) {
        const int64_t tile = u / p.n_chunks, run_end = min(u1, (tile + 1) * p.n_chunks);
        doublex4 acc[4][NT];
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = doublex4{0.0, 0.0, 0.0, 0.0};
        for (; u < run_end; ++u) {
            const int64_t chunk = u - tile * p.n_chunks;
            const u32x4* sp = (const u32x4*)((const uint8_t*)Sv + u * TILE_ELEMS * EB + (int64_t)wv * (TILE_ELEMS * EB / 4)) + lane;
            u32x4 cur[4], nxt[4];
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) cur[rg] = __builtin_nontemporal_load(sp + rg * 64);
            __syncthreads();
#pragma unroll 16
            for (int f = t; f < KC * K; f += 256) {
                const int r = f / K, c = f % K;
                Hs[r * LD + c] = c < k ? H[(chunk * KC + r) * k + c] : 0.0f;
            }
            __syncthreads();
#pragma unroll 1
            for (int s = 0; s < NS; ++s) {
                // the last sub-step loads itself again, unused
                const int sn = s + 1 < NS ? s + 1 : s;
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) nxt[rg] = __builtin_nontemporal_load(sp + (sn * 4 + rg) * 64);
#pragma unroll
                for (int q = 0; q < E / 4; ++q) {          // elements 4 q .. 4 q + 3 of the vectors
                    float x[4][4];
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const u32x4 r = cur[rg];
                        if (KIND == 0) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) x[rg][e] = __uint_as_float(r[e]);
                        } else if (KIND == 1) {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                x[rg][e] = bf16_bits_to_f32((uint16_t)(r[(2 * q + (e >> 1)) & 3] >> (16 * (e & 1))));
                        } else {
                            const int code = (int)r[q & 3];
                            x[rg][0] = __builtin_amdgcn_cvt_f32_fp8(code, 0);
                            x[rg][1] = __builtin_amdgcn_cvt_f32_fp8(code, 1);
                            x[rg][2] = __builtin_amdgcn_cvt_f32_fp8(code, 2);
                            x[rg][3] = __builtin_amdgcn_cvt_f32_fp8(code, 3);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float* hrow = Hs + (4 * E * s + E * lg + 4 * q + e) * LD + lr;
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const double b = (double)hrow[16 * nt];
#pragma unroll
                            for (int rg = 0; rg < 4; ++rg)
                                acc[rg][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[rg][e], b, acc[rg][nt], 0, 0, 0);
                        }
                        // LDS reads and conversions of later elements stay behind (hoisted: 3 % slower)
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) cur[rg] = nxt[rg];
            }
        }
        double* dst = part + (w + tile) * TR * (int64_t)k + (64 * wv + lg) * k + lr;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (16 * nt + lr < k) {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                    for (int v = 0; v < 4; ++v) dst[(16 * rg + 4 * v) * k + 16 * nt] = acc[rg][nt][v];
            }
    }
}

template <int KIND>
static void launch_f64_tiled_kind(const void* S, const float* H, int64_t k, double* part, const PlanView& p,
                                  hipStream_t stream) {
    const dim3 grid(p.P), block(256);
#define F64_TILED(NT) hipLaunchKernelGGL((stream_f64_tiled<KIND, NT>), grid, block, 0, stream, S, H, (int)k, part, p)
    if (k <= 16) F64_TILED(1);
    else if (k <= 32) F64_TILED(2);
    else if (k <= 48) F64_TILED(3);
    else F64_TILED(4);
#undef F64_TILED
}

hipError_t launch_stream_f64_tiled(const void* S, int32_t stype, const float* H, int64_t k, double* part,
                                   const PlanView& p, hipStream_t stream) {
    if (k < 1 || k > KMAX || !p.full || p.tall) return hipErrorInvalidValue;
    if (stype == SYMNMF_S_FP32) launch_f64_tiled_kind<0>(S, H, k, part, p, stream);
    else if (stype == SYMNMF_S_BF16) launch_f64_tiled_kind<1>(S, H, k, part, p, stream);
    else if (stype == SYMNMF_S_FP8) launch_f64_tiled_kind<2>(S, H, k, part, p, stream);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// One work-group per (chunk, block of CB columns of H): the block's 256 x CB
// values (scaled by wt) are staged in LDS with 16-byte loads, then every
// thread assembles whole 16-byte image vectors (all three bf16 planes at once
// for KIND 1, 2) and writes them in order.  Each 16-column block is a
// contiguous run of every plane of the image.  At k = 64 a work-group takes
// 16 columns (17 KB of LDS, eight work-groups per CU instead of two); below,
// the whole chunk.  The update kernels keep the images of a state's iterate
// current themselves (write_image_slice); this kernel writes those of a new
// state, of a factor handed in, and the chunks of a row panel whose first row
// is no multiple of 64.
template <int KIND, int K>
constexpr int image_cols_per_wg() { return K >= 64 ? 16 : K; }

// H has k <= K columns, rows ldh apart; the image's other columns are zero.
template <int KIND, int K>
__global__ __launch_bounds__(256) void h_image_kernel(const float* __restrict__ H, int k, int ldh, int64_t chunk0,
                                                      float wt, u32x4* __restrict__ img,
                                                      const float* __restrict__ H2 = nullptr) {
    using IS = ImageShape<KIND, K>;
    constexpr int CB = image_cols_per_wg<KIND, K>();
    constexpr int LDH = CB + 1;                           // padded row: column reads spread over banks
    constexpr int EPV = KIND == 0 ? 4 : 8;                // H values per image vector
    constexpr int VP = KC * K / EPV;                      // vectors per plane
    constexpr int VB = VP / (K / CB);                     // ... per plane and column block
    __shared__ float Hs[KC * LDH];
    const int64_t chunk = chunk0 + blockIdx.x;
    const int blk = blockIdx.y;
    if (k == K && ldh == K) {
        const float* src = H + chunk * KC * K + CB * blk;
        for (int q = threadIdx.x; q < KC * CB / 4; q += 256) {
            const int r = q / (CB / 4), c = 4 * (q % (CB / 4));
            const float4 x = *(const float4*)(src + (int64_t)r * K + c);
            float* d = Hs + r * LDH + c;
            d[0] = x.x * wt;
            d[1] = x.y * wt;
            d[2] = x.z * wt;
            d[3] = x.w * wt;
        }
    } else {
        // columns 64 and up of a wide pass are the first ones of H2
        const float* src = (K > 64 && CB * blk >= 64 ? H2 - 64 : H) + chunk * KC * ldh;
        for (int q = threadIdx.x; q < KC * CB; q += 256) {
            const int r = q / CB, c = CB * blk + q % CB;
            Hs[r * LDH + q % CB] = c < k ? src[r * ldh + c] * wt : 0.0f;
        }
    }
    __syncthreads();
    u32x4* out = img + chunk * IS::NV;
    for (int v = blk * VB + threadIdx.x; v < (blk + 1) * VB; v += 256) {
        int kk0, col;
        image_vector_origin<KIND>(v, kk0, col);
        col -= CB * blk;
        if (KIND == 0) {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(uint32_t, Hs[(kk0 + e) * LDH + col]);
            out[v] = o;
        } else {
            uint16_t hi[8], mid[8], lo[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) split3_bf16(Hs[(kk0 + e) * LDH + col], hi[e], mid[e], lo[e]);
            u32x4 a, b, c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = (uint32_t)hi[2 * e] | ((uint32_t)hi[2 * e + 1] << 16);
                b[e] = (uint32_t)mid[2 * e] | ((uint32_t)mid[2 * e + 1] << 16);
                c[e] = (uint32_t)lo[2 * e] | ((uint32_t)lo[2 * e + 1] << 16);
            }
            out[v] = a;
            out[VP + v] = b;
            out[2 * VP + v] = c;
        }
    }
}

int64_t h_image_words(int32_t stype, int64_t k, int64_t n_chunks) {
    const int64_t kw = mfma_width(k);
    const int64_t per = stype == SYMNMF_S_FP32 ? KC * kw : 3 * KC * kw / 2;
    return per * n_chunks;
}

hipError_t launch_h_image(const float* H, int32_t stype, int64_t k, int64_t chunk0, int64_t n_chunks, float wt,
                          uint32_t* img, hipStream_t stream, int64_t ldh) {
    if (ldh == 0) ldh = k;
    if (k < 1 || k > KMAX || n_chunks < 1 || ldh < k || ldh > KMAX) return hipErrorInvalidValue;
    const int64_t kw = mfma_width(k);
    dim3 grid(n_chunks, kw == 64 ? 4 : 1), block(256);
#define IMG(KIND, KK) \
    hipLaunchKernelGGL((h_image_kernel<KIND, KK>), grid, block, 0, stream, H, (int)k, (int)ldh, chunk0, wt, \
                       (u32x4*)img)
    if (stype == SYMNMF_S_FP32) {
        if (kw == 16) IMG(0, 16); else if (kw == 32) IMG(0, 32); else IMG(0, 64);
    } else if (stype == SYMNMF_S_BF16) {
        if (kw == 16) IMG(1, 16); else if (kw == 32) IMG(1, 32); else IMG(1, 64);
    } else if (stype == SYMNMF_S_FP8) {
        if (kw == 16) IMG(2, 16); else if (kw == 32) IMG(2, 32); else IMG(2, 64);
    } else {
        return hipErrorInvalidValue;
    }
#undef IMG
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// MFMA stream kernel.
//
// FP32 S (v_mfma_f32_16x16x4_f32): sub-step s (0..15) covers 16 columns;
//   lane (r, g) holds the float4 S[row][16 s + 4 g .. +3] of row
//   64 wv + 16 rg + r; MFMA number m reduces over columns 16 s + 4 g + m.
// BF16 S (v_mfma_f32_16x16x32_bf16, H = hi + mid + lo in three bf16 planes):
//   sub-step s (0..7) covers 32 columns; lane (r, g) holds S[row][32 s + 8 g
//   .. +7].
// FP8 S: sub-step s (0..3) covers 64 columns; lane (r, g) holds the 16 codes
//   S[row][64 s + 16 g .. +15], widened to two bf16x8 halves h; half h reduces
//   over columns 64 s + 16 g + 8 h + i.  Codes are unscaled (the update kernel
//   applies the panel scale) and the diagonal is stored as 0 (added back from
//   the FP32 diagonal).
// DB: two LDS image buffers (the next image is written while the current one
// is read); PF: the next image is then fetched into registers at the start of
// a unit (otherwise it is copied at the unit boundary).  Without DB the one
// buffer is refilled in QP parts: every (plane, 16-column) block of the image
// holds its sub-steps in order, so once all waves are past the sub-steps of
// part r (a barrier) the next image's part r is written over it (the last part
// at the unit's end); each part is fetched into registers one part ahead.
// ---------------------------------------------------------------------------
// SUM: where a unit's FP32 MFMA sums go at its end.  SUM_RUN: they go on, one
// chain for the tile's run of units.  SUM_F64: into FP64 sums, the partials are
// written as doubles (the objective pass).  SUM_UNIT: into FP32 sums of units
// (MU steps of FP32 S at ranks other than 16, 32 and 64: one chain was 1 to 5 %
// further from 64 bits at n = 13000 to 20000 than a thread per row with its
// slightly shorter runs.  Error of a gradient, k = 20, n = 18000: 6.8e-7 in one
// chain, 6.6e-7 with a thread per row, 2.2e-7 so; 248.9 us a step either way).
constexpr int SUM_RUN = 0, SUM_F64 = 1, SUM_UNIT = 2;
constexpr int RING_F32 = 8;

// TALL (full plans): 8 waves, the two halves stream row tiles 2q and 2q+1 of a
// (tile pair, chunk) unit against one chunk image, halving image traffic per
// byte of S.
template <int KIND, int NT, bool DB, bool PF, int SUM, bool TALL>
__global__ __launch_bounds__(TALL ? 512 : 256, TALL ? 1 : 2) void stream_mfma(const void* __restrict__ Sv,
                                                                             const u32x4* __restrict__ img1,
                                                                             const u32x4* __restrict__ img2,
                                                                             void* __restrict__ part, PlanView plan) {
    // tall kernels only stream full plans: with full fixed at compile time the
    // plan-table lookups (global loads with their waits) drop out of the loop
    PlanView p = plan;
    if (TALL) p.full = 1;
    constexpr int K = 16 * NT;
    constexpr int NTHR = TALL ? 512 : 256;
    using IS = ImageShape<KIND, K>;
    constexpr int NV = IS::NV;
    constexpr int CPT = NV / NTHR;                         // image vectors per thread
    static_assert(NV % NTHR == 0, "image vectors must split evenly over the threads");
    constexpr bool SPLIT = !DB;                            // single buffer, refilled in parts
    constexpr int QP = CPT % 4 == 0 ? 4 : 2;               // parts per image
    constexpr int NSV = NV / ((KIND == 0 ? 1 : 3) * NT);   // vectors per (plane, 16-column) block
    constexpr int HSV = NSV / QP;                          // ... in one part of its sub-steps
    constexpr int CPH = CPT / QP;                          // image vectors per thread and part
    static_assert(!SPLIT || (CPT % QP == 0 && NSV % QP == 0), "image parts must split evenly");
    constexpr int NS = KIND == 0 ? 16 : (KIND == 1 ? 8 : 4);
    constexpr int EB = KIND == 0 ? 4 : (KIND == 1 ? 2 : 1);
    // S prefetch ring and distance (sub-steps): deeper for FP32 S, whose sub-steps
    // are the slowest, to keep more bytes in flight per wave
    constexpr int RING = (KIND <= 1 && NT <= 2 && SUM != SUM_F64) ? RING_F32 : 4, D = RING - 1;
    static_assert(NS % RING == 0, "ring must divide the sub-steps of a unit");
    static_assert(!SPLIT || NS % QP == 0, "image parts must hold whole sub-steps");
    __shared__ u32x4 lds[(DB ? 2 : 1) * NV];
    int64_t U; int32_t na;
    plan_bounds(p, U, na);
    if (U == 0) return;
    const int64_t Pe = U < p.P ? U : p.P;
    const int64_t w = blockIdx.x;
    if (w >= Pe) return;
    const int64_t u0 = wg_start(w, U, Pe);
    const int64_t u1 = wg_start(w + 1, U, Pe);
    const int lane = threadIdx.x & 63, wv = (threadIdx.x >> 6) & 3;
    const int half = TALL ? (int)(threadIdx.x >> 8) : 0;   // tile of the pair (tall)
    const int lr = lane & 15, lg = lane >> 4;
    const int tid = threadIdx.x;

    // this wave's contiguous run of a unit's tile, in 16-byte vectors, plus the
    // lane (tall: the odd last pair has no second tile; that half re-reads the
    // first tile and writes nothing)
    auto s_run = [&](int32_t aa, int32_t ch) -> const u32x4* {
        const int64_t tile = TALL ? min((int64_t)2 * aa + half, (int64_t)p.n_tiles - 1) : (int64_t)tile_of(p, aa);
        return (const u32x4*)((const uint8_t*)Sv + ((int64_t)tile * p.n_chunks + ch) * TILE_ELEMS * EB +
                              (int64_t)wv * (TILE_ELEMS * EB / 4)) + lane;
    };
    auto image = [&](int32_t ch, float wt) -> const u32x4* {
        return (wt > 1.5f ? img2 : img1) + (int64_t)ch * NV;
    };

    int32_t a = find_active(p, u0, na);
    int32_t chunk;
    float wt;
    unit_decode(p, u0, a, chunk, wt);
    {
        const u32x4* src = image(chunk, wt);
        for (int i = tid; i < NV; i += NTHR) lds[i] = src[i];
    }
    const u32x4* sp = s_run(a, chunk);
    u32x4 ring[RING][4];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) ring[d][rg] = __builtin_nontemporal_load(sp + (d * 4 + rg) * 64);
    __syncthreads();

    floatx4 acc[4][NT];
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    typedef std::conditional_t<SUM == SUM_F64, double, float> sum_t;
    constexpr bool SUMS = SUM != SUM_RUN;
    sum_t sums[SUMS ? 4 : 1][SUMS ? NT : 1][SUMS ? 4 : 1];
    if (SUMS) {
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) sums[SUMS ? rg : 0][SUMS ? nt : 0][SUMS ? v : 0] = 0;
    }

    // vector index of the j-th vector of this thread's share of image part r
    auto part_index = [&](int j, int r) -> int {
        const int q = tid + NTHR * j;
        return (q / HSV) * NSV + r * HSV + q % HSV;
    };
    u32x4 hreg[SPLIT ? CPH : (PF ? CPT : 1)];
    int32_t a_next = a;
    for (int64_t u = u0; u < u1; ++u) {
        const int cur = DB ? (int)((u - u0) & 1) : 0;
        const bool more = u + 1 < u1;
        int32_t chunk_n = chunk;
        float wt_n = 1.0f;
        const u32x4* sp_n = sp;
        if (more) {
            unit_decode(p, u + 1, a_next, chunk_n, wt_n);
            sp_n = s_run(a_next, chunk_n);
        }
        // Every load below is issued whether or not a next unit exists (on the
        // last unit they re-read this unit's own image and S run, in bounds and
        // unused): loads under a branch would leave the compiler's wait counts
        // at the joins of the unrolled loop set for the path without them,
        // draining the S prefetch ring near every unit boundary.
        const u32x4* src_n = image(chunk_n, wt_n);
        if (SPLIT) {
#pragma unroll
            for (int j = 0; j < CPH; ++j) hreg[j] = src_n[part_index(j, 0)];
        } else if (PF) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) hreg[i] = src_n[tid + NTHR * i];
        }
        const u32x4* hb = lds + cur * NV;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (SPLIT && s > 0 && s % (NS / QP) == 0) {
                // all waves are done with part r - 1 of the current image, and
                // the last part written at the previous unit's end is visible;
                // on the last unit the write lands in a consumed part, unread
                __syncthreads();
                const int r = s / (NS / QP);
#pragma unroll
                for (int j = 0; j < CPH; ++j) {
                    lds[part_index(j, r - 1)] = hreg[j];
                    hreg[j] = src_n[part_index(j, r)];
                }
            }
            // keep D sub-steps of S in flight, crossing into the next unit
            const int sd = s + D;
            if (sd < NS) {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    ring[sd % RING][rg] = __builtin_nontemporal_load(sp + (sd * 4 + rg) * 64);
            } else {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    ring[sd % RING][rg] = __builtin_nontemporal_load(sp_n + ((sd - NS) * 4 + rg) * 64);
            }
            // keep the loads here: the scheduler would otherwise sink them
            // towards their use and shorten the prefetch distance
            __builtin_amdgcn_sched_barrier(0);
            if (KIND == 0) {
                floatx4 bv[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    bv[nt] = __builtin_bit_cast(floatx4, hb[((nt * 16 + s) * 4 + lg) * 16 + lr]);
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const floatx4 av = __builtin_bit_cast(floatx4, ring[s % RING][rg]);
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            acc[rg][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m], bv[nt][m], acc[rg][nt], 0, 0, 0);
                    }
            } else {
#pragma unroll
                for (int h = 0; h < (KIND == 2 ? 2 : 1); ++h) {
                    bf16x8 av[4];
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const u32x4 r = ring[s % RING][rg];
                        if (KIND == 2) {
                            const uint32_t w0 = h ? r[2] : r[0];
                            const uint32_t w1 = h ? r[3] : r[1];
                            bf16x2 q0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false);
                            bf16x2 q1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true);
                            bf16x2 q2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false);
                            bf16x2 q3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true);
                            av[rg] = bf16x8{q0[0], q0[1], q1[0], q1[1], q2[0], q2[1], q3[0], q3[1]};
                        } else {
                            av[rg] = __builtin_bit_cast(bf16x8, r);
                        }
                    }
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) {
                        bf16x8 bv[NT];
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const int v16 = KIND == 2 ? ((((nt * 4 + s) * 2 + h) * 4 + lg) * 16 + lr)
                                                      : (((nt * 8 + s) * 4 + lg) * 16 + lr);
                            bv[nt] = __builtin_bit_cast(bf16x8, hb[pl * (IS::PLANE / 8) + v16]);
                        }
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
                                acc[rg][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[rg], bv[nt], acc[rg][nt],
                                                                                      0, 0, 0);
                    }
                }
            }
        }
        if (SUMS) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) sums[SUMS ? rg : 0][SUMS ? nt : 0][SUMS ? v : 0] += (sum_t)acc[rg][nt][v];
                    acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        }
        // end of this tile's run: write the partial and start the next tile
        if (!more || a_next != a) {
            const int64_t slot = TALL ? 2 * (w + a) + half : (w + a);
            const bool store = !TALL || 2 * (int64_t)a + half < p.n_tiles;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (!store) continue;
                        const int64_t o = slot * (int64_t)TR * K + (64 * wv + 16 * rg + 4 * lg + v) * K + 16 * nt + lr;
                        if (SUMS) {
                            ((sum_t*)part)[o] = sums[SUMS ? rg : 0][SUMS ? nt : 0][SUMS ? v : 0];
                            sums[SUMS ? rg : 0][SUMS ? nt : 0][SUMS ? v : 0] = 0;
                        } else {
                            ((float*)part)[o] = acc[rg][nt][v];
                        }
                    }
                    acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        }
        if (more && SPLIT) {
            // all waves are done with the last part; the other parts of the
            // next image are visible now, the last one becomes visible at the
            // next unit's first part barrier
            __syncthreads();
#pragma unroll
            for (int j = 0; j < CPH; ++j) lds[part_index(j, QP - 1)] = hreg[j];
            a = a_next;
            chunk = chunk_n;
            sp = sp_n;
        } else if (more) {
            u32x4* dstb = lds + (cur ^ 1) * NV;
            if (PF) {
#pragma unroll
                for (int i = 0; i < CPT; ++i) dstb[tid + NTHR * i] = hreg[i];
            } else {
                const u32x4* src = image(chunk_n, wt_n);
                for (int i = tid; i < NV; i += NTHR) dstb[i] = src[i];
            }
            __syncthreads();
            a = a_next;
            chunk = chunk_n;
            sp = sp_n;
        }
    }
}

// ---------------------------------------------------------------------------
// Full steps of a few units.  A unit of the kernel above keeps a CU's matrix
// cores busy for 7 (BF16) to 14 us (FP32, k = 32), so a step with fewer units
// than a few per CU takes as long as its longest run of units, most CUs idle.
// Here a work-group takes 64 rows of a tile and its four waves a quarter of
// the chunk's columns each (whole sub-steps), so a unit is spread over four
// CUs and sixteen waves; each wave reads its S and its part of the image (from
// L2) straight into registers, one unit ahead, and the four waves' sums meet in
// LDS once per tile.  The partial of work-group w for tile a goes to slot
// w + a as usual, written by the four work-groups 4 w .. 4 w + 3.
// The inverse of an ADMM step (which runs here up to 1024 instruments), that
// nothing waits for before the update, is formed by a work-group of its own
// beside the others.  A step so / with a launch for it between the stream and
// the update, n = 512, FP32: k = 16 18.1 / 22.7 us, k = 32 24.6 / 29.9, k = 64
// 54.4 / 62.8.
// ---------------------------------------------------------------------------
template <int KIND, int NT>
__global__ __launch_bounds__(256, NT == 4 ? 1 : 2) void stream_quarter(const void* __restrict__ Sv,
                                                                      const u32x4* __restrict__ img,
                                                                      float* __restrict__ part, PlanView p,
                                                                      AdmmInverse inv) {
    constexpr int K = 16 * NT;
    using IS = ImageShape<KIND, K>;
    constexpr int EB = KIND == 0 ? 4 : (KIND == 1 ? 2 : 1);
    constexpr int NS = KIND == 0 ? 16 : (KIND == 1 ? 8 : 4);
    constexpr int QS = NS / 4;                             // sub-steps of a wave
    constexpr int NH = KIND == 2 ? 2 : 1, NP = KIND == 0 ? 1 : 3;
    constexpr int NB = QS * NH * NP * NT;                  // image vectors of a lane
    __shared__ __align__(16) float red[4][64 * K];
    const int64_t U = (int64_t)p.n_tiles * p.n_chunks;
    const int64_t Pe = U < p.P ? U : p.P;
    if (inv.gram && blockIdx.x == 0) {
        static_assert(sizeof(red) >= 4 * KMAX * sizeof(double), "the inverse works in the sums' LDS");
        admm_inverse<float, NT>(inv.gram, inv.k, inv.rho, inv.minv, (double*)red);
        return;
    }
    const int block = (int)blockIdx.x - (inv.gram ? 1 : 0);
    const int64_t w = block >> 2;
    const int sub = block & 3;
    if (w >= Pe) return;
    const int64_t u0 = wg_start(w, U, Pe), u1 = wg_start(w + 1, U, Pe);
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;

    auto load = [&](int64_t tile, int64_t ch, u32x4 (&s)[QS][4], u32x4 (&b)[NB]) {
        const u32x4* sp = (const u32x4*)((const uint8_t*)Sv + (tile * p.n_chunks + ch) * TILE_ELEMS * EB +
                                         (int64_t)sub * (TILE_ELEMS * EB / 4)) + lane;
        const u32x4* hb = img + ch * IS::NV;
#pragma unroll
        for (int q = 0; q < QS; ++q)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) s[q][rg] = __builtin_nontemporal_load(sp + ((wv * QS + q) * 4 + rg) * 64);
#pragma unroll
        for (int q = 0; q < QS; ++q)
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int pl = 0; pl < NP; ++pl)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        b[((q * NH + h) * NP + pl) * NT + nt] =
                            hb[pl * (IS::PLANE / 8) + (((nt * NS + wv * QS + q) * NH + h) * 4 + lg) * 16 + lr];
    };

    floatx4 acc[4][NT];
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    // The units of a tile are not summed in one chain of roundings: at 16 columns,
    // where there is room, every unit by itself and the units' sums apart (ADMM,
    // k = 2, n = 12000, two steps: 3.8e-7 from the FP64 result against 1.4e-6 in
    // one chain; 1 to 6 % slower), at more columns RUN units by themselves, their
    // sums in LDS, where the tile's sums meet anyway.  Error of a gradient, FP32 S,
    // k = 20, n = 6000 / 8200 / 12200: 2.7 / 4.2 / 5.2e-7 in one chain, 1.9 / 2.2 /
    // 1.7e-7 so; a thread per row, whose runs are half as long, had 2.7 / 3.3 /
    // 3.5e-7.  0 to 2.5 % slower.
    constexpr bool SUMS = NT == 1;
    constexpr int RUN = 4;                                 // 256 columns a wave: a unit's of the tall kernel
    floatx4 sum[SUMS ? 4 : 1];
#pragma unroll
    for (int rg = 0; rg < (SUMS ? 4 : 1); ++rg) sum[rg] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4* held = (floatx4*)red[wv] + lane;              // this lane's sums of the tile's earlier runs
    int in_run = 0;
    bool any_held = false;
    u32x4 s[QS][4], b[NB], sn[QS][4], bn[NB];
    int64_t tile = u0 / p.n_chunks, ch = u0 - tile * p.n_chunks;
    load(tile, ch, s, b);
    for (int64_t u = u0; u < u1; ++u) {
        // the last unit loads itself again: in bounds, unused
        int64_t tile_n = tile, ch_n = ch;
        if (u + 1 < u1 && ++ch_n == p.n_chunks) {
            ch_n = 0;
            ++tile_n;
        }
        load(tile_n, ch_n, sn, bn);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < QS; ++q) {
            if (KIND == 0) {
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            acc[rg][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                __builtin_bit_cast(floatx4, s[q][rg])[m], __builtin_bit_cast(floatx4, b[q * NT + nt])[m],
                                acc[rg][nt], 0, 0, 0);
            } else {
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    bf16x8 av[4];
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        const u32x4 r = s[q][rg];
                        if (KIND == 2) {
                            const uint32_t w0 = h ? r[2] : r[0], w1 = h ? r[3] : r[1];
                            bf16x2 q0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false);
                            bf16x2 q1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true);
                            bf16x2 q2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false);
                            bf16x2 q3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true);
                            av[rg] = bf16x8{q0[0], q0[1], q1[0], q1[1], q2[0], q2[1], q3[0], q3[1]};
                        } else {
                            av[rg] = __builtin_bit_cast(bf16x8, r);
                        }
                    }
                    // the lowest plane of H first: its products and the middle one's are small beside
                    // the highest one's, and a tile of few columns rounds at full size once, not three
                    // times (BF16, n = 20, k = 2: error of the gradient 7.6e-8 the other way round,
                    // 4.2e-8 so, 6.7e-8 with a thread per row; n = 256: 6.7e-8, 5.2e-8, 2.0e-7)
#pragma unroll
                    for (int pl = NP - 1; pl >= 0; --pl)
#pragma unroll
                        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
                                acc[rg][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    av[rg], __builtin_bit_cast(bf16x8, b[((q * NH + h) * NP + pl) * NT + nt]),
                                    acc[rg][nt], 0, 0, 0);
                }
            }
        }
        if (SUMS) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[SUMS ? rg : 0][v] += acc[rg][0][v];
                acc[rg][0] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
        const bool last = u + 1 == u1 || tile_n != tile;
        if (!SUMS && !last && ++in_run == RUN) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    floatx4* h = held + (rg * NT + nt) * 64;
                    *h = any_held ? *h + acc[rg][nt] : acc[rg][nt];
                    acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            in_run = 0;
            any_held = true;
        }
        if (last) {
            if (SUMS) {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    acc[rg][0] = sum[SUMS ? rg : 0];
                    sum[SUMS ? rg : 0] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            } else if (any_held) {
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = held[(rg * NT + nt) * 64] + acc[rg][nt];
                // the wave's lanes have read theirs before any writes its rows over them
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            in_run = 0;
            any_held = false;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[wv][(16 * rg + 4 * lg + v) * K + 16 * nt + lr] = acc[rg][nt][v];
                    acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            __syncthreads();
            float* dst = part + ((w + tile) * TR + 64 * sub) * (int64_t)K;
#pragma unroll
            for (int f = 4 * t; f < 64 * K; f += 1024) {
                const floatx4 r0 = *(const floatx4*)&red[0][f], r1 = *(const floatx4*)&red[1][f];
                const floatx4 r2 = *(const floatx4*)&red[2][f], r3 = *(const floatx4*)&red[3][f];
                floatx4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (r0[e] + r1[e]) + (r2[e] + r3[e]);
                *(floatx4*)&dst[f] = o;
            }
            __syncthreads();
        }
        tile = tile_n;
        ch = ch_n;
#pragma unroll
        for (int q = 0; q < QS; ++q)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) s[q][rg] = sn[q][rg];
#pragma unroll
        for (int i = 0; i < NB; ++i) b[i] = bn[i];
    }
}

// ---------------------------------------------------------------------------
// Products summed by increasing column, one FP32 multiply-add after another, as
// a thread per row forms them (v_mfma_f32_16x16x4_f32 adds its four products in
// the order of the lane groups): the steps of ADMM and of the adaptive rules at
// ranks that are no width of the kernels above, whose trajectories amplify the
// last bits (ten ADMM steps at n = 5900 in another order end 2e-5 to 5e-5 from
// each other in the gradient).  A lane's consecutive columns of S become the
// lane groups' columns by a 4 x 4 transpose over the groups, two register swaps
// for two registers; codes are widened to floats first.  H comes from an FP32
// image in LDS, read so that lane group g gets the g-th of four rows.
// Four waves of 64 rows, a unit at a time, P work-groups in even runs of units.
// A launch at n = 5900 (576 units for 512 work-groups, so some have two; the
// even runs are part of the order) takes 38.2 us at k = 12, FP32 (a plain read of
// those 139 MB takes 20) and 83.8 us at k = 50, BF16 (its FP32 matrix
// instructions alone take 31).  Ten ADMM steps,
// against a thread per row in FP32 multiply-adds, in ms: n = 5900, k = 12, FP32
// 4.02 / 0.63; k = 25, BF16 6.58 / 0.77; k = 50, BF16 15.1 / 1.43; k = 22, FP8
// 6.05 / 0.77; n = 1800, k = 36, BF16 6.12 / 0.70, the same bits each time.
// ---------------------------------------------------------------------------
// t[G] of lane group g <- t[g] of lane group G
__device__ inline void group_transpose(float (&t)[4]) {
    auto swap32 = [](float& x, float& y) {
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                        false, false);
        x = __builtin_bit_cast(float, (uint32_t)r[0]);
        y = __builtin_bit_cast(float, (uint32_t)r[1]);
    };
    auto swap16 = [](float& x, float& y) {
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                        false, false);
        x = __builtin_bit_cast(float, (uint32_t)r[0]);
        y = __builtin_bit_cast(float, (uint32_t)r[1]);
    };
    swap32(t[0], t[2]);
    swap32(t[1], t[3]);
    swap16(t[0], t[1]);
    swap16(t[2], t[3]);
}

template <int KIND, int NT>
__global__ __launch_bounds__(256, NT == 4 ? 1 : 2) void stream_ordered(const void* __restrict__ Sv,
                                                                      const u32x4* __restrict__ img1,
                                                                      const u32x4* __restrict__ img2,
                                                                      float* __restrict__ part, PlanView p) {
    constexpr int K = 16 * NT, NV = KC * K / 4;
    constexpr int EB = KIND == 0 ? 4 : (KIND == 1 ? 2 : 1);
    constexpr int NS = KIND == 0 ? 16 : (KIND == 1 ? 8 : 4);
    constexpr int NH = 16 / NS;                            // floats of a lane's vector / 4
    constexpr int RING = 4, D = RING - 1;
    __shared__ u32x4 lds[NV];
    const float* hs = (const float*)lds;
    int64_t U;
    int32_t na;
    plan_bounds(p, U, na);
    if (U == 0) return;
    const int64_t Pe = U < p.P ? U : p.P;
    const int64_t w = blockIdx.x;
    if (w >= Pe) return;
    const int64_t u0 = wg_start(w, U, Pe), u1 = wg_start(w + 1, U, Pe);
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lr = lane & 15, lg = lane >> 4;
    auto s_run = [&](int32_t aa, int32_t ch) -> const u32x4* {
        return (const u32x4*)((const uint8_t*)Sv + ((int64_t)tile_of(p, aa) * p.n_chunks + ch) * TILE_ELEMS * EB +
                              (int64_t)wv * (TILE_ELEMS * EB / 4)) + lane;
    };
    int32_t a = find_active(p, u0, na), chunk;
    float wt;
    unit_decode(p, u0, a, chunk, wt);
    const u32x4* sp = s_run(a, chunk);
    u32x4 ring[RING][4];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) ring[d][rg] = __builtin_nontemporal_load(sp + (d * 4 + rg) * 64);
    floatx4 acc[4][NT];
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    int32_t a_next = a;
    for (int64_t u = u0; u < u1; ++u) {
        const bool more = u + 1 < u1;
        const u32x4* src = (wt > 1.5f ? img2 : img1) + (int64_t)chunk * NV;
        u32x4 h[NV / 256];
#pragma unroll
        for (int i = 0; i < NV / 256; ++i) h[i] = src[t + 256 * i];
        int32_t chunk_n = chunk;
        float wt_n = wt;
        const u32x4* sp_n = sp;                            // the last unit reads its own S again, unused
        if (more) {
            unit_decode(p, u + 1, a_next, chunk_n, wt_n);
            sp_n = s_run(a_next, chunk_n);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NV / 256; ++i) lds[t + 256 * i] = h[i];
        __syncthreads();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int sd = s + D;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
                ring[sd % RING][rg] = __builtin_nontemporal_load((sd < NS ? sp + (sd * 4 + rg) * 64
                                                                          : sp_n + ((sd - NS) * 4 + rg) * 64));
            __builtin_amdgcn_sched_barrier(0);
            // x[rg][q][G]: columns of float 4 q + (lane group), of lane group G
            float x[4][NH][4];
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const u32x4 r = ring[s % RING][rg];
#pragma unroll
                for (int q = 0; q < NH; ++q) {
                    float(&y)[4] = x[rg][q];               // floats 4 q .. 4 q + 3 of the vector
                    if (KIND == 0) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[e] = __uint_as_float(r[e]);
                    } else if (KIND == 1) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            y[e] = bf16_bits_to_f32((uint16_t)(r[(2 * q + (e >> 1)) & 3] >> (16 * (e & 1))));
                    } else {
                        const int code = (int)r[q];
                        y[0] = __builtin_amdgcn_cvt_f32_fp8(code, 0);
                        y[1] = __builtin_amdgcn_cvt_f32_fp8(code, 1);
                        y[2] = __builtin_amdgcn_cvt_f32_fp8(code, 2);
                        y[3] = __builtin_amdgcn_cvt_f32_fp8(code, 3);
                    }
                    group_transpose(x[rg][q]);
                }
            }
#pragma unroll
            for (int j = 0; j < 4 * NH; ++j) {             // columns 4 j .. 4 j + 3 of the sub-step
                const int g16 = NH * s + (j >> 2);         // 16-row group of the chunk
                float b[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) b[nt] = hs[(((nt * 16 + g16) * 4 + (j & 3)) * 16 + lr) * 4 + lg];
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[rg][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[rg][j % NH][j / NH], b[nt], acc[rg][nt], 0, 0, 0);
            }
        }
        if (!more || a_next != a) {
            float* dst = part + (w + a) * (int64_t)TR * K;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) dst[(64 * wv + 16 * rg + 4 * lg + v) * K + 16 * nt + lr] = acc[rg][nt][v];
                    acc[rg][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
        }
        a = a_next;
        chunk = chunk_n;
        wt = wt_n;
        sp = sp_n;
    }
}

// One work-group per CU (64 w of four): with two or four per CU a tile has more
// partials to write and to sum (n = 4100, k = 32, FP32: 40.6, 48.4 and 58.1 us a
// step).  The line lies where MU steps of this kernel and of the tall one cross,
// us here / there, FP32, BF16, FP8 S.  Up to 32 columns (k = 32): n = 512 21 / 37,
// 21 / 25, 21 / 25; 8192 (U = 1024) 63 / 77, 46 / 59, 40 / 47; 12000 (U = 2209)
// 114 / 133 on FP32, which is level at 16000, where BF16 and FP8 lose.  64
// columns: n = 512 34 / 61, 32 / 39, 33 / 40; 6000 (U = 576) 88 / 109, 60 / 67,
// 58 / 62; 6900 (U = 729) 106 / 107, 69 / 66, 65 / 62; all lose or tie at 8192.
int32_t stream_quarter_wgs(int cus, int32_t stype, int64_t n_tiles, int64_t n_chunks, int64_t k) {
    const int64_t U = n_tiles * n_chunks, P = std::max(cus / 4, 1);
    const bool fp32 = stype == SYMNMF_S_FP32;
    const int64_t most = mfma_width(k) == 64 ? (fp32 ? 768 : 640) : (fp32 ? 2304 : 1024);
    if (U > most) return 0;
    return (int32_t)std::min(U, P);
}

int stream_uses_mfma(int32_t stype, int h_f64, int acc_f64, int64_t k) {
    if (h_f64 || acc_f64 || stype == SYMNMF_S_FP64) return 0;
    return (k >= 1 && k <= KMAX) ? 1 : 0;
}

template <typename ST>
static hipError_t launch_generic(const void* S, int64_t ld, const double* H, int64_t k, double* part, const PlanView& p,
                                 hipStream_t stream) {
    dim3 grid(p.P), block(256);
    if (k <= 8)
        hipLaunchKernelGGL((stream_generic<ST, 8>), grid, block, 0, stream, (const ST*)S, ld, H, (int)k, part, p);
    else if (k <= 16)
        hipLaunchKernelGGL((stream_generic<ST, 16>), grid, block, 0, stream, (const ST*)S, ld, H, (int)k, part, p);
    else if (k <= 32)
        hipLaunchKernelGGL((stream_generic<ST, 32>), grid, block, 0, stream, (const ST*)S, ld, H, (int)k, part, p);
    else
        hipLaunchKernelGGL((stream_generic<ST, 64>), grid, block, 0, stream, (const ST*)S, ld, H, (int)k, part, p);
    return hipGetLastError();
}

// LDS per work-group (image buffers): FP32 k=16/32 double-buffered (32/64 KB),
// k=64 single (64 KB); BF16/FP8 keep three bf16 planes: k=16 double (48 KB),
// k=32 single (48 KB), k=64 single (96 KB, one work-group per CU).
// Tall kernels (one 8-wave work-group per CU) double-buffer the images up to
// k = 32 (FP32 64 KB, BF16 / FP8 96 KB) and FP32 at k = 64 (128 KB); BF16 / FP8
// at k = 64 keep one 96 KB image.
template <int KIND>
static void launch_mfma_kind(const void* S, const u32x4* img1, const u32x4* img2, void* part, int64_t k,
                             const PlanView& p, hipStream_t stream, const AdmmInverse& inv) {
    dim3 grid(p.P);
    k = mfma_width(k);
    if (p.ordered) {
        if (k == 16) hipLaunchKernelGGL((stream_ordered<KIND, 1>), grid, dim3(256), 0, stream, S, img1, img2, (float*)part, p);
        else if (k == 32) hipLaunchKernelGGL((stream_ordered<KIND, 2>), grid, dim3(256), 0, stream, S, img1, img2, (float*)part, p);
        else hipLaunchKernelGGL((stream_ordered<KIND, 4>), grid, dim3(256), 0, stream, S, img1, img2, (float*)part, p);
        return;
    }
    if (p.quarter) {
        const dim3 qg(4 * p.P + (inv.gram ? 1 : 0)), qb(256);
        if (k == 16) hipLaunchKernelGGL((stream_quarter<KIND, 1>), qg, qb, 0, stream, S, img1, (float*)part, p, inv);
        else if (k == 32) hipLaunchKernelGGL((stream_quarter<KIND, 2>), qg, qb, 0, stream, S, img1, (float*)part, p, inv);
        else hipLaunchKernelGGL((stream_quarter<KIND, 4>), qg, qb, 0, stream, S, img1, (float*)part, p, inv);
        return;
    }
    if (p.tall) {
        dim3 block(512);
        if constexpr (KIND == 0)
            if (p.by_unit) {
                if (k == 16) hipLaunchKernelGGL((stream_mfma<0, 1, true, true, SUM_UNIT, true>), grid, block, 0, stream, S, img1, img2, part, p);
                else if (k == 32) hipLaunchKernelGGL((stream_mfma<0, 2, true, true, SUM_UNIT, true>), grid, block, 0, stream, S, img1, img2, part, p);
                else hipLaunchKernelGGL((stream_mfma<0, 4, true, false, SUM_UNIT, true>), grid, block, 0, stream, S, img1, img2, part, p);
                return;
            }
        if (k == 16) hipLaunchKernelGGL((stream_mfma<KIND, 1, true, true, SUM_RUN, true>), grid, block, 0, stream, S, img1, img2, part, p);
        else if (k == 32) hipLaunchKernelGGL((stream_mfma<KIND, 2, true, true, SUM_RUN, true>), grid, block, 0, stream, S, img1, img2, part, p);
        else hipLaunchKernelGGL((stream_mfma<KIND, 4, KIND == 0, false, SUM_RUN, true>), grid, block, 0, stream, S, img1, img2, part, p);
        return;
    }
    dim3 block(256);
    if (k == 16) hipLaunchKernelGGL((stream_mfma<KIND, 1, true, true, SUM_RUN, false>), grid, block, 0, stream, S, img1, img2, part, p);
    else if (k == 32) hipLaunchKernelGGL((stream_mfma<KIND, 2, KIND == 0, true, SUM_RUN, false>), grid, block, 0, stream, S, img1, img2, part, p);
    else hipLaunchKernelGGL((stream_mfma<KIND, 4, false, false, SUM_RUN, false>), grid, block, 0, stream, S, img1, img2, part, p);
}

// Wide pass: FP32 S, tall full plans, 80 columns, the first 64 of them those of X
// and the others the first of X2 (rows 64 apart).  For a factor of more than 64
// columns with at most 16 left, e.g. 141 = 64 + 64 + 13: a pass of 16 columns
// takes as long as S takes to read, 0.27 ms at n = 20000, and its products a
// quarter of the 0.46 ms of 64 columns: 0.58 ms for both.  (96
// columns do not fit the registers beside the S in flight.)
int64_t wide_image_words(int64_t n_chunks) { return KC * WIDE_COLS * n_chunks; }

hipError_t launch_stream_wide(const void* S, const float* X, const float* X2, uint32_t* img, float* part,
                              const PlanView& p, hipStream_t stream) {
    if (!p.full || !p.tall) return hipErrorInvalidValue;
    u32x4* im = (u32x4*)img;
    hipLaunchKernelGGL((h_image_kernel<0, WIDE_COLS>), dim3((unsigned)p.n_chunks, WIDE_COLS / 16), dim3(256), 0, stream,
                       X, WIDE_COLS, 64, (int64_t)0, 1.0f, im, X2);
    hipLaunchKernelGGL((stream_mfma<0, WIDE_COLS / 16, false, false, SUM_RUN, true>), dim3(p.P), dim3(512), 0, stream, S,
                       im, im, (void*)part, p);
    return hipGetLastError();
}

int stream_tall_supported(int32_t stype, int h_f64, int64_t k) {
    return stream_uses_mfma(stype, h_f64, 0, k);
}

template <int KIND>
static void launch_mfma_kind_acc64(const void* S, const u32x4* img, void* part, int64_t k, const PlanView& p,
                                   hipStream_t stream) {
    dim3 grid(p.P), block(256);
    if (k == 16) hipLaunchKernelGGL((stream_mfma<KIND, 1, true, false, SUM_F64, false>), grid, block, 0, stream, S, img, img, part, p);
    else hipLaunchKernelGGL((stream_mfma<KIND, 2, KIND == 0, false, SUM_F64, false>), grid, block, 0, stream, S, img, img, part, p);
}

int stream_acc64_supported(int32_t stype, int64_t k) {
    return (stype == SYMNMF_S_FP32 || stype == SYMNMF_S_BF16 || stype == SYMNMF_S_FP8) && (k == 16 || k == 32);
}

hipError_t launch_stream_acc64(const void* S, int32_t stype, int64_t k, const void* img, double* part,
                               const PlanView& p, hipStream_t stream) {
    if (!stream_acc64_supported(stype, k) || !img || p.tall) return hipErrorInvalidValue;   // 4-wave kernel only
    const u32x4* i1 = (const u32x4*)img;
    if (stype == SYMNMF_S_FP32) launch_mfma_kind_acc64<0>(S, i1, part, k, p, stream);
    else if (stype == SYMNMF_S_BF16) launch_mfma_kind_acc64<1>(S, i1, part, k, p, stream);
    else launch_mfma_kind_acc64<2>(S, i1, part, k, p, stream);
    return hipGetLastError();
}

int stream_wgs_per_cu(int32_t stype, int64_t k) {
    if ((stype == SYMNMF_S_BF16 || stype == SYMNMF_S_FP8) && k == 64) return 1;
    return 2;
}

hipError_t launch_stream(const void* S, int32_t stype, int64_t ld, const void* H, int h_f64, int64_t k,
                         void* part, int acc_f64, const PlanView& p, hipStream_t stream, const void* img1,
                         const void* img2, const AdmmInverse& inv) {
    if (k < 1 || k > KMAX || (inv.gram && !p.quarter)) return hipErrorInvalidValue;
    if (stream_uses_mfma(stype, h_f64, acc_f64, k)) {
        if (!img1) return hipErrorInvalidValue;
        const u32x4* i1 = (const u32x4*)img1;
        const u32x4* i2 = (const u32x4*)(img2 ? img2 : img1);
        float* pf = (float*)part;
        if (stype == SYMNMF_S_FP32) launch_mfma_kind<0>(S, i1, i2, pf, k, p, stream, inv);
        else if (stype == SYMNMF_S_BF16) launch_mfma_kind<1>(S, i1, i2, pf, k, p, stream, inv);
        else if (stype == SYMNMF_S_FP8) launch_mfma_kind<2>(S, i1, i2, pf, k, p, stream, inv);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (!h_f64 || !acc_f64) return hipErrorInvalidValue;
    const double* Hd = (const double*)H;
    double* pd = (double*)part;
    switch (stype) {
        case SYMNMF_S_FP32: return launch_generic<float>(S, ld, Hd, k, pd, p, stream);
        case SYMNMF_S_BF16: return launch_generic<uint16_t>(S, ld, Hd, k, pd, p, stream);
        case SYMNMF_S_FP8: return launch_generic<uint8_t>(S, ld, Hd, k, pd, p, stream);
        case SYMNMF_S_FP64:
            if ((k == 16 || k == 32) && std::getenv("SYMNMF_F64_GENERIC") == nullptr) {
                dim3 grid(p.P), block(256);
                if (k == 16)
                    hipLaunchKernelGGL((stream_f64_mfma<1>), grid, block, 0, stream, (const double*)S, ld, Hd, pd, p);
                else
                    hipLaunchKernelGGL((stream_f64_mfma<2>), grid, block, 0, stream, (const double*)S, ld, Hd, pd, p);
                return hipGetLastError();
            }
            return launch_generic<double>(S, ld, Hd, k, pd, p, stream);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Dense product rows from the partial tiles of a full pass, summed over the
// work-groups that streamed each tile in increasing order.  32 rows to a
// work-group and eight elements to a thread, the loads of all of them issued
// together for every partial: with a 256-row tile to a work-group, its
// elements one after another, n = 20000 (79 tiles, 64 columns, 39 MB) was 64
// dependent steps on 79 CUs and took 133 us; 8 us now.
// ---------------------------------------------------------------------------
constexpr int DENSE_ROWS = 32, DENSE_NE = 8;

template <typename T>
__global__ __launch_bounds__(256) void dense_rows_kernel(const T* __restrict__ part, int64_t rows, int k, int kp,
                                                         PlanView p, const T* __restrict__ X, int64_t ldo,
                                                         const float* __restrict__ scale,
                                                         const float* __restrict__ diag, int64_t panel_rows,
                                                         T* __restrict__ out) {
    const int32_t tile = blockIdx.x / (TR / DENSE_ROWS);
    const int r0 = (int)(blockIdx.x % (TR / DENSE_ROWS)) * DENSE_ROWS;
    int64_t w_lo, w_hi, sb, sm;
    partial_slots(p, tile, w_lo, w_hi, sb, sm);
    const int64_t row0 = (int64_t)tile * TR + r0;
    for (int f0 = threadIdx.x; f0 < DENSE_ROWS * k; f0 += 256 * DENSE_NE) {
        int r[DENSE_NE], c[DENSE_NE];
        T s[DENSE_NE];
#pragma unroll
        for (int e = 0; e < DENSE_NE; ++e) {
            const int f = min(f0 + 256 * e, DENSE_ROWS * k - 1);
            r[e] = f / k;
            c[e] = f - r[e] * k;
            s[e] = 0;
        }
        for (int64_t q = w_lo; q <= w_hi; ++q) {
            const T* pq = part + ((sm * q + sb) * TR + r0) * (int64_t)kp;
#pragma unroll
            for (int e = 0; e < DENSE_NE; ++e) s[e] += pq[r[e] * kp + c[e]];
        }
#pragma unroll
        for (int e = 0; e < DENSE_NE; ++e) {
            const int64_t row = row0 + r[e];
            if (f0 + 256 * e >= DENSE_ROWS * k || row >= rows) continue;
            T v = s[e];
            if (scale) v = v / (T)scale[row / panel_rows] + (T)diag[row] * X[row * ldo + c[e]];
            out[row * ldo + c[e]] = v;
        }
    }
}

template <typename T>
hipError_t launch_dense_rows(const T* part, int64_t rows, int64_t k, int64_t kp, const PlanView& p, const T* X,
                             int64_t ldo, const float* scale, const float* diag, int64_t panel_rows, T* out,
                             hipStream_t stream) {
    if (!p.full || k < 1 || k > kp || ldo < k || rows > (int64_t)p.n_tiles * TR) return hipErrorInvalidValue;
    hipLaunchKernelGGL(dense_rows_kernel<T>, dim3((unsigned)p.n_tiles * (TR / DENSE_ROWS)), dim3(256), 0, stream, part,
                       rows, (int)k, (int)kp, p, X, ldo, scale, diag, panel_rows, out);
    return hipGetLastError();
}
template hipError_t launch_dense_rows<float>(const float*, int64_t, int64_t, int64_t, const PlanView&, const float*,
                                             int64_t, const float*, const float*, int64_t, float*, hipStream_t);
template hipError_t launch_dense_rows<double>(const double*, int64_t, int64_t, int64_t, const PlanView&, const double*,
                                              int64_t, const float*, const float*, int64_t, double*, hipStream_t);

// ---------------------------------------------------------------------------
// Device self-check of the FP8 -> BF16 conversion instruction against the
// E4M3 definition (every finite code).  bad[0] counts mismatches.
// ---------------------------------------------------------------------------
__global__ void fp8_decode_check(int32_t* bad) {
    const int code = threadIdx.x;                       // 0..255
    if ((code & 0x7f) == 0x7f) return;                  // NaN codes
    const uint32_t word = (uint32_t)code | ((uint32_t)code << 8) | ((uint32_t)code << 16) | ((uint32_t)code << 24);
    bf16x2 lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(word, 1.0f, false);
    bf16x2 hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(word, 1.0f, true);
    const float ref = fp8e4m3_to_f32((uint8_t)code);
    const float v[4] = {(float)lo[0], (float)lo[1], (float)hi[0], (float)hi[1]};
    for (int i = 0; i < 4; ++i)
        if (v[i] != ref) atomicAdd(bad, 1);
}

hipError_t launch_fp8_decode_check(int32_t* bad, hipStream_t stream) {
    hipLaunchKernelGGL(fp8_decode_check, dim3(1), dim3(256), 0, stream, bad);
    return hipGetLastError();
}

// Plain grid-stride 16-byte copy of `bytes` (a multiple of 16): a kernel of
// known traffic for calibrating hardware byte counters.
__global__ __launch_bounds__(256) void copy_probe_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                         int64_t n16) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = __builtin_nontemporal_load(src + i);
}

// Plain read of ``bytes`` (a multiple of 16): grid-stride nontemporal 16-byte
// loads, folded into one word per work-group so the loads stay live.
__global__ __launch_bounds__(256) void read_probe_kernel(const u32x4* __restrict__ src, int64_t count,
                                                         uint32_t* __restrict__ sink) {
    uint32_t acc = 0;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        const u32x4 v = __builtin_nontemporal_load(src + i);
        acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
    for (int o = 32; o > 0; o >>= 1) acc ^= __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) sink[blockIdx.x * 4 + (threadIdx.x >> 6)] = acc;
}

hipError_t launch_read_probe(const void* src, int64_t bytes, uint32_t* sink, int64_t sink_words,
                             hipStream_t stream) {
    const int64_t blocks = sink_words / 4 < 2048 ? sink_words / 4 : 2048;
    if (blocks < 1 || bytes % 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(read_probe_kernel, dim3(blocks), dim3(256), 0, stream, (const u32x4*)src, bytes / 16, sink);
    return hipGetLastError();
}

hipError_t launch_copy_probe(const void* src, void* dst, int64_t bytes, hipStream_t stream) {
    hipLaunchKernelGGL(copy_probe_kernel, dim3(4096), dim3(256), 0, stream, (const u32x4*)src, (u32x4*)dst, bytes / 16);
    return hipGetLastError();
}

}  // namespace symnmf
