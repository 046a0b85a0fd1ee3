// Layout of the chunk images of H that the MFMA stream reads, and the update
// kernels' writer of it.
#pragma once
#include "common.h"

namespace symnmf {

// ---------------------------------------------------------------------------
// H images.  KIND 0 (FP32 S): floats in the order Hs[nt][s][g][c][m];
// KIND 1 (BF16 S): three bf16 planes, each Hb[nt][s][g][c][i];
// KIND 2 (FP8 S): three bf16 planes, each Hb[nt][s][h][g][c][i].
// (nt = H column / 16, c = H column % 16; the other indices split the chunk
// column kk as the matching kernel's sub-step reads it.)
// ---------------------------------------------------------------------------
__device__ inline void split3_bf16(float x, uint16_t& hi, uint16_t& mid, uint16_t& lo) {
    hi = f32_to_bf16_bits(x);
    const float r1 = x - bf16_bits_to_f32(hi);
    mid = f32_to_bf16_bits(r1);
    const float r2 = r1 - bf16_bits_to_f32(mid);
    lo = f32_to_bf16_bits(r2);
}

// First chunk row kk0 and H column of image vector v (16 bytes: 4 floats for
// KIND 0, 8 bf16 of one plane otherwise); the vector holds rows kk0, kk0 + 1, ...
// of that column, in the order given above.
template <int KIND>
__device__ inline void image_vector_origin(int v, int& kk0, int& col) {
    const int c = v & 15, g = (v >> 4) & 3;
    if (KIND == 0) {
        kk0 = 16 * ((v >> 6) & 15) + 4 * g;
        col = 16 * (v >> 10) + c;
    } else if (KIND == 1) {
        kk0 = 32 * ((v >> 6) & 7) + 8 * g;
        col = 16 * (v >> 9) + c;
    } else {
        kk0 = 64 * ((v >> 7) & 3) + 16 * g + 8 * ((v >> 6) & 1);
        col = 16 * (v >> 9) + c;
    }
}

template <int KIND, int K>
struct ImageShape {
    static constexpr int BUFW = KIND == 0 ? KC * K : 3 * KC * K / 2;   // 32-bit words per chunk image
    static constexpr int NV = BUFW / 4;                                 // 16-byte vectors per image
    static constexpr int PLANE = KC * K;                                // bf16 elements per plane
};

// Images of the 64 rows [g0, g0 + 64) of H, g0 a multiple of 64 (a quarter of a
// chunk, a run of whole sub-steps): row r < valid from Hn, the others from Ho
// (both LDS, rows of K floats); img2 (may be null) gets the images of 2 H.
// Called by all threads of the work-group that has just formed the rows,
// so that H is not read again: a launch of its own for every step took 2.6 us
// of a step at n = 512, 7 / 13.5 us (FP32 / FP8 S) at n = 10^5, k = 32, and
// 156 us on the n = 10^6 row share, where it rewrote the images of the 987500
// rows that no step of the share changes.
template <int KIND, int K, int THREADS>
__device__ inline void write_image_slice_kind(const float* Hn, const float* Ho, int valid, int64_t g0, u32x4* img1,
                                              u32x4* img2) {
    using IS = ImageShape<KIND, K>;
    constexpr int EPV = KIND == 0 ? 4 : 8;
    constexpr int VP = KC * K / EPV;                       // vectors per plane
    const int q = (int)((g0 & (KC - 1)) >> 6);
    const int64_t base = (g0 / KC) * IS::NV;
    for (int i = threadIdx.x; i < 64 * K / EPV; i += THREADS) {
        // vector v of the image and the slice row kk of its first entry
        const int c = i & 15, g = (i >> 4) & 3;
        int v, kk, nt;
        if (KIND == 0) {
            const int s = (i >> 6) & 3;
            nt = i >> 8;
            v = nt * 1024 + (4 * q + s) * 64 + g * 16 + c;
            kk = 16 * s + 4 * g;
        } else if (KIND == 1) {
            const int s = (i >> 6) & 1;
            nt = i >> 7;
            v = nt * 512 + (2 * q + s) * 64 + g * 16 + c;
            kk = 32 * s + 8 * g;
        } else {
            const int h = (i >> 6) & 1;
            nt = i >> 7;
            v = nt * 512 + q * 128 + h * 64 + g * 16 + c;
            kk = 16 * g + 8 * h;
        }
        float x[EPV];
#pragma unroll
        for (int e = 0; e < EPV; ++e) x[e] = (kk + e < valid ? Hn : Ho)[(kk + e) * K + 16 * nt + c];
#pragma unroll
        for (int copy = 0; copy < 2; ++copy) {
            u32x4* img = copy ? img2 : img1;
            if (!img) continue;
            const float wt = copy ? 2.0f : 1.0f;
            if (KIND == 0) {
                u32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(uint32_t, x[e] * wt);
                img[base + v] = o;
            } else {
                u32x4 o[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint16_t h0, m0, l0, h1, m1, l1;
                    split3_bf16(x[(2 * e) % EPV] * wt, h0, m0, l0);
                    split3_bf16(x[(2 * e + 1) % EPV] * wt, h1, m1, l1);
                    o[0][e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
                    o[1][e] = (uint32_t)m0 | ((uint32_t)m1 << 16);
                    o[2][e] = (uint32_t)l0 | ((uint32_t)l1 << 16);
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) img[base + pl * VP + v] = o[pl];
            }
        }
    }
}

// kind: the KIND of the storage type (0 FP32, 1 BF16, 2 FP8)
template <int K, int THREADS>
__device__ inline void write_image_slice(int kind, const float* Hn, const float* Ho, int valid, int64_t g0, void* img1,
                                         void* img2) {
    if (kind == 0) write_image_slice_kind<0, K, THREADS>(Hn, Ho, valid, g0, (u32x4*)img1, (u32x4*)img2);
    else if (kind == 1) write_image_slice_kind<1, K, THREADS>(Hn, Ho, valid, g0, (u32x4*)img1, (u32x4*)img2);
    else write_image_slice_kind<2, K, THREADS>(Hn, Ho, valid, g0, (u32x4*)img1, (u32x4*)img2);
}

}  // namespace symnmf
