// Work plan of a sub-sampled step, built on the device so that steps stay
// asynchronous (no host round trip per iteration).
//
// Row-Stochastic SVRG (appendix, family 3): the rows of the sampled blocks I
// take their exact gradient, so their tiles stream every column chunk with
// weight 1.
//
// Block-SVRG AdaptGrow (appendix, family 3): with sampled block sets I and J,
//   g_I = 2 (H_I (H_J^T H_J) - S_IJ H_J),  g_J = 2 (H_J (H_I^T H_I) - S_JI H_I),
// summed on rows in both sets.  Per row tile the S.H term is one weighted sum
// over column chunks:
//   class 0 (rows in I only): chunks of J, weight 1, Gram_eff = Gram_J
//   class 1 (rows in J only): chunks of I, weight 1, Gram_eff = Gram_I
//   class 2 (rows in I and J): chunks of I u J, weight [b in J] + [b in I],
//                              Gram_eff = Gram_I + Gram_J
// so S_IJ and S_JI are read once, in trace form, with no |I| x |J| residual.
#include "common.h"

namespace symnmf {

constexpr int MAX_BLOCKS = 4096;

// One work-group.  Only the shuffles are a serial chain (one exchange in LDS per
// sampled block, I and J on two waves at once, their uniforms drawn beforehand
// by all threads); the lists come from prefix sums 256 entries at a time.
// Everything on one thread took 40 us at n = 20000 (20 blocks, 79 tiles); this
// takes 6.1 us.
constexpr int PT = 256;

// exclusive prefix of v over the work-group, total in *sum; sh: PT / 64 ints
__device__ inline int block_prefix(int v, int* sum, int* sh) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
    }
    __syncthreads();
    if (lane == 63) sh[wv] = incl;
    __syncthreads();
    int base = 0, all = 0;
    for (int q = 0; q < PT / 64; ++q) {
        if (q < wv) base += sh[q];
        all += sh[q];
    }
    *sum = all;
    return base + incl - v;
}

__global__ __launch_bounds__(PT) void plan_kernel(PlanRequest r, int32_t* __restrict__ base) {
    __shared__ int32_t perm[2][MAX_BLOCKS], pick[2][MAX_BLOCKS];
    __shared__ uint8_t flag[2][MAX_BLOCKS];
    __shared__ int sh[PT / 64];
    const int t = threadIdx.x, nt = r.n_tiles, nc = r.n_chunks, nb = r.n_blocks;
    int32_t* hdr = base;
    int32_t* active_tile = base + 8;
    int32_t* active_class = active_tile + nt;
    int32_t* unit_offset = active_class + nt;
    int32_t* class_chunks = unit_offset + nt + 1;
    int32_t* class_weight = class_chunks + 3 * nc;
    int32_t* tile_active = class_weight + 3 * nc;

    // the sampler of sample_block_flags for the sets I (stream 0) and J (stream 1)
    const int sets = r.mode == 2 && r.independent ? 2 : 1;
    for (int q = 0; q < 2; ++q) {
        const uint64_t key = splitmix64(r.seed, (uint64_t)(2 * r.t + q));
        for (int i = t; i < nb; i += PT) {
            perm[q][i] = i;
            flag[q][i] = 0;
            if (q < sets && i < r.m) pick[q][i] = i + (int)(uniform24(key, (uint64_t)i) * (double)(nb - i));
        }
    }
    __syncthreads();
    if ((t & 63) == 0 && (t >> 6) < sets) {
        int32_t* p = perm[t >> 6];
        for (int i = 0; i < r.m; ++i) {
            const int j = pick[t >> 6][i];
            const int32_t a = p[i], b = p[j];
            p[j] = a;
            p[i] = b;
        }
    }
    __syncthreads();
    for (int i = t; i < r.m; i += PT)
        for (int q = 0; q < sets; ++q) flag[q][perm[q][i]] = 1;
    __syncthreads();
    const uint8_t* fI = flag[0];
    // J = I without independent sets; no J for row steps (flag[1] is clear)
    const uint8_t* fJ = r.mode == 2 && !r.independent ? flag[0] : flag[1];
    int len[3] = {0, 0, 0};
    if (r.mode == 1) {
        for (int c = t; c < nc; c += PT) {
            class_chunks[c] = c;
            class_weight[c] = 1;
        }
        len[0] = nc;
    } else {
        for (int c0 = 0; c0 < nc; c0 += PT) {
            const int c = c0 + t, b = c / r.chunks_per_block;
            const int inI = c < nc ? fI[b] : 0, inJ = c < nc ? fJ[b] : 0;
            const int in[3] = {inJ, inI, inI | inJ}, weight[3] = {1, 1, inI + inJ};
            for (int q = 0; q < 3; ++q) {
                int sum;
                const int at = len[q] + block_prefix(in[q], &sum, sh);
                if (in[q]) {
                    class_chunks[q * nc + at] = c;
                    class_weight[q * nc + at] = weight[q];
                }
                len[q] += sum;
            }
        }
    }
    int na = 0, U = 0;
    for (int i0 = 0; i0 < nt; i0 += PT) {
        const int i = i0 + t, b = i / r.tiles_per_block;
        const int inI = i < nt ? fI[b] : 0, inJ = i < nt ? fJ[b] : 0;
        const int active = inI | inJ;
        const int cls = r.mode == 1 ? 0 : (inI && inJ ? 2 : (inI ? 0 : 1));
        int sum, units;
        const int at = na + block_prefix(active, &sum, sh);
        const int off = U + block_prefix(active ? len[cls] : 0, &units, sh);
        if (i < nt) tile_active[i] = active ? at : -1;
        if (active) {
            active_tile[at] = i;
            active_class[at] = cls;
            unit_offset[at] = off;
        }
        na += sum;
        U += units;
    }
    if (t == 0) {
        unit_offset[na] = U;
        hdr[0] = na;
        hdr[1] = U;
        hdr[2] = 0;
        hdr[3] = len[0];
        hdr[4] = len[1];
        hdr[5] = len[2];
    }
}

hipError_t launch_plan(const PlanRequest& r, int32_t* plan_base, hipStream_t stream) {
    if (r.n_blocks > MAX_BLOCKS || r.m < 1 || r.m > r.n_blocks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(PT), 0, stream, r, plan_base);
    return hipGetLastError();
}

}  // namespace symnmf
