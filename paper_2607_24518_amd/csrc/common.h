// Internal declarations shared by the HIP sources of the SymNMF library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <cstdlib>

#include "../../include/symnmf.h"

namespace symnmf {

// Row tile of S handled by one work unit / one update work-group, and the
// column chunk streamed per unit.  Storage pads rows and columns of S and the
// rows of H to multiples of these, so no kernel needs a bounds test on the
// streamed data.
constexpr int TR = 256;
constexpr int KC = 256;
constexpr int KMAX = 64;
// The update kernel works on row slices of SR = TR / SUBT rows (one
// work-group each); per-slice FP64 partials (Gram, trace, KKT) are indexed
// slice = SUBT * tile + sub.
constexpr int SUBT = 4;
constexpr int SR = TR / SUBT;
constexpr int64_t PAD = 256;

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Columns the MFMA stream works on for rank k: its column blocks are 16 wide and
// it exists for 1, 2 and 4 of them; the columns past k are zero in the images of
// H and in the partials, whose rows have this stride.  The padded products are
// free where they matter: at any rank but 16, 32 and 64 a thread per row of S
// was the alternative, and that took 247 us a step at n = 4100, k = 20 where the
// 32-column MFMA stream takes 29 us.
inline int64_t mfma_width(int64_t k) { return k <= 16 ? 16 : (k <= 32 ? 32 : 64); }

// ---------------------------------------------------------------------------
// Tiled storage of S (FP32, BF16, FP8).  S is cut into 256 x 256 tiles,
// stored tile after tile in (row tile, column chunk) order.  Inside a tile the
// elements appear in exactly the order the MFMA stream kernel consumes them:
// [wave wv 0..3][sub-step s][row group rg 0..3][lane l 0..63][E elements],
// where one lane holds E consecutive columns (16 bytes: E = 4 FP32, 8 BF16,
// 16 FP8) of row 64 wv + 16 rg + (l % 16), starting at column
// s (4E) + (l / 16) E.  Each wave instruction therefore reads 1 KB of
// contiguous memory and each wave streams 64 (FP32) / 32 / 16 KB sequentially
// per tile.  FP64 storage (parity runs) is plain row-major with leading
// dimension ld.
// ---------------------------------------------------------------------------
constexpr int64_t TILE_ELEMS = (int64_t)TR * KC;

__host__ __device__ inline int64_t tiled_offset(int64_t r, int64_t c, int64_t n_chunks, int E) {
    const int64_t R = r >> 8, C = c >> 8;
    const int rr = (int)(r & 255), cc = (int)(c & 255);
    const int wv = rr >> 6, rg = (rr >> 4) & 3, lr = rr & 15;
    const int W = 4 * E;
    const int NS = 256 / W;
    const int s = cc / W, lg = (cc % W) / E, e = cc % E;
    const int64_t in_tile = (((int64_t)(wv * NS + s) * 4 + rg) * 64 + (lg * 16 + lr)) * E + e;
    return (R * n_chunks + C) * TILE_ELEMS + in_tile;
}
inline int elems_per_16B(int32_t dtype) {
    return dtype == SYMNMF_S_FP32 ? 4 : (dtype == SYMNMF_S_BF16 ? 8 : 16);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Storage conversions (round to nearest even)
// ---------------------------------------------------------------------------
__host__ __device__ inline uint16_t f32_to_bf16_bits(float x) {
    uint32_t u = __builtin_bit_cast(uint32_t, x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__host__ __device__ inline float bf16_bits_to_f32(uint16_t b) {
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// OCP FP8 E4M3 (bias 7, no infinities, max 448, subnormal quantum 2^-9),
// saturating, round to nearest even.
__host__ __device__ inline uint8_t f32_to_fp8e4m3(float x) {
    uint8_t sign = (x < 0.0f || (x == 0.0f && __builtin_signbit(x))) ? 0x80 : 0;
    float a = __builtin_fabsf(x);
    if (!(a == a)) return 0x7f;                       // NaN
    if (a >= 448.0f) return sign | 0x7e;
    if (a < 0.015625f) {                              // below 2^-6: subnormal grid 2^-9
        float q = __builtin_rintf(a * 512.0f);        // 0..8 (8 = smallest normal, code 0x08)
        return sign | (uint8_t)q;
    }
    int e;
    float m = __builtin_frexpf(a, &e);                // a = m 2^e, m in [0.5, 1)
    float mant = __builtin_rintf((m * 2.0f - 1.0f) * 8.0f);   // 0..8
    int E = e - 1 + 7;
    if (mant >= 8.0f) { mant = 0.0f; E += 1; }
    uint32_t code = ((uint32_t)E << 3) | (uint32_t)mant;
    if (code > 0x7e) code = 0x7e;
    return sign | (uint8_t)code;
}
__host__ __device__ inline float fp8e4m3_to_f32(uint8_t b) {
    int e = (b >> 3) & 15, m = b & 7;
    float v = e == 0 ? (float)m * (1.0f / 512.0f) : __builtin_ldexpf(1.0f + (float)m * 0.125f, e - 7);
    return (b & 0x80) ? -v : v;
}

template <typename T> __device__ inline double load_as_f64(const T* p);
template <> __device__ inline double load_as_f64<double>(const double* p) { return *p; }
template <> __device__ inline double load_as_f64<float>(const float* p) { return (double)*p; }
template <> __device__ inline double load_as_f64<uint16_t>(const uint16_t* p) { return (double)bf16_bits_to_f32(*p); }
template <> __device__ inline double load_as_f64<uint8_t>(const uint8_t* p) { return (double)fp8e4m3_to_f32(*p); }

// ---------------------------------------------------------------------------
// Work plan of one S.H pass.
//
// A pass covers "active" row tiles; active tile a streams the column-chunk
// list of its class (0..2), each chunk with weight 1 or 2 (the weight
// multiplies the H rows of that chunk, exactly).  Unit = (active tile, list
// position).  Units are numbered tile-major (active tile a owns units
// [unit_offset[a], unit_offset[a+1])) and split evenly over the Pe = min(P, U)
// persistent work-groups: WG w owns [w U / Pe, (w+1) U / Pe).  Every maximal
// run of one tile inside one WG's range writes one partial S.H tile at index
// (w + a) of the partial buffer; (w, a) -> w + a is one-to-one because the
// ranges are ordered, so the buffer needs at most (P + active tiles) tiles.
// The update kernel sums the partials of tile a in increasing w, so results
// do not depend on scheduling.
//
// The device-side plan lives in one int32 array (layout below) written by the
// plan kernel; a "full" pass (every tile, every chunk, weight 1) needs none of
// it.
// ---------------------------------------------------------------------------
struct PlanView {
    int32_t full;
    int32_t tall;             // full plans only: units are (pair of row tiles, chunk), see below
    int32_t quarter;          // full plans only: four work-groups per w, one per 64 rows of its tiles
    int32_t ordered;          // products summed by increasing column (stream_ordered)
    int32_t by_unit;          // tall plans of FP32 S: units summed by themselves
    int32_t n_tiles;          // row tiles of the stored panel
    int32_t n_chunks;         // column chunks (ld / KC)
    int32_t P;                // launched persistent work-groups
    // device arrays (unused when full)
    const int32_t* hdr;       // [0] n_active, [1] U lo, [2] U hi, [3] class_len[0..2] at 3..5
    const int32_t* active_tile;    // [n_tiles]
    const int32_t* active_class;   // [n_tiles]
    const int32_t* unit_offset;    // [n_tiles + 1]
    const int32_t* class_chunks;   // [3][n_chunks]
    const int32_t* class_weight;   // [3][n_chunks]
    const int32_t* tile_active;    // [n_tiles] active index or -1
};

// int32 words of the device plan for given sizes
inline int64_t plan_words(int64_t n_tiles, int64_t n_chunks) {
    return 8 + 3 * n_tiles + 1 + 6 * n_chunks + n_tiles;
}
inline PlanView plan_view(int32_t* base, int32_t full, int32_t n_tiles, int32_t n_chunks, int32_t P) {
    PlanView v;
    v.full = full; v.tall = 0; v.quarter = 0; v.ordered = 0; v.by_unit = 0; v.n_tiles = n_tiles; v.n_chunks = n_chunks; v.P = P;
    v.hdr = base;
    v.active_tile = base + 8;
    v.active_class = v.active_tile + n_tiles;
    v.unit_offset = v.active_class + n_tiles;
    v.class_chunks = v.unit_offset + n_tiles + 1;
    v.class_weight = v.class_chunks + 3 * n_chunks;
    v.tile_active = v.class_weight + 3 * n_chunks;
    return v;
}

// Tall full plans: a unit is (pair q of row tiles 2q and 2q+1, chunk), streamed
// by one 8-wave work-group whose two halves share the chunk image; the partial
// of tile 2q + h from work-group w goes to index 2 (w + q) + h (one-to-one for
// the same reason as above), so the buffer needs 2 (P + pairs) tiles.
__host__ __device__ inline int64_t tall_pairs(int64_t n_tiles) { return (n_tiles + 1) / 2; }

// Work-groups of a tall full pass: one per CU, except that when a whole
// number m of work-groups per tile pair fills at least 95 % of the CUs the
// pass uses exactly pairs * m.  The contiguous unit ranges then split every
// pair into the same m chunk segments, so all work-groups walk the same m
// chunk positions at the same time and the H images they stage are served
// from L2 / MALL instead of being fetched from HBM once per pair
// (SYMNMF_TALL_ALIGN=0 turns this off).
inline int32_t tall_wgs(int cus, int64_t n_tiles) {
    const int64_t pairs = tall_pairs(n_tiles);
    const char* e = std::getenv("SYMNMF_TALL_ALIGN");
    if (pairs <= cus && !(e && e[0] == '0')) {
        const int64_t m = cus / pairs;
        if (20 * pairs * m >= 19 * (int64_t)cus) return (int32_t)(pairs * m);
    }
    return cus;
}

__host__ __device__ inline int64_t wg_start(int64_t w, int64_t U, int64_t Pe) { return w * U / Pe; }
// the work-group whose range holds unit u
__host__ __device__ inline int64_t wg_owner(int64_t u, int64_t U, int64_t Pe) { return ((u + 1) * Pe - 1) / U; }

__device__ inline int64_t upd_unit_off(const PlanView& p, int32_t a) {
    return p.full ? (int64_t)a * p.n_chunks : (int64_t)p.unit_offset[a];
}

// The S.H partial tiles of active tile act: index (w + act), or 2 (w + pair) +
// half for tall full plans, over the work-groups w_lo..w_hi that streamed its
// units (none when act < 0).
__device__ inline void partial_slots(const PlanView& p, int32_t act, int64_t& w_lo, int64_t& w_hi,
                                     int64_t& slot_base, int64_t& slot_mul) {
    w_lo = 0;
    w_hi = -1;
    slot_base = act;
    slot_mul = 1;
    if (act < 0) return;
    int64_t U;
    if (p.full && p.tall) {
        const int64_t q = act >> 1;
        U = tall_pairs(p.n_tiles) * p.n_chunks;
        const int64_t Pe = U < p.P ? U : p.P;
        w_lo = wg_owner(q * p.n_chunks, U, Pe);
        w_hi = wg_owner((q + 1) * p.n_chunks - 1, U, Pe);
        slot_base = 2 * q + (act & 1);
        slot_mul = 2;
    } else {
        if (p.full) U = (int64_t)p.n_tiles * p.n_chunks;
        else U = (int64_t)(uint32_t)p.hdr[1] | ((int64_t)p.hdr[2] << 32);
        const int64_t Pe = U < p.P ? U : p.P;
        w_lo = wg_owner(upd_unit_off(p, act), U, Pe);
        w_hi = wg_owner(upd_unit_off(p, act + 1) - 1, U, Pe);
    }
}

// SplitMix64 (Steele, Lea & Flood 2014): output number c of the stream keyed s.
__host__ __device__ inline uint64_t splitmix64(uint64_t key, uint64_t c) {
    uint64_t z = key + (c + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__host__ __device__ inline double uniform24(uint64_t key, uint64_t c) {
    return (double)(splitmix64(key, c) >> 40) * (1.0 / 16777216.0);
}

// Index-set sampler of the stochastic variants: m distinct blocks of
// [0, nb) by a partial Fisher-Yates shuffle (Knuth, TAOCP 2, Algorithm P)
// driven by the SplitMix64 stream keyed by (seed, 2t + stream); flags[b] = 1
// for the chosen blocks.  perm: nb ints of scratch.
__host__ __device__ inline void sample_block_flags(uint64_t seed, int64_t t, int stream, int nb, int m,
                                                   int32_t* perm, uint8_t* flags) {
    const uint64_t key = splitmix64(seed, (uint64_t)(2 * t + stream));
    for (int i = 0; i < nb; ++i) perm[i] = i;
    for (int i = 0; i < m; ++i) {
        const double u = uniform24(key, (uint64_t)i);
        const int j = i + (int)(u * (double)(nb - i));
        const int32_t tmp = perm[i];
        perm[i] = perm[j];
        perm[j] = tmp;
    }
    for (int i = 0; i < nb; ++i) flags[i] = 0;
    for (int i = 0; i < m; ++i) flags[perm[i]] = 1;
}

// The inverse an ADMM step needs, minv = (2 gram + rho I)^-1 (k x k), formed by the stream's launch
// where the plan is a quarter-tile one; gram null: none.
struct AdmmInverse {
    const double* gram = nullptr;
    int k = 0;
    double rho = 0.0;
    float* minv = nullptr;
};
// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
// stream.hip: partial S.H of every active tile.  S: rows_pad x ld of stype;
// H: global rows, n_pad x k (h_f64: double); part: (P + n_tiles) * TR * k of
// the accumulation type (acc_f64: double).  Returns hipErrorInvalidValue for
// combinations without a kernel.
// MFMA kernels (stream_uses_mfma) write partial rows of mfma_width(k) entries and
// read H through chunk images instead of H:
// img1 = images of H, img2 = images of 2H (block steps; may equal img1 otherwise);
// ordered plans: FP32 images whatever the storage type.
hipError_t launch_stream(const void* S, int32_t stype, int64_t ld, const void* H, int h_f64, int64_t k,
                         void* part, int acc_f64, const PlanView& plan, hipStream_t stream,
                         const void* img1 = nullptr, const void* img2 = nullptr,
                         const AdmmInverse& inv = AdmmInverse());
// 32-bit words of the H images of all n_chunks chunks for this storage type and rank
int64_t h_image_words(int32_t stype, int64_t k, int64_t n_chunks);
// Write the images of chunks [chunk0, chunk0 + n_chunks) of wt * H (FP32, 256 rows x k per chunk,
// rows ldh apart, 0 = k; img: those of all chunks), zero past column k.
hipError_t launch_h_image(const float* H, int32_t stype, int64_t k, int64_t chunk0, int64_t n_chunks, float wt,
                          uint32_t* img, hipStream_t stream, int64_t ldh = 0);
// product of FP32 S with 80 columns at once, 64 of X and 16 of X2 (rows 64 apart), on a tall full
// plan; partial rows of 80 entries; img: wide_image_words
constexpr int WIDE_COLS = 80;
int64_t wide_image_words(int64_t n_chunks);
hipError_t launch_stream_wide(const void* S, const float* X, const float* X2, uint32_t* img, float* part,
                              const PlanView& plan, hipStream_t stream);
// out (rows x k, row stride ldo) = the dense product from the partials of a full pass (float or
// double, rows of kp); FP8: / scale + diag X, X the streamed factor's rows of this panel (stride ldo)
template <typename T>
hipError_t launch_dense_rows(const T* part, int64_t rows, int64_t k, int64_t kp, const PlanView& plan, const T* X,
                             int64_t ldo, const float* scale, const float* diag, int64_t panel_rows, T* out,
                             hipStream_t stream);
hipError_t launch_copy_probe(const void* src, void* dst, int64_t bytes, hipStream_t stream);
// plain read of bytes (multiple of 16); sink: sink_words words (>= 4), one per wave
hipError_t launch_read_probe(const void* src, int64_t bytes, uint32_t* sink, int64_t sink_words,
                             hipStream_t stream);
// Objective pass on the MFMA path: FP32 sums within each 256-column chunk,
// FP64 across chunks; FP64 partials.  img: chunk images of FP32 H.
int stream_acc64_supported(int32_t stype, int64_t k);
hipError_t launch_stream_acc64(const void* S, int32_t stype, int64_t k, const void* img, double* part,
                               const PlanView& p, hipStream_t stream);
// Objective pass at any rank: FP64 products and sums of tiled S with FP32 H (rows of k, padded to
// whole chunks); FP64 partials of a full plan, rows of k.
hipError_t launch_stream_f64_tiled(const void* S, int32_t stype, const float* H, int64_t k, double* part,
                                   const PlanView& p, hipStream_t stream);
int stream_uses_mfma(int32_t stype, int h_f64, int acc_f64, int64_t k);
// resident work-groups per CU of the stream kernel for this storage and rank
int stream_wgs_per_cu(int32_t stype, int64_t k);
// whether full steps of this storage and rank run the tall (8-wave) kernel
int stream_tall_supported(int32_t stype, int h_f64, int64_t k);
// work-groups w of a full step that runs the quarter-tile kernel (a plan with quarter = 1), or 0
// where the step has too many units for it
int32_t stream_quarter_wgs(int cus, int32_t stype, int64_t n_tiles, int64_t n_chunks, int64_t k);

// plan.hip: build the device plan of a sub-sampled step.
struct PlanRequest {
    int32_t mode;            // 1 = row SVRG (I only), 2 = block SVRG
    int32_t n_tiles, n_chunks, tiles_per_block, chunks_per_block, n_blocks;
    int32_t m;               // sampled blocks per set
    int32_t independent;
    uint64_t seed;
    int64_t t;
};
hipError_t launch_plan(const PlanRequest& r, int32_t* plan_base, hipStream_t stream);

struct UpdateArgs {
    int64_t rows, rows_pad, n, k;           // panel rows, padded rows, instruments, rank
    int64_t row0;                           // global row of panel row 0
    int32_t method, softplus;
    double eta, eps, alpha, mu;
    const void* H;        // H_t   (n_pad x k, global rows)
    void* Hn;             // H_{t+1}
    void* G;              // AdaGrad G / RMSprop v   (rows_pad x k, panel rows)
    void* M;              // RMSprop momentum
    void* Theta;          // softplus parameter
    void* Mu;             // snapshot gradient (SVRG), may be null
    void* Gout;           // gradient of this step, may be null
    const void* part;     // S.H partials
    int64_t kp;           // row stride of the partials: mfma_width(k) or k
    const void* gram_eff; // [3][k][k] effective Gram per class (state precision)
    double cgrad;         // 4 (full / row steps) or 2 (block steps)
    int32_t store_mu;     // full SVRG step: mu <- g
    int32_t fp8;          // FP8 storage: scale partials, add the diagonal back
    int32_t block_step;   // Block-SVRG sampled step: the diagonal term S_ii h_i carries the
                          // weight of column i's chunk for the row's class (0, 0, 2)
    const float* panel_scale;
    const float* diag;    // FP8: S_ii of every panel row
    int64_t panel_rows;   // below 2^31 (clamped)
    double* tile_gram;    // [tiles][k][k] Gram of H_{t+1} rows
    double* tile_tr;      // [tiles] sum H_t * SH_t
    double* tile_kkt;     // [tiles] sum proj(g)^2
    int32_t* tile_bad;    // [tiles] non-finite gradient count
    void* img1;           // chunk images of H_{t+1} to bring up to date (null: none), of 2 H_{t+1}
    void* img2;           // in img2 (may be null); row0 is then a multiple of 64
    int32_t img_kind;     // 0 FP32 S, 1 BF16, 2 FP8
    int64_t n_chunks;     // column chunks of S
    double rho;           // ADMM consensus penalty
    void* minv;           // ADMM: (2 W^T W + rho I)^-1, k x k (state precision)
    double beta1, beta2, beta3;   // Adam / NAdam / Adan decays
    double bc1, bc2, bc3;         // 1 - beta^(t+1): bias corrections of this step
    int32_t first;                // first step (Adan: zero gradient difference)
    void* D;              // Adan average of gradient differences
    void* Gp;             // Adan previous gradient
};
hipError_t launch_update(const UpdateArgs& a, int h_f64, const PlanView& plan, hipStream_t stream);
// ADMM step (full plans): the k x k inverse from the FP64 Gram of W_t, then the
// fused statistics + H / W / U update (a.M holds U).
hipError_t launch_admm(const UpdateArgs& a, const double* gram64, int h_f64, const PlanView& plan,
                       hipStream_t stream);

// Per-slice FP64 Gram partials (SUBT per tile) of rows [row0, row0 + tiles*TR) of H.
hipError_t launch_tile_gram(const void* H, int h_f64, int64_t row0, int64_t rows, int64_t tiles, int64_t k,
                            double* tile_gram, hipStream_t stream);
// FP64 Gram of the rows of [0, n) outside [skip_lo, skip_hi).
hipError_t launch_gram_rows(const void* H, int h_f64, int64_t n, int64_t skip_lo, int64_t skip_hi, int64_t k,
                            double* out, hipStream_t stream);

// Reduce tile partials: Gram_{t+1} (gram_next64, and gram_eff = 3 copies in
// state precision), and the statistics of H_t: stats[0] = tr(H^T S H),
// [1] = ||grad_proj||^2, [2] = non-finite count, [3] = ||Gram_t||_F^2.
hipError_t launch_finalize(int64_t tiles, int64_t k, const double* tile_gram, const double* tile_tr,
                           const double* tile_kkt, const int32_t* tile_bad, const double* gram_fixed,
                           const double* gram_cur64, double* gram_next64, void* gram_eff, int h_f64,
                           double* stats, hipStream_t stream);

// Effective Gram matrices of a block step: out[0] = Gram_J, out[1] = Gram_I,
// out[2] = Gram_I + Gram_J from the per-slice Gram partials of H_t and the
// classes of the plan's tiles.
hipError_t launch_gram_select(int64_t k, const double* tile_gram, const PlanView& plan, void* gram_eff, int h_f64,
                              hipStream_t stream);

hipError_t launch_init_H(float* H, int64_t n, int64_t k, uint64_t seed, float scale, hipStream_t stream);
hipError_t launch_copy_h(const void* src, int src_f64, void* dst, int dst_f64, int64_t count, hipStream_t stream);
// Zero `bytes` bytes at p on `stream` with a kernel (no memset node).
hipError_t launch_zero(void* p, int64_t bytes, hipStream_t stream);
hipError_t launch_softplus_init(void* H, void* Theta, int h_f64, int64_t count, hipStream_t stream);
hipError_t launch_sum(const void* x, int x_f64, int64_t m, double* out, hipStream_t stream);
hipError_t launch_piecewise_apply(void* G, const void* g, int h_f64, int64_t m, double c, const double* med,
                                  hipStream_t stream);

// select.hip: element number ``rank`` (0-based, ascending) of the keys x_i^2
// (square = 1) or x_i (square = 0; x_i >= 0 required) over m values, by an
// MSB-first radix selection on the IEEE bit patterns (monotone for
// non-negative values).  The value goes to out_dev[0] (double).  tmp: device
// scratch of select_tmp_bytes().
int64_t select_tmp_bytes();
// the histogram counters are 32-bit: at most 2^32 - 1 values per selection
constexpr int64_t SELECT_MAX_M = 0xffffffffll;
hipError_t launch_select(const void* x, int x_f64, int square, int64_t m, int64_t rank, void* tmp,
                         double* out_dev, hipStream_t stream);

// Allocation-free entry points: the device address of the file-scope scratch
// array of select.hip on ``device``.  noalloc_scratch_init (device current)
// looks it up once per device; noalloc_scratch returns it (null and *err set
// when the lookup failed or was never made).
constexpr int64_t NOALLOC_SCRATCH_BYTES = 4096;
hipError_t noalloc_scratch_init(int device);
void* noalloc_scratch(int device, hipError_t* err);

// build_s.hip
struct BuildOut {
    void* data; float* scale; float* diag;
    int64_t rows, rows_pad, ld, n, row0; int32_t dtype; int64_t panel_rows;
};
// Flag bits set by the input checks of the S build: a non-finite X entry, a
// negative entry where raw TPDM marginals need X >= 0; the low bits count
// zero-variance columns.
constexpr int32_t BAD_NONFINITE = 1 << 30;
constexpr int32_t BAD_NEGATIVE = 1 << 29;
// zeros in columns n .. ldz - 1 of rows < K and in rows K .. Kpad - 1 of Z (words 32-bit words per element)
hipError_t launch_zero_pads(void* Z, int64_t K, int64_t Kpad, int64_t n, int64_t ldz, int words, hipStream_t stream);
hipError_t launch_standardise(const float* X, int64_t T, int64_t n, void* Z, int z_f64, int64_t ldz, int32_t* bad,
                              hipStream_t stream);
// TPDM: Omega (n_exc x ldz, FP32 or FP64) = column-normalised angular rows; raises the input
// check's bits in *flag.
hipError_t launch_tpdm_omega(const float* X, int64_t T, int64_t n, int lower, int raw, void* Omega, int z_f64,
                             int64_t ldz, int64_t n_exc, void* work, int32_t* flag, hipStream_t stream);
int64_t tpdm_work_bytes(int64_t T, int64_t n, int64_t n_exc, int raw);
// sums: device FP64 array of syrk_sum_words(o) words; [0..2] = sum S, sum S^2,
// sum S_stored^2 on return.  panel_max: FP8 only, zeroed, one word per panel.
int64_t syrk_sum_words(const BuildOut& o);
hipError_t launch_syrk_store(const void* Z, int z_f64, int64_t K, int64_t ldz, const BuildOut& o, double* sums,
                             uint32_t* panel_max, hipStream_t stream);
// The same product for BF16 / FP8 storage on the bf16 matrix cores with Z
// split into two bf16 planes; ws holds the planes (syrk_split_ws_bytes).
// Z: Kpad x ldz FP32 with K valid rows.
int64_t syrk_split_ws_bytes(int64_t K, int64_t ldz);
hipError_t launch_syrk_split_store(const float* Z, int64_t K, int64_t ldz, const BuildOut& o, double* sums,
                                   uint32_t* panel_max, void* ws, hipStream_t stream);
// sums: 4 + 3 * rows_pad words
hipError_t launch_store_dense(const void* src, int src_f64, const BuildOut& o, double* sums,
                              uint32_t* panel_max, hipStream_t stream);
hipError_t launch_fp8_decode_check(int32_t* bad, hipStream_t stream);
// objective pass: per-slice tr(H^T S H) partial and Gram of H (FP32 or FP64 H, FP64 partials of
// a full plan).
hipError_t launch_objective_tiles(const UpdateArgs& a, int h_f64, const PlanView& plan, hipStream_t stream);

// warmstart.hip
hipError_t launch_omega(uint64_t seed, int64_t n, int64_t rows_alloc, int w, float* out, hipStream_t stream);
// C = op(A) op(B) + bias with epilogue (0 none, 1 GELU, 2 softplus, 3 max(aux + x, 0), 4 x GELU'(aux)
// with FP64 column sums over every 64 rows in part, gemm_row_blocks(M) x N); aux: M x N, rows ldaux
// apart; Z: pre-epilogue copy or null.  splits > 1 (a value of gemm_splits; no bias, epilogue or
// Z): C holds that many M x N partials, one per range of K.
hipError_t launch_gemm(int ta, int tb, int b_bf16, int epi, const float* A, const void* B, const float* bias, float* C,
                       float* Z, int64_t M, int64_t N, int64_t K, int64_t splits, hipStream_t stream,
                       const float* aux = nullptr, int64_t ldaux = 0, double* part = nullptr);
int64_t gemm_splits(int64_t M, int64_t N, int64_t K);
// the most gemm_splits returns for any reduction length up to K
int64_t gemm_max_splits(int64_t M, int64_t N, int64_t K);
int64_t gemm_row_blocks(int64_t M);
// Partials of the parameters' gradient: weights (W1, W2, W3) as split-K partials, biases (b1, b2,
// b3) as FP64 row-block sums.
struct GradParts {
    const float* wpart[3];
    int64_t wsize[3], splits[3];
    const double* bpart[3];
    int64_t bsize[3], bblocks[3];
};
// G = summed partials, then AdamW step t (1, 2, ...), unless coef[3] != 0
hipError_t launch_grad_adamw(const GradParts& gp, const double* coef, float* P, float* G, float* M, float* V, float lr,
                             float b1, float b2, float eps, float wd, int64_t t, hipStream_t stream);
hipError_t launch_to_bf16(const float* x, uint16_t* y, int64_t m, hipStream_t stream);
// successive projection on R (k columns of m FP64, destroyed); pick: k device int64; bval/bidx: 2 nb entries
hipError_t launch_spa(double* R, int64_t m, int64_t k, double* bval, int64_t* bidx, int nb, int64_t* pick,
                      hipStream_t stream);
int64_t xty_work_doubles(int64_t m, int64_t kx, int64_t ky);
hipError_t launch_xty(const float* X, int64_t ldx, int64_t kx, const float* Y, int64_t ldy, int64_t ky, int64_t m,
                      double* work, double* out, hipStream_t stream);
hipError_t launch_jacobi_topk(const double* G, int64_t w, int64_t k, double* M, double* lam, int32_t* status,
                              hipStream_t stream);
hipError_t launch_project_rows(const float* Y, int64_t m, int64_t w, const double* W, int64_t k, int64_t ldo,
                               int out_f64, void* out, hipStream_t stream);
hipError_t launch_anchor_solve(const float* Y, int64_t w, const double* M, int64_t k, const int64_t* anchors,
                               double* W, int32_t* status, hipStream_t stream);
hipError_t launch_gram3(const float* A, const float* B, int64_t k, int64_t m, double* work, double* out,
                        hipStream_t stream);
hipError_t launch_loss_coef(const double* gram3, int64_t k, int kind, double* coef, hipStream_t stream);
// part: loss_backward_blocks(m) x k FP64 column sums of dZ
hipError_t launch_loss_backward(const float* A, const float* B, const double* gram3, const double* coef, const float* X,
                                int64_t ldx, const float* Z, int residual, int64_t k, int64_t m, float* dZ, double* part,
                                hipStream_t stream);
int64_t loss_backward_blocks(int64_t m);
hipError_t launch_clip_cols(const float* X, int64_t m, int64_t w, int64_t k, float* out, hipStream_t stream);
hipError_t launch_scale(float* x, int64_t m, float a, hipStream_t stream);
hipError_t launch_span_overlap(const double* MA, const double* AtB, const double* MB, int64_t k, double* out,
                               hipStream_t stream);

}  // namespace symnmf
