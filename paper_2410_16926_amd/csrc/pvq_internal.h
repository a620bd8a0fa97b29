// Internal interface between the host side of libpvq (argument checks, size tables, context) and
// its kernels.  Not installed; the public contract is include/pvq.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>
#include <stdint.h>

#include "pvq.h"
#include "pvq_fast8.h"

// Tables of the coordinate-by-coordinate decoder (pvq_walk.hip), one blob copied to LDS by every workgroup behind the
// amplitude table: a guess row of bytes per d' = D-1 .. 2, then the rows of thresholds T_j (below) for d' = D-1 .. 2, each
// in the width of its dimension's arithmetic, with an entry of all ones behind T_{2K+1}, padded to a multiple of 16
// bytes.  Where a row lies follows from the schedule (known when the kernels are compiled) and three sizes
// (pvq_walk.h: guess_row, row_bytes).
struct pvq_walk_params {
    uint32_t bytes;         // of the blob, the amplitude table in front included (a multiple of 16)
    int K;
    int dX, dA, dB;         // the width schedule: dimensions above dX in `words` words, above dA in three quarters of them (of two: as doubles), above dB in half, the rest in a quarter
    uint32_t more;          // bit DP: some bucket of row DP holds more than one threshold besides its guess
    uint32_t part_bytes[3]; // bytes of a row with entries of 4, 8 and 16 bytes (a row of 12-byte entries: the first two)
    uint32_t last_index[4]; // N(D,K) - 1
};

// A multi-word integer (w[0] the lowest word) as 32 bits that order like the integer wherever they differ: its
// bit length in the upper 10 bits, below them the 22 leading bits (0 for 0).  key(a) < key(b) implies a < b;
// equal keys decide nothing.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline uint32_t pvq_wide_key(const uint32_t *w, int words)
{
    uint32_t hi = 0, lo = 0;
    int t = -1;
    for (int i = 0; i < words; i++)
        if (w[i] != 0) { t = i; hi = w[i]; lo = i > 0 ? w[i - 1] : 0u; }
    if (t < 0) return 0;
    const int lead = __builtin_clz(hi);
    const uint32_t top = lead ? (hi << lead) | (lo >> (32 - lead)) : hi;
    return ((uint32_t)(32 * t + 32 - lead) << 22) | (top >> 10);
}

// A multi-word integer as a float64 that orders like the integer wherever they differ: its highest word that is not
// zero and the one below, rounded to nearest (the same for every integer, so equal values decide nothing).
inline double pvq_wide_double(const uint32_t *w, int words)
{
    int t = words - 1;
    while (t > 0 && w[t] == 0) t--;
    return ldexp((double)w[t] * 4294967296.0 + (t > 0 ? (double)w[t - 1] : 0.0), 32 * t - 32);   // (the product is exact)
}

// Thresholds.  With U(d,x) = N(d,0) + ... + N(d,x) and q = N(d,k) - 1 - r for the residual r in the
// sub-pyramid of d dimensions and k pulses, the points that leave C pulses to the d - 1 coordinates behind lie at
//     2 U(d-1,C-1) <= q < 2 U(d-1,C),
// the negative ones (q - 2 U(d-1,C-1) < N(d-1,C)) first; C = k, the magnitude 0, has that half only.  So row d - 1 is
// one ascending sequence of thresholds
//     T_{2C} = 2 U(d-1,C-1),  T_{2C+1} = T_{2C} + N(d-1,C),      C = 0 .. K,
// a coordinate of the point is its position j in it (C = j / 2 pulses left, positive iff j is odd), the next q is
// q - T_j, and after the last coordinate q = 0.  Hence N(D,K) - 1 - index = the sum of the thresholds of all
// coordinates: an encoder adds them up, a decoder finds them one after the other.
// Contexts with D = 64 or 128: rows are at least as long as the windows of 64 that a decoder reads, with all ones behind the thresholds.
inline int pvq_wide_row(int K) { return K < 31 ? 64 : 2 * K + 2; }
inline int pvq_wide_key_row(int K) { return 2 * K + 2 + 6 + 3 & ~3; }   // (whole pieces of 16 bytes)
// The other decoder's first guess: keys by bit length and the three bits behind the leading one (their bits 18 to 31, less 21).
inline int pvq_wide_buckets(int words) { return (32 * words + 1) * 8; }

// The D = 8 / 24-bit encoder's offsets: [7][PVQ_ENC8_MAX_K + 1][2 PVQ_ENC8_MAX_K + 1] words: coordinate, pulses left, value +
// PVQ_ENC8_MAX_K.  K is 15 or 16 with 24-bit indices.
constexpr int PVQ_ENC8_MAX_K = 16;
constexpr int PVQ_ENC8_WORDS = 7 * (PVQ_ENC8_MAX_K + 1) * (2 * PVQ_ENC8_MAX_K + 1);

struct pvq_ctx {
    int D, K;
    int index_bits;
    int words;       // 32-bit words of one table entry / one index in registers: 1, 2 or 4 (wide: 4..16)
    int wide;        // 1: D = 64 or 128; kernels in pvq_wide.hip
    int scale_bits;  // 0 = float32 amplitudes
    int device;
    // Device tables.  Entries are `words` little-endian 32-bit words.
    //   tab_u[dp][k+1] = sum_{i=0..k} N(dp, i), tab_u[dp][0] = 0,  dp = 0..D-1, k = -1..K  (cumulative form of
    //                    App. C.2's V table, shifted so that the empty sum is an entry)
    //   wide: tab_u[dp][j] = T_j of row dp, j = 0 .. 2K+1 (rows of pvq_wide_row entries); tab_key[dp][j] = pvq_wide_key of it
    //         (rows of pvq_wide_key_row words); tab_guess[dp][bucket] = the last j whose key lies below the bucket
    uint32_t *tab_u;
    const uint32_t *tab_key;   // (this and the next two: behind the thresholds, in tab_u's allocation)
    const uint16_t *tab_guess;
    const double *tab_near;    // wide: pvq_wide_double of tab_u's entries (behind a row's thresholds: infinity)
    uint32_t last_index[16];   // N(D,K) - 1
    float *edges;   // 2^scale_bits - 1 float32 edges (or nullptr)
    float *sqrtc;   // 2^scale_bits float32 sqrt(centers) (or nullptr)
    // Table-driven decoder (D = 8, one-word indices, tables that fit LDS); fast8_blob == nullptr
    // when the configuration has none.
    unsigned char *fast8_blob;
    pvq_fast8_params fast8;
    // Coordinate-by-coordinate decoder's tables (every context with D <= 32); nullptr if they were not made.
    unsigned char *walk_blob = nullptr;
    pvq_walk_params walk;
    int amplitude;   // PVQ_AMP_NORM or PVQ_AMP_LS
    // Per-coordinate index offsets for the D = 8 / 24-bit encoder (PVQ_ENC8_WORDS words, padded to a multiple of 16 bytes);
    // nullptr when the configuration has none.
    uint32_t *enc8_offs;
};

struct pvq_encode_args {
    int ls_amplitude;   // 1: least-squares amplitudes instead of norms
    const void *W;
    int64_t rows, cols, ldw, groups;
    uint32_t *index_out;
    void *scale_out;
    float *rownorm_out;
    int8_t *pulses_out;
    int64_t index_row_words, scale_row_words;
};

struct pvq_decode_args {
    const uint32_t *index;
    const void *scale;
    const float *rownorm;
    int64_t rows, cols, groups;
    int64_t index_row_words, scale_row_words;
    void *W_out;
    int64_t ldw;
    const void *x;  // gemv only
    int batch;
    int64_t ldx;
    float *y;
    int64_t ldy;
};

// Each returns a hipError_t from the launch (hipSuccess if enqueued).
// false: a row's share of LDS (size table, and with amplitude codes the row's amplitudes) exceeds 64 KB
bool pvq_encode_fits(const pvq_ctx *ctx, const pvq_encode_args &a);
hipError_t pvq_launch_encode(const pvq_ctx *ctx, const pvq_encode_args &a, int dtype, hipStream_t s);

hipError_t pvq_launch_fill_zero(float *p, int64_t n, hipStream_t s);   // p[0..n) = 0 by a kernel

// error correction of Sec. 3.3 Step 6 (pvq_correct.hip): W rows x cols float32 in place, cols a multiple
// of 64, U cols x cols upper triangular, work 2 x rows x 128 floats (the t values of two panels, used in turn)
hipError_t pvq_launch_correct(const pvq_ctx *ctx, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                              int64_t ldu, float *work, hipStream_t s);
// the same with work of 4 x rows x 128 floats: two panels a launch where that is faster
hipError_t pvq_launch_correct_two_panels(const pvq_ctx *ctx, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                                         int64_t ldu, float *work, hipStream_t s);
// the same with the library's static work buffer (at most pvq_correct_static_max_rows() rows), on `s` alone
int64_t pvq_correct_static_max_rows(void);
hipError_t pvq_launch_correct_static(const pvq_ctx *ctx, float *W, int64_t rows, int64_t cols, int64_t ldw,
                                     const float *U, int64_t ldu, hipStream_t s);

// size table on the GPU (pvq_size_table.hip): (D+1) x (K+1) entries of `words` words, one workgroup
hipError_t pvq_launch_size_table(int D, int K, int words, uint32_t *table, uint32_t *overflow, hipStream_t s);

// randomised Hadamard rotation of rows (pvq_hadamard.hip); arguments already validated
hipError_t pvq_launch_hadamard(const void *X, int in_dtype, int64_t rows, int64_t cols, int64_t ldx, int block,
                               const uint8_t *signs, int signs_after, void *Y, int out_dtype, int64_t ldy,
                               hipStream_t s);

// groups of 64 / 128 values, indices of up to 512 bits (pvq_wide.hip); for contexts with wide == 1
hipError_t pvq_wide_launch_encode(const pvq_ctx *ctx, const pvq_encode_args &a, int dtype, hipStream_t s);
hipError_t pvq_wide_launch_decode(const pvq_ctx *ctx, const pvq_decode_args &a, int out_dtype, hipStream_t s);
// rotation of rows (blocks of `block` values, optional signs) and encoding in one kernel; D = 128, words <= 12
hipError_t pvq_wide_launch_rotate_encode(const pvq_ctx *ctx, const pvq_encode_args &a, int dtype, int block,
                                         const uint8_t *signs, hipStream_t s);

// coordinate-by-coordinate decoder with one table probe per coordinate (pvq_walk.hip)
bool pvq_walk_usable(const pvq_ctx *ctx);
hipError_t pvq_walk_launch_decode(const pvq_ctx *ctx, const pvq_decode_args &a, int out_dtype, hipStream_t s);
// tile_rows: 4, 8 (up to 8 vectors) or 16 rows a tile, or 0 for the split that should take least
hipError_t pvq_walk_launch_gemv(const pvq_ctx *ctx, const pvq_decode_args &a, int tile_rows, hipStream_t s);

// D = 8 / 24-bit encoder (pvq_encode8.hip)
bool pvq_encode8_usable(const pvq_ctx *ctx, const pvq_encode_args &a);
hipError_t pvq_encode8_launch(const pvq_ctx *ctx, const pvq_encode_args &a, int dtype, hipStream_t s);
// ... with the rotation of the rows (blocks of `block` values, optional signs) fused in front
bool pvq_rotate_encode8_usable(const pvq_ctx *ctx, const pvq_encode_args &a, int block);
hipError_t pvq_rotate_encode8_launch(const pvq_ctx *ctx, const pvq_encode_args &a, int dtype, int block,
                                     const uint8_t *signs, hipStream_t s);

// D = 8 table-driven kernels (pvq_fast8.hip).  `*_usable` says whether the shape qualifies, `*_pays` whether it is theirs.
bool pvq_fast8_decode_usable(const pvq_ctx *ctx, const pvq_decode_args &a);
bool pvq_fast8_gemv_usable(const pvq_ctx *ctx, const pvq_decode_args &a);
bool pvq_fast8_gemv_pays(const pvq_ctx *ctx, const pvq_decode_args &a);
hipError_t pvq_fast8_launch_decode(const pvq_ctx *ctx, const pvq_decode_args &a, int out_dtype, hipStream_t s);
hipError_t pvq_fast8_launch_gemv(const pvq_ctx *ctx, const pvq_decode_args &a, hipStream_t s);
// The passes of a fused product: which kind of kernel takes how many vectors (a batch of up to 16 vectors
// is at most 16 passes).  pvq_fast8_plan_gemv fills out[] and returns the number of passes.
enum {
    PVQ_PASS_GENERIC = 0,     // pvq_walk.hip: coordinate-by-coordinate decoder, one pass per call, dot products on the matrix cores
    PVQ_PASS_VALU = 1,        // gemv8_kernel: 1, 2 or 4 vectors, float32 multiply-adds on the vector ALU (by rule 4 only below 4096 groups)
    PVQ_PASS_VALU_ROWS = 2,   // gemv8_row_kernel: one vector, every wave owns whole rows
    PVQ_PASS_MFMA = 4,        // gemv8_mfma_kernel: 3..16 vectors, the groups' dot products on the matrix cores
};
struct pvq_gemv_pass { int kind, nvec; };
int pvq_fast8_plan_gemv(const pvq_ctx *ctx, const pvq_decode_args &a, pvq_gemv_pass *out);
hipError_t pvq_fast8_prepare(void);  // one-time device queries
