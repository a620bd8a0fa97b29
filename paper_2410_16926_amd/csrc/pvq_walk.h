// The coordinate-by-coordinate decoder with one table probe per coordinate: its step, shared by the kernels
// (pvq_walk.hip, which explains the method) and by a host replay that checks the tables.
#pragma once

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "pvq_fast8.h"      // PVQ_HD
#include "pvq_internal.h"   // pvq_walk_params

namespace pvq_walk {

PVQ_HD uint32_t float_bits(float f)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __float_as_uint(f);
#else
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
#endif
}

PVQ_HD float bits_float(uint32_t u)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __uint_as_float(u);
#else
    float f;
    memcpy(&f, &u, 4);
    return f;
#endif
}

template <int W> struct wide;
template <> struct wide<1> { using type = uint32_t; };
template <> struct wide<2> { using type = uint64_t; };
template <> struct wide<4> { using type = unsigned __int128; };

// ---- layout of the blob (shared with the host builder) ---------------------------------------------------
// Words of row DP's integers under the schedule (D, W, DX, DA, DB): dimensions (DP + 1 are left) above DX in W words,
// above DA in three quarters (of two words: in both, as doubles), above DB in half of them, the rest in a quarter.
constexpr int words_of_row(int dp, int W, int DX, int DA, int DB) { return dp >= DX ? W : dp >= DA ? (W == 2 ? 2 : 3 * W / 4) : dp >= DB ? W / 2 : W / 4; }
// Whether row DP keeps q + 1/2 and the thresholds as doubles (exact: q < 2^52), scaled by kDoubleUnit.
constexpr bool double_row(int dp, int W, int DX, int DA) { return W == 2 && dp < DX && dp >= DA; }
// the scale: 1/2, the least q + 1/2, gets the exponent that 1 has as a float, and the buckets start where those of floats do
constexpr double kDoubleUnit = 0x1p-895;
// Fraction bits of guess row DP, chosen so that a bucket of q holds one threshold besides the one its guess stands for
// (the rows of few dimensions grow slowly and get finer buckets).  Enough for every K of the schedules
// that have no search behind the guess (searches); with the others pvq_walk_params::more says for which rows they are not.
constexpr int guess_bits(int dp, int D)
{
    return D == 32 ? (dp == 2 ? 6 : dp <= 5 ? 5 : dp <= 13 ? 4 : 3) : dp == 2 ? 5 : dp <= 10 ? 4 : 3;
}
constexpr bool searches(int D, int W, int DX, int DA) { return DA == 0 ? W == 4 || (W == 2 && D <= 16) : W == 4 && DX == DA; }
// Whether a coordinate reads entry j + 1 from entry j's address (walk_step's NEXT): two vector instructions a coordinate less,
// a few registers more, since both reads are one.  Decoding, with integers of up to two words, it takes less time or the same.
// In the products the registers decide how many workgroups a unit holds, and with them the split (us, two addresses / one):
//  - groups of 8 and 16 without the search behind the guess: as many waves either way, and 0 to 7 % faster (D = 16, K = 33:
//    28672 x 8192 times five vectors 121 / 114, 14336 x 4096 times one 29.9 / 29.0);
//  - not with the search: tiles of 16 rows take more than 64 registers then (28672 x 8192 times five vectors, D = 16, K = 45:
//    141 / 174, K = 58: 148 / 195);
//  - groups of 32: tiles of 16 rows, which are held to 64 registers (gemv_waves; 8192 x 14336 times five, K = 4: 61 / 49; without
//    the bound seven waves or five, 54, and 28672 x 8192, K = 14, 105 / 123), and with two words those of four (8192 x 14336
//    times one, K = 8: 56.0 / 50.7); with one word the kernel for 5 to 8 vectors in tiles of four would lose a wave
//    (3001 x 11008, K = 4: 20.8 / 27.8);
//  - with four words one read of both comes back later than two (groups of 32, 104 bits, to bfloat16: 45.9 / 47.6).
constexpr uint32_t next_from_decode(int W) { return W <= 2 ? 1 : 0; }
constexpr uint32_t next_from_product(int D, int W, int DX, int DA, int R)
{
    return W <= 2 && !searches(D, W, DX, DA) && (D <= 16 || W == 2 || R == 16) ? 1 : 0;
}
// entries of guess row DP: every value of the row's integer type lands inside (up to 2^(32 words), where the largest round to)
constexpr uint32_t guess_entries(int dp, int D, int words) { return ((uint32_t)(32 * words) << guess_bits(dp, D)) + 1u; }
// The guess of bucket b of row DP lies at byte guess_offset(DP) + b.  Buckets are floats shifted down, of which 1 is the
// smallest, so b starts at 127 << guess_bits, and the rows follow one another from the highest dimension, the coarsest,
// on (the lower ones start far enough behind the amplitude table in front for the offset to be a plain
// immediate: a row never starts below its 127 << guess_bits).
constexpr uint32_t kWalkHead = 1024;               // the amplitude table, 256 floats
constexpr uint32_t guess_row(int dp, int D, int W, int DX, int DA, int DB)
{
    uint32_t at = kWalkHead;
    for (int j = D - 1; j >= dp; j--) {
        const uint32_t least = 127u << guess_bits(j, D);
        at = at < least ? least : at;
        if (j > dp) at += guess_entries(j, D, words_of_row(j, W, DX, DA, DB));
    }
    return at;
}
// end of the guess rows, where the thresholds start
constexpr uint32_t threshold_base(int D, int W, int DX, int DA, int DB)
{
    return (guess_row(2, D, W, DX, DA, DB) + guess_entries(2, D, words_of_row(2, W, DX, DA, DB)) + 15u) / 16u * 16u;
}
// Rows of thresholds follow in the order DP = D-1 .. 2, each of 2K + 3 entries, padded to 16 bytes; rows of three words
// in two parts, the lower two words of all entries in front of the third ones.
// bytes of a row
PVQ_HD uint32_t row_bytes(const pvq_walk_params &p, int words)
{
    return words == 1 ? p.part_bytes[0] : words == 2 ? p.part_bytes[1] : words == 3 ? p.part_bytes[0] + p.part_bytes[1] : p.part_bytes[2];
}

// q (its lowest bit set, so that it is not zero) as a float: each operation rounds to nearest, which the builder of the
// guess rows allows for.
template <int WP>
PVQ_HD float float_of(const uint32_t *q)
{
    float f = (float)(WP == 1 ? q[0] | 1u : q[WP - 1]);
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
    for (int x = WP - 2; x >= 0; x--) f = fmaf(f, 4294967296.0f, (float)(x == 0 ? q[0] | 1u : q[x]));
    return f;
}

// d = a - b over WP words; returns the borrow
template <int WP>
PVQ_HD uint32_t subtract(uint32_t *d, const uint32_t *a, const uint32_t *b)
{
    uint32_t borrow = 0;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
    for (int x = 0; x < WP; x++) d[x] = __builtin_subc(a[x], b[x], borrow, &borrow);
    return borrow;
}

PVQ_HD uint32_t double_high(double v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__double2hiint(v);
#else
    uint64_t u;
    memcpy(&u, &v, 8);
    return (uint32_t)(u >> 32);
#endif
}

// One of a row's entries, or a guess, at a byte of the tables: LDS address in a kernel, where they start at 0 (the launch
// checks it; an address formed from the array's name would be an addition more).
template <typename T>
PVQ_HD T table_at(const unsigned char *tables, uint32_t byte)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(byte);
#else
    T v;
    memcpy(&v, __builtin_assume_aligned(tables + byte, sizeof(T)), sizeof(T));
    return v;
#endif
}
typedef uint32_t word4 __attribute__((vector_size(16)));

// entry j + NEXT of the row of thresholds at byte `at`  (NEXT is part of the instruction: entry j and the one behind it are
// two offsets from one address)
template <int WP, uint32_t NEXT = 0>
PVQ_HD void threshold(const unsigned char *tables, const pvq_walk_params &p, uint32_t at, uint32_t j, uint32_t *t)
{
    if constexpr (WP == 1) t[0] = table_at<uint32_t>(tables, (at + 4u * j) + 4u * NEXT);
    if constexpr (WP == 2 || WP == 3) {
        const uint64_t v = table_at<uint64_t>(tables, (at + 8u * j) + 8u * NEXT);
        t[0] = (uint32_t)v; t[1] = (uint32_t)(v >> 32);
    }
    if constexpr (WP == 3) t[2] = table_at<uint32_t>(tables, (at + p.part_bytes[1] + 4u * j) + 4u * NEXT);
    if constexpr (WP == 4) {
        const word4 v = table_at<word4>(tables, (at + 16u * j) + 16u * NEXT);
        t[0] = v[0]; t[1] = v[1]; t[2] = v[2]; t[3] = v[3];
    }
}

// The coordinate of row DP (DP + 1 dimensions left), whose thresholds start at byte `at`: its place j in them
// (pvq_internal.h).  q loses T_j.  NEXT: 1 if the second threshold is read from the first one's address.
template <int DP, int D, int W, int DX, int DA, int DB, uint32_t NEXT>
PVQ_HD uint32_t walk_step(const unsigned char *tables, const pvq_walk_params &p, uint32_t at, uint32_t more, uint32_t ones, uint32_t *q)
{
    constexpr int WP = words_of_row(DP, W, DX, DA, DB);
    if constexpr (DP == 1) {
        // T = 0, 1, 2, 4, 6, ...
        const uint32_t j = std::min(q[0], (q[0] >> 1) + 1u);
        q[0] = q[0] < 2u ? 0u : q[0] & 1u;
        return j;
    } else {
        constexpr int MB = guess_bits(DP, D);
        constexpr uint32_t guesses = guess_row(DP, D, W, DX, DA, DB) - (127u << MB);
        uint32_t j = table_at<uint8_t>(tables, guesses + (float_bits(float_of<WP>(q)) >> (23 - MB)));
        uint32_t t0[WP], t1[WP], d0[WP], d1[WP];
        threshold<WP>(tables, p, at, j, t0);
        threshold<WP, NEXT>(tables, p, at, j + 1 - NEXT, t1);
        subtract<WP>(d0, q, t0);
        uint32_t borrow = subtract<WP>(d1, q, t1), unused;
        const bool up = !borrow;
        j = __builtin_subc(j, NEXT ? ones : 0xFFFFFFFFu, borrow, &unused);       // j + 1 - borrow
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
        for (int x = 0; x < WP; x++) d0[x] = up ? d1[x] : d0[x];
        if constexpr (searches(D, W, DX, DA)) {
            // A bucket with more thresholds: one read more in nearly every wave, in the rows that have such (in all rows of a
            // context that has one, and in front of the pair, it cost D = 32, K = 80 114 instead of 71 us for 14336 x 4096 to
            // bf16, D = 16, K = 45 71 instead of 50).
            if (more >> DP & 1u) {                                 // (the same for all lanes)
                bool on = up;
                while (on) {                                       // (ends: q lies below the entry behind the thresholds)
                    threshold<WP, NEXT>(tables, p, at, j + 1 - NEXT, t1);
                    on = !subtract<WP>(d1, q, t1);
                    j += on ? 1u : 0u;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
                    for (int x = 0; x < WP; x++) d0[x] = on ? d1[x] : d0[x];
                }
            }
        }
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
        for (int x = 0; x < WP; x++) q[x] = d0[x];
        return j;
    }
}

// walk_step for a row of doubles: no conversion in front of the guess, whose bucket is in q's upper bits as they are, and one
// instruction where integers of two words take two.  v: q + 1/2, never 0, so that a difference's sign tells which is larger.
// 14336 x 4096, D = 16, K = 33, integers / doubles: one vector 27.9 / 27.0 us, 16 vectors 38.9 / 37.3, to bfloat16 35.3 / 34.3 (vector
// instructions of the product 448 / 420).  Groups of 32 with integers of four words keep q in them: the five rows that could have
// doubles (at most 52 bits, more than 32) would save three instructions in a hundred.  Squares by the dot instruction of bfloat16
// pairs instead of a multiply-add each took longer (D = 32, K = 60, one vector 45.4 / 45.7).
template <int DP, int D, int W, int DX, int DA, int DB, uint32_t NEXT>
PVQ_HD uint32_t walk_step_double(const unsigned char *tables, uint32_t at, uint32_t ones, double &v)
{
    constexpr int MB = guess_bits(DP, D);
    constexpr uint32_t guesses = guess_row(DP, D, W, DX, DA, DB) - (127u << MB);
    const uint32_t j = table_at<uint8_t>(tables, guesses + (double_high(v) >> (20 - MB)));
    const double d0 = v - table_at<double>(tables, at + 8u * j);
    const double d1 = v - table_at<double>(tables, (at + 8u * (j + 1u - NEXT)) + 8u * NEXT);
    const uint32_t borrow = !(d1 > 0.0);
    uint32_t unused;
    v = borrow ? d0 : d1;
    return __builtin_subc(j, ones, borrow, &unused);               // j + 1 - borrow
}

// The state of a walk: the residual, pulses left, sum of squares.
template <int D, int W, int DX, int DA, int DB, uint32_t NEXT>
struct walk_state {
    uint32_t q[W];
    uint32_t k, at, more, ones;
    float n2;
    double v;                                                      // in rows of doubles: (q + 1/2) * kDoubleUnit

    template <int I, typename Emit>
    PVQ_HD void coordinate(const unsigned char *tables, const pvq_walk_params &p, Emit &emit)
    {
        constexpr int DP = D - 1 - I;
        uint32_t j;
        if constexpr (double_row(DP, W, DX, DA)) {
            if constexpr (I == 0 || !double_row(DP + 1, W, DX, DA))
                v = fma((double)q[1], kDoubleUnit * 0x1p32, fma((double)q[0], kDoubleUnit, kDoubleUnit * 0.5));
            j = walk_step_double<DP, D, W, DX, DA, DB, NEXT>(tables, at, ones, v);
            if constexpr (!double_row(DP - 1, W, DX, DA)) q[0] = (uint32_t)(v * (1.0 / kDoubleUnit));
        } else {
            j = walk_step<DP, D, W, DX, DA, DB, NEXT>(tables, p, at, more, ones, q);
        }
        at += row_bytes(p, words_of_row(D - 1 - I, W, DX, DA, DB));
        const uint32_t C = j >> 1;
        const float m = (float)(k - C);
        k = C;
        n2 = fmaf(m, m, n2);                                       // (exact: at most K^2 < 2^14)
        emit(I, bits_float(j << 31 | float_bits(m)));
    }
    template <typename Emit, int... Is>
    PVQ_HD void all(const unsigned char *tables, const pvq_walk_params &p, Emit &emit, std::integer_sequence<int, Is...>)
    {
        (coordinate<Is>(tables, p, emit), ...);
    }
};

// The whole point from its index c, negated (the place of a positive coordinate is odd, which becomes a sign bit):
// emit(i, -y_i) for i = 0 .. D-1 in order, +0 where y_i is 0; returns sum y_i^2.  An index that is no codeword decodes as
// the last one.
template <int D, int W, int DX, int DA, int DB, uint32_t NEXT, typename Emit>
PVQ_HD float unrank_walk(typename wide<W>::type c, const unsigned char *tables, const pvq_walk_params &p, Emit &&emit)
{
    static_assert(DX <= D && DA <= DX && DB <= DA, "width schedule");
    walk_state<D, W, DX, DA, DB, NEXT> st;
    uint32_t index[W];
    for (int x = 0; x < W; x++) index[x] = (uint32_t)(c >> (32 * x));
    const bool none = subtract<W>(st.q, p.last_index, index);
    for (int x = 0; x < W; x++) st.q[x] = none ? 0u : st.q[x];
    st.k = (uint32_t)p.K; st.n2 = 0.0f;
    st.at = threshold_base(D, W, DX, DA, DB);
    st.more = p.more;
    st.ones = ~0u;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(st.ones));                                       // (a constant would be added by itself, after the borrow)
    asm volatile("" : "+s"(st.at), "+s"(st.more));                 // (else a kernel's loop keeps registers per row: 106 scalar ones, seven waves)
#endif
    st.all(tables, p, emit, std::make_integer_sequence<int, D - 1>{});
    // the two points +k, -k of P(1,k): q = 1, 0
    const float m = (float)st.k;
    emit(D - 1, bits_float(st.q[0] << 31 | float_bits(m)));
    return fmaf(m, m, st.n2);
}

}  // namespace pvq_walk

// Which width schedule a context gets: fit_3q / fit_half / fit_quarter = the largest number of dimensions d whose
// N(d,K) fits three quarters / half / a quarter of the index's words.  Names only schedules listed in PVQ_WALK_DISPATCH.
// fit_double = the largest one whose N(d,K) is at most 2^52.  Groups of 16 whose last 8 dimensions fit a word have doubles
// above them, all or (K = 34 to 36) all but the first: N(15,36) < 2^52.
inline void pvq_walk_schedule(int D, int words, int fit_3q, int fit_half, int fit_quarter, int fit_double, int *dX, int *dA, int *dB)
{
    *dA = 0; *dB = 0;
    if (D == 16 && words == 2 && fit_half >= 8) *dA = 8;
    if (D == 32 && words == 2 && fit_half >= 12) *dA = 12;
    if (D == 32 && words == 4 && fit_half >= 15 && fit_quarter >= 6) { *dA = 15; *dB = 6; }
    *dX = *dA;
    if (D == 16 && words == 2 && *dA == 8) *dX = fit_double >= 16 ? 16 : 15;
    if (D == 32 && words == 4 && *dA == 15 && fit_3q >= 28) *dX = 28;
}

// The instantiated width schedules <D, W, DX, DA, DB>: CALL(D, W, DX, DA, DB) for the schedule (dX, dA, dB) chosen for a
// context of group size D with `words`-word indices.
#define PVQ_WALK_DISPATCH(CALL, D_, W_, dX_, dA_, dB_)                                                       \
    do {                                                                                                     \
        if ((D_) == 8) {                                                                                     \
            if ((W_) == 1) return CALL(8, 1, 0, 0, 0);                                                       \
            return CALL(8, 2, 0, 0, 0);                                                                      \
        }                                                                                                    \
        if ((D_) == 16) {                                                                                    \
            if ((W_) == 1) return CALL(16, 1, 0, 0, 0);                                                      \
            if ((W_) == 2) { if ((dX_) == 16) return CALL(16, 2, 16, 8, 0); if ((dX_) == 15) return CALL(16, 2, 15, 8, 0); return CALL(16, 2, 0, 0, 0); }     \
            return CALL(16, 4, 0, 0, 0);                                                                     \
        }                                                                                                    \
        if ((W_) == 1) return CALL(32, 1, 0, 0, 0);                                                          \
        if ((W_) == 2) { if ((dA_) == 12) return CALL(32, 2, 12, 12, 0); return CALL(32, 2, 0, 0, 0); }      \
        if ((dX_) == 28) return CALL(32, 4, 28, 15, 6);                                                      \
        if ((dA_) == 15 && (dB_) == 6) return CALL(32, 4, 15, 15, 6);                                        \
        return CALL(32, 4, 0, 0, 0);                                                                         \
    } while (0)
