// Table-driven decoder for D = 8 with single-word indices.
//
// App. B.3 walks one coordinate at a time and, inside a coordinate, one magnitude at a time: about
// D + K dependent table reads per group.  The same enumeration order can be inverted in a few
// steps if whole pairs of coordinates are located at once.  In the sub-pyramid with d open
// dimensions and k pulses, the points that share the next two coordinates (a, b) form one
// contiguous block of N(d-2, k-|a|-|b|) indices, and blocks follow each other in the visiting order
// of a, then of b (0, +1, -1, +2, -2, ...).  So a stage is: find the block that holds the residual
// index r, emit (a, b), subtract the block's start, continue with d-2 dimensions.
//
// Stages for D = 8:
//   S0  (d=8, k=K)   pair (y0,y1)  -> residual in (6, k1)
//   S1  (d=6, k1)    pair (y2,y3)  -> residual in (4, k2), of 16 bits from here on
//   S2  (d=4, k2)    single y4     -> residual in (3, k3)
//   T3  (d=3, k3)    direct table over every (k3, r): y5, y6, y7
// Finding a block: a bucket table indexed by (row k, r >> shift) names the block that holds the
// bucket's first index (candidate A) and a second block starting inside the bucket (candidate B, with
// its start relative to the bucket).  The block table entry carries the block's start and end; if
// r lies beyond the end (a bucket with several small blocks) the lane steps on block by block.
// Residuals are carried with a per-row bias that makes r >> shift the bucket's place in the stage's
// whole bucket table (see the block entries).  All tables sit in one blob that a workgroup copies into
// LDS; a kernel may read some of S0's block entries from the blob itself.
//
// The lookups in LDS, spread over all of it, and the instructions, those of the lanes that step on among them, are what
// the kernels spend their time on.  So the block entries of S1 and S2 are 8 bytes (a gather of 16 bytes a lane takes the
// LDS twice as long), which leaves room for finer buckets and S0's blocks beside them; a row's first bucket starts as far in
// front of its first index as lets the fewest indices step on; and S1's entries name three blocks.  K = 16, chance that one of a
// wave's 256 groups of normal weights steps on in S0, S1 and S2: 0.1, 0.5 and 0; with entries of 16 bytes, two blocks named and
// rows that start with a bucket 0.1, 0.9 and 0.6 (S0's blocks in device memory; in LDS with coarser buckets 0.4).  Products of
// 28672 x 8192 with 1, 4 and 16 vectors then 68, 83 and 102 us, now 56, 68 and 96; 8192 x 28672 with 16 94 and 89;
// 10000 x 3000 decoded to bf16 42 and 29.
//
// Values are emitted as packed bf16 pairs (exact for |y| <= 256) ready for v_dot2_f32_bf16, which also forms
// sum(y^2): exactly, on top of 2^22, so that the low bits of the float are 2 * sum(y^2).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define PVQ_HD __host__ __device__ inline
#else
#define PVQ_HD inline
#endif

// Keeps a 16-byte table entry together: without it the compiler reads the one field a loop tests
// first and the other three later, which costs a second LDS round trip per stage.
#if defined(__HIP_DEVICE_COMPILE__)
#define PVQ_KEEP_TOGETHER(q) asm volatile("" : "+v"(q))
#else
#define PVQ_KEEP_TOGETHER(q) ((void)0)
#endif

// a block entry as one 16-byte value (one register tuple on the device)
typedef uint32_t pvq_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t pvq_u32x2 __attribute__((ext_vector_type(2)));

struct pvq_fast8_params {
    uint32_t blob_bytes;  // whole blob: what a workgroup copies into LDS
    uint32_t lds_bytes;   // blob_bytes without its last table, 1/sqrt(n2) (a kernel with its own gain
                          // table leaves that out)
    uint32_t n_minus_1;   // N(8,K) - 1: stored indices are clamped to it
    uint32_t bk0, bk1, bk2, t3;   // byte offsets of the three bucket tables and of T3
    uint32_t bl0, bl1;            // ... and of S0's and S1's block tables (S2's is at the blob's start)
    uint32_t invs;        // 1 / sqrt(n2) as a float at invs + 2 * n2 (0 for n2 = 0); n2 is as odd or even as K
    uint32_t s0, s1, s2;  // bucket shifts of the three searched stages; of 24-bit indices pvq_fast8_shift24
    uint32_t k2max;       // n2 <= K*K
};

// Three bucket-entry forms.
// "two-candidate" (S0, 32 bits): bits 0..11 index of A in the stage's block table, bits 12..15 index distance from A
// to B, the top `shift` bits the start of B inside the bucket less one (all ones: no B), so that
// r << (32 - shift) is above the whole entry exactly when r has reached B.  B is the block starting inside the
// bucket that covers most of it.
// "three-candidate" (S1, 32 bits): the block after A too, whose start less one is in the `shift` bits below those;
// B (the distance from the block after A) is then the best of those that follow.
// "next-block" (S2, 16 bits): B is always the block after A, which lets one addition do the whole selection:
// entry = ((index of A - bucket number) << shift) + (2^shift - start of B inside the bucket), so that
// (entry + r) >> shift = index of A, plus one exactly when r has reached B (the low parts carry), modulo 2^16.
constexpr uint32_t kFast8IndexBits = 12;
constexpr uint32_t kFast8DbBits = 4;
constexpr uint32_t kFast8MaxShift = 13;   // all bucket shifts stay at or below this
constexpr uint32_t kFast8MaxShift1 = 8;   // S1's: two starts in an entry
// The bucket shifts for 24-bit indices (K = 15 and 16), which the kernels know when they are compiled: the starts in S1's
// entries are whole bytes then, compared without being moved, and S2's buckets so fine that no index steps on.
constexpr uint32_t pvq_fast8_shift24(int stage) { return stage == 0 ? 11 : stage == 1 ? 8 : 3; }
template <int STAGE, bool B24>
PVQ_HD uint32_t pvq_fast8_shift(const pvq_fast8_params &p)
{
    return B24 ? pvq_fast8_shift24(STAGE) : STAGE == 0 ? p.s0 : STAGE == 1 ? p.s1 : p.s2;
}
// LDS left for the blob: the 160 KiB of a compute unit minus 5 KiB for the kernels' own buffers
// (partial sums: 2 KiB; amplitude table: 1 KiB, or a fused gain table in place of 1/sqrt(n2))
constexpr uint32_t kFast8MaxBytes = 160 * 1024 - 5120;

// S0's block entry (16 bytes, read as one uint4): x = start, y = end (0xFFFFFFFF for the last block of the
// row), z = values as bf16 pair, w = 2^22 + a^2 + b^2 as a float's bits.  start and end are biased: a residual is
// carried as r + (its row's first bucket in the stage's bucket table) << shift + (the row's start in that
// bucket), so that r >> shift finds the bucket without a row offset; x = start - the next stage's row bias.
struct pvq_fast8_block {
    uint32_t start, end, values, squares;
};
// S1's and S2's (8 bytes): the low half of `range` is start + this row's bias - the next stage's row bias, modulo
// 2^16 (the next stage's residuals have 16 bits), its high half the end of what that stage's row then holds:
// a residual at or above it lies in a later block.  S2's values: the coordinate in the low half.
struct pvq_fast8_small_block {
    uint32_t range, values;
};

constexpr uint32_t kFast8Squares = 0x4A800000u;   // the bits of the float 2^22

// acc + a^2 + b^2 for a bf16 pair (a, b), acc as the bits of a float
PVQ_HD uint32_t pvq_fast8_add_squares(uint32_t acc, uint32_t pair)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef __attribute__((ext_vector_type(2))) __bf16 pair_t;
    const pair_t v = __builtin_bit_cast(pair_t, pair);
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_fdot2_f32_bf16(v, v, __builtin_bit_cast(float, acc), false));
#else
    const float lo = __builtin_bit_cast(float, pair << 16), hi = __builtin_bit_cast(float, pair & 0xFFFF0000u);
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, acc) + lo * lo + hi * hi);
#endif
}

// A searched stage for NG independent groups at once, in two halves so that all bucket reads are
// issued together and then all block reads (the latencies of the groups overlap instead of adding up).
//
// First half: the bucket lookups in the stage's bucket table (r is biased with its row, see the block entries); returns in
// addr[j] the byte offset of the block entry chosen for r[j].
// STAGE 0: two-candidate entries, block entries of 16 bytes; 1: three-candidate; 2: next-block.
template <int NG, int STAGE, bool B24>
PVQ_HD void pvq_fast8_find(const unsigned char *lds, const pvq_fast8_params &p, const uint32_t (&r)[NG], uint32_t (&addr)[NG])
{
    const uint32_t shift = pvq_fast8_shift<STAGE, B24>(p);
    uint32_t e[NG];
#pragma unroll
    for (int j = 0; j < NG; j++) {
        if constexpr (STAGE == 2) e[j] = *reinterpret_cast<const uint16_t *>(lds + p.bk2 + (r[j] >> shift) * 2u);
        else e[j] = *reinterpret_cast<const uint32_t *>(lds + (STAGE == 0 ? p.bk0 : p.bk1) + (r[j] >> shift) * 4u);
    }
#pragma unroll
    for (int j = 0; j < NG; j++) {
        if constexpr (STAGE == 2) {
            const uint32_t x = (uint16_t)(e[j] + r[j]);
            addr[j] = B24 ? x & ~7u : (x >> shift) << 3;
        } else {
            const uint32_t db = (e[j] >> kFast8IndexBits) & ((1u << kFast8DbBits) - 1u), x = r[j] << (32u - shift);
            uint32_t idx = e[j] & ((1u << kFast8IndexBits) - 1u);
            if constexpr (STAGE == 0) idx += x > e[j] ? db : 0u;
            else if constexpr (B24) idx += ((r[j] & 0xFFu) > e[j] >> 24 ? db : 0u) + ((r[j] & 0xFFu) > ((e[j] >> 16) & 0xFFu) ? 1u : 0u);
            else idx += (x > e[j] ? db : 0u) + (x > e[j] << shift ? 1u : 0u);
            addr[j] = STAGE == 0 ? p.bl0 + (idx << 4) : p.bl1 + (idx << 3);
        }
    }
}

// Second half for S0, after b[j] has been read from `lds + addr[j]`: a bucket with several small blocks
// makes the few lanes concerned move on block by block; then r[j] becomes the residual inside the
// block found.  `addr_of(addr)` fills in the entries' addresses when they are needed: a
// caller that did not keep them looks them up again, which only the rare groups that move on pay for.
template <int NG, typename AddrOf>
PVQ_HD void pvq_fast8_settle(const unsigned char *lds, uint32_t (&r)[NG], pvq_u32x4 (&b)[NG], AddrOf &&addr_of)
{
    bool miss = false, mj[NG];
#pragma unroll
    for (int j = 0; j < NG; j++) {
        PVQ_KEEP_TOGETHER(b[j]);
        mj[j] = r[j] >= b[j].y;
        miss = miss || mj[j];
    }
    if (miss) {
        // (stepping all NG groups together, one round trip per step of the furthest group, measured
        // slower than one short loop per group)
        uint32_t addr[NG];
        addr_of(addr);
#pragma unroll
        for (int j = 0; j < NG; j++) {
            if (mj[j]) {
                do {
                    addr[j] += 16;
                    b[j] = *reinterpret_cast<const pvq_u32x4 *>(lds + addr[j]);
                    PVQ_KEEP_TOGETHER(b[j]);
                } while (r[j] >= b[j].y);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NG; j++) r[j] -= b[j].x;
}

// both halves for S1 and S2: residuals of 16 bits from here on
template <int NG, int STAGE, bool B24>
PVQ_HD void pvq_fast8_stage(const unsigned char *lds, const pvq_fast8_params &p, uint32_t (&r)[NG], pvq_u32x2 (&b)[NG])
{
    uint32_t addr[NG], next[NG];
    pvq_fast8_find<NG, STAGE, B24>(lds, p, r, addr);
#pragma unroll
    for (int j = 0; j < NG; j++) b[j] = *reinterpret_cast<const pvq_u32x2 *>(lds + addr[j]);
    bool miss = false, mj[NG];
#pragma unroll
    for (int j = 0; j < NG; j++) {
        PVQ_KEEP_TOGETHER(b[j]);
        next[j] = (uint16_t)((uint16_t)r[j] - (uint16_t)b[j].x);
        mj[j] = next[j] >= b[j].x >> 16;
        miss = miss || mj[j];
    }
    // (24-bit indices: S2's entries name every block of their buckets)
    if (!(STAGE == 2 && B24) && miss) {
#pragma unroll
        for (int j = 0; j < NG; j++) {
            if (mj[j]) {
                do {
                    addr[j] += 8;
                    b[j] = *reinterpret_cast<const pvq_u32x2 *>(lds + addr[j]);
                    PVQ_KEEP_TOGETHER(b[j]);
                    next[j] = (uint16_t)((uint16_t)r[j] - (uint16_t)b[j].x);
                } while (next[j] >= b[j].x >> 16);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NG; j++) r[j] = next[j];
}

// S0 for NG stored indices, up to the places of the block entries in the tables: a caller that reads those entries from device memory can start S0 of its next indices
// while it still decodes the current ones.  r = the indices, clamped to the last valid one.
template <int NG, bool B24>
PVQ_HD void pvq_fast8_s0_find(const unsigned char *lds, const pvq_fast8_params &p, const uint32_t (&c)[NG],
                              uint32_t (&r)[NG], uint32_t (&addr)[NG])
{
#pragma unroll
    for (int j = 0; j < NG; j++) r[j] = c[j] < p.n_minus_1 ? c[j] : p.n_minus_1;
    pvq_fast8_find<NG, 0, B24>(lds, p, r, addr);
}

// The rest of the decoder, from S0's block entries b (as read from the addresses that
// pvq_fast8_s0_find gave for the clamped indices r) on.  Per index:
// four bf16 pairs (y0,y1) (y2,y3) (y4,y5) (y6,y7) and the bits of the float 2^22 + sum y^2: kFast8Squares + 2 * sum y^2.  Each pair is handed to
// `emit(j, pair number, word)` as soon as its stage has found it, so that a consumer that folds
// pairs into sums (the fused product) keeps one accumulator per group alive instead of the block
// entries.
template <int NG, bool B24, typename Emit>
PVQ_HD void pvq_fast8_rest(const unsigned char *lds, const pvq_fast8_params &p,
                           uint32_t (&r)[NG], pvq_u32x4 (&b)[NG], Emit &&emit, uint32_t (&squares)[NG])
{
    uint32_t acc[NG];
    pvq_u32x2 b1[NG], t[NG];
    pvq_fast8_settle<NG>(lds, r, b, [&](uint32_t (&out)[NG]) {
        uint32_t same[NG];
        pvq_fast8_s0_find<NG, B24>(lds, p, r, same, out);
    });
#pragma unroll
    for (int j = 0; j < NG; j++) { emit(j, 0, b[j].z); acc[j] = b[j].w; }
    pvq_fast8_stage<NG, 1, B24>(lds, p, r, b1);
#pragma unroll
    for (int j = 0; j < NG; j++) { emit(j, 1, b1[j].y); acc[j] = pvq_fast8_add_squares(acc[j], b1[j].y); }
    pvq_fast8_stage<NG, 2, B24>(lds, p, r, b1);
#pragma unroll
    for (int j = 0; j < NG; j++) t[j] = *reinterpret_cast<const pvq_u32x2 *>(lds + p.t3 + (r[j] << 3));
#pragma unroll
    for (int j = 0; j < NG; j++) {
        const uint32_t pair = t[j].x | b1[j].y;
        emit(j, 2, pair);
        emit(j, 3, t[j].y);
        squares[j] = pvq_fast8_add_squares(pvq_fast8_add_squares(acc[j], pair), t[j].y);
    }
}

// Whole decoder, one index set after the other.  `lds`: the blob (on the device: its copy in LDS).
template <int NG, bool B24, typename Emit>
PVQ_HD void pvq_fast8_decode_emit(const unsigned char *lds, const pvq_fast8_params &p,
                                  const uint32_t (&c)[NG], Emit &&emit, uint32_t (&squares)[NG])
{
    uint32_t r[NG], addr[NG];
    pvq_u32x4 b[NG];
    pvq_fast8_s0_find<NG, B24>(lds, p, c, r, addr);
#pragma unroll
    for (int j = 0; j < NG; j++) b[j] = *reinterpret_cast<const pvq_u32x4 *>(lds + addr[j]);
    pvq_fast8_rest<NG, B24>(lds, p, r, b, emit, squares);
}

// The same with the pairs stored.
template <int NG, bool B24>
PVQ_HD void pvq_fast8_decode(const unsigned char *lds, const pvq_fast8_params &p,
                             const uint32_t (&c)[NG], uint32_t (&pairs)[NG][4], uint32_t (&squares)[NG])
{
    pvq_fast8_decode_emit<NG, B24>(lds, p, c, [&](int j, int pair, uint32_t w) { pairs[j][pair] = w; }, squares);
}

// Host side: builds the blob for (8, K) if it fits `max_bytes`; returns false otherwise.
#include <vector>
bool pvq_fast8_build(int K, uint32_t max_bytes, std::vector<unsigned char> &blob, pvq_fast8_params &p);
