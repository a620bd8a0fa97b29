// Host construction of the tables used by the D = 8 table-driven decoder (see pvq_fast8.h), and a
// host self-test that replays the device walk over a range of indices.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "pvq.h"
#include "pvq_diagnostics.h"
#include "pvq_fast8.h"
#include "pvq_small_table.h"

namespace {

using namespace pvq_small;

struct Block {
    uint64_t start, size;
    uint32_t values, n2;
    int next_k;
};

// Bucket row over one row of blocks: entry j describes indices [j << shift, (j+1) << shift), counted from `front` in
// front of the row's first; NEXT: with the block after A (three candidates).  Returns how many indices are in none of their
// bucket's blocks; without `out` it only counts them, and passes over the buckets inside one block.
template <bool NEXT>
uint64_t build_bucket_row(const std::vector<Block> &blocks, uint32_t first_index, uint64_t total, int shift, uint64_t front,
                          std::vector<uint32_t> *out)
{
    const uint64_t width = (uint64_t)1 << shift;
    const uint64_t nb = (total + front + width - 1) / width;
    uint64_t missed = 0;
    size_t a = 0;
    for (uint64_t j = 0; j < nb; j++) {
        const uint64_t lo = j * width < front ? 0 : j * width - front, hi = std::min((j + 1) * width - front, total);
        while (a + 1 < blocks.size() && blocks[a + 1].start <= lo) a++;
        if (!out && a + 1 == blocks.size()) break;
        if (!out && blocks[a + 1].start >= hi) {
            j = ((blocks[a + 1].start + front) >> shift) - 1;
            continue;
        }
        auto cover = [&](size_t b) {           // of a block that starts inside the bucket, or of A from lo on
            return b < blocks.size() && blocks[b].start < hi ? std::min(hi, blocks[b].start + blocks[b].size) - std::max(lo, blocks[b].start) : 0;
        };
        auto start = [&](size_t b) { return (uint32_t)(blocks[b].start + front - j * width); };
        const size_t from = a + (NEXT ? 1 : 0);
        uint32_t db = 0, thr = (uint32_t)width;
        uint64_t best = 0;
        for (size_t b = from + 1; b < blocks.size() && blocks[b].start < hi && b - from < ((size_t)1 << kFast8DbBits); b++)
            if (cover(b) > best) { best = cover(b); db = (uint32_t)(b - from); thr = start(b); }
        uint32_t e = (first_index + (uint32_t)a) | (db << kFast8IndexBits) | ((thr - 1) << (32 - shift));
        missed += hi - lo - cover(a) - best;
        if (NEXT) {
            missed -= cover(a + 1);
            e |= ((cover(a + 1) ? start(a + 1) : (uint32_t)width) - 1) << (32 - 2 * shift);
        }
        if (out) out->push_back(e);
    }
    return missed;
}

// Bucket row in the next-block form: (index of A - bucket number) << shift, plus 2^shift minus the
// start of the block after A inside the bucket (nothing if it starts beyond the bucket).  The bucket
// number counts over all rows of the stage, as the biased residuals do (see write_blocks).
template <typename E>
uint64_t build_next_bucket_row(const std::vector<Block> &blocks, uint32_t first_index, uint64_t total, int shift, uint64_t front,
                               std::vector<E> *out)
{
    const uint64_t row_bucket = out ? out->size() : 0;   // the row's first bucket, counted over the whole stage
    const uint64_t width = (uint64_t)1 << shift;
    const uint64_t nb = (total + front + width - 1) / width;
    uint64_t missed = 0;
    size_t a = 0;
    for (uint64_t j = 0; j < nb; j++) {
        const uint64_t lo = j * width < front ? 0 : j * width - front, hi = std::min((j + 1) * width - front, total);
        while (a + 1 < blocks.size() && blocks[a + 1].start <= lo) a++;
        if (!out && a + 1 == blocks.size()) break;
        if (!out && blocks[a + 1].start >= hi) {
            j = ((blocks[a + 1].start + front) >> shift) - 1;
            continue;
        }
        uint64_t low = 0, covered = std::min(hi, blocks[a].start + blocks[a].size);
        if (a + 1 < blocks.size() && blocks[a + 1].start < hi) {
            low = width - (blocks[a + 1].start + front - j * width);
            covered = std::min(hi, blocks[a + 1].start + blocks[a + 1].size);
        }
        missed += hi - covered;
        const uint64_t high = (uint64_t)first_index + a - (row_bucket + j);   // modulo the entry width
        if (out) out->push_back((E)((high << shift) + low));
    }
    return missed;
}

// How far in front of a row its buckets start (below 2^shift, in up to 16 steps) for the fewest missed indices
template <typename Build>
uint64_t best_front(int shift, Build &&missed_with)
{
    const uint64_t width = (uint64_t)1 << shift;
    uint64_t best = 0, fewest = missed_with((uint64_t)0);
    for (uint64_t front = std::max<uint64_t>(1, width / 16); front < width && fewest > 0; front += std::max<uint64_t>(1, width / 16)) {
        const uint64_t missed = missed_with(front);
        if (missed < fewest) { fewest = missed; best = front; }
    }
    return best;
}

void align16(std::vector<unsigned char> &blob) { blob.resize((blob.size() + 15) & ~(size_t)15); }

template <typename T>
uint32_t append(std::vector<unsigned char> &blob, const std::vector<T> &v)
{
    align16(blob);
    const uint32_t off = (uint32_t)blob.size();
    blob.resize(off + v.size() * sizeof(T));
    if (!v.empty()) memcpy(blob.data() + off, v.data(), v.size() * sizeof(T));
    return off;
}

// known: the shifts are those that the kernels know
bool build_with_shifts(int K, const SmallTable &N, int s0, int s1, int s2, bool known, uint32_t max_bytes,
                       std::vector<unsigned char> &blob, pvq_fast8_params &p)
{
    // ---- block lists --------------------------------------------------------------------
    auto pair_blocks = [&](int rest_dims, int k) {
        std::vector<Block> v;
        uint64_t start = 0;
        for (int a : visiting_order(k))
            for (int b : visiting_order(k - abs(a))) {
                const int m = abs(a) + abs(b);
                Block blk{start, N.at(rest_dims, k - m), bf16_of_int(a) | (bf16_of_int(b) << 16),
                          (uint32_t)(a * a + b * b), k - m};
                v.push_back(blk);
                start += blk.size;
            }
        return v;
    };
    auto single_blocks = [&](int rest_dims, int k) {
        std::vector<Block> v;
        uint64_t start = 0;
        for (int a : visiting_order(k)) {
            Block blk{start, N.at(rest_dims, k - abs(a)), bf16_of_int(a), (uint32_t)(a * a), k - abs(a)};
            v.push_back(blk);
            start += blk.size;
        }
        return v;
    };

    std::vector<std::vector<Block>> rows0{pair_blocks(6, K)}, rows1, rows2;
    for (int k = 0; k <= K; k++) { rows1.push_back(pair_blocks(4, k)); rows2.push_back(single_blocks(3, k)); }

    // ---- T3: every (k, r) of the last three coordinates ---------------------------------------
    std::vector<uint32_t> t3;  // two words per entry
    std::vector<uint32_t> t3_row(K + 1);
    for (int k = 0; k <= K; k++) {
        t3_row[k] = (uint32_t)t3.size() * 4;
        for (int a : visiting_order(k))
            for (int b : visiting_order(k - abs(a))) {
                const int rem = k - abs(a) - abs(b);
                for (int sgn = 0; sgn < (rem ? 2 : 1); sgn++) {
                    const int c = sgn ? -rem : rem;
                    t3.push_back(bf16_of_int(a) << 16);
                    t3.push_back(bf16_of_int(b) | (bf16_of_int(c) << 16));
                }
            }
        if ((t3.size() * 4 - t3_row[k]) / 8 != N.at(3, k)) return false;
    }

    size_t least = t3.size() * 4 + rows0[0].size() * 16 + (N.at(8, K) >> s0) * 4;   // (before any work on buckets that will not fit)
    for (int k = 0; k <= K; k++)
        least += (rows1[k].size() + rows2[k].size()) * 8 + (N.at(6, k) >> s1) * 4 + (N.at(4, k) >> s2) * 2;
    if (least > max_bytes) return false;

    // ---- bucket rows --------------------------------------------------------------------------
    std::vector<uint32_t> bk0, bk1;
    std::vector<uint16_t> bk2;
    std::vector<uint32_t> bias1(K + 1), bias2(K + 1);   // what a row's residuals are carried with (see write_blocks)
    build_bucket_row<false>(rows0[0], 0, N.at(8, K), s0, 0, &bk0);
    uint32_t first = 0;
    for (int k = 0; k <= K; k++) {
        const uint64_t front = best_front(s1, [&](uint64_t f) {
            return build_bucket_row<true>(rows1[k], 0, N.at(6, k), s1, f, nullptr);
        });
        bias1[k] = ((uint32_t)bk1.size() << s1) + (uint32_t)front;
        build_bucket_row<true>(rows1[k], first, N.at(6, k), s1, front, &bk1);
        first += (uint32_t)rows1[k].size();
    }
    if (first > (1u << kFast8IndexBits)) return false;   // S1's block numbers must fit the entries
    first = 0;
    uint64_t missed2 = 0;
    for (int k = 0; k <= K; k++) {
        const uint64_t front = best_front(s2, [&](uint64_t f) {
            return build_next_bucket_row<uint16_t>(rows2[k], 0, N.at(4, k), s2, f, nullptr);
        });
        bias2[k] = ((uint32_t)bk2.size() << s2) + (uint32_t)front;
        missed2 += build_next_bucket_row<uint16_t>(rows2[k], first, N.at(4, k), s2, front, &bk2);
        first += (uint32_t)rows2[k].size();
    }
    if (first >= (1u << (16 - s2))) return false;   // S2's block numbers must fit the 16-bit entries
    if (known && missed2 > 0) return false;         // (the kernels do not look)
    // a residual of S2 has 16 bits, also before a step to the following block (at most a bucket of S1 too large)
    if (((uint64_t)bk2.size() << s2) + ((uint64_t)1 << s1) > 65536) return false;

    // ---- lay the blob out ---------------------------------------------------------------------
    // sizes are known now; offsets of the rows that `meta` words point to must be fixed before the
    // block tables are written
    auto up16 = [](size_t x) { return (x + 15) & ~(size_t)15; };
    size_t nblk0 = rows0[0].size(), nblk1 = 0, nblk2 = 0;
    for (auto &r : rows1) nblk1 += r.size();
    for (auto &r : rows2) nblk2 += r.size();
    size_t off = 0;
    const size_t o_bl2 = off; off = up16(off + nblk2 * 8);   // (at 0: the kernels add nothing)
    const size_t o_bk0 = off; off = up16(off + bk0.size() * 4);
    const size_t o_bk1 = off; off = up16(off + bk1.size() * 4);
    const size_t o_bk2 = off; off = up16(off + bk2.size() * 2);
    const size_t o_t3 = off;  off = up16(off + t3.size() * 4);
    const size_t o_bl0 = off; off = up16(off + nblk0 * 16);
    const size_t o_bl1 = off; off = up16(off + nblk1 * 8);
    // 1/sqrt(n2) comes last of what goes to LDS: a kernel that builds its own gain table leaves it out
    const size_t lds_bytes = off;
    const size_t o_invs = off; off = up16(off + (size_t)(K * K / 2 + 1) * 4);
    if (off > max_bytes) return false;

    // Residuals travel biased: inside stage S a residual r of row k is kept as r + ((first bucket of row k, counted over
    // the stage) << shift_S) + (how far in front of the row that bucket starts), so that r >> shift_S is the bucket's place
    // in the stage's whole bucket table and no row offset has to be carried or added.  A block entry's `start` therefore
    // holds start + this row's bias - the next stage's row bias.  For T3 the bias is the row's first entry (shift 0).
    auto bias3 = [&](int k) { return t3_row[k] / 8u; };
    std::vector<pvq_fast8_block> bl0;
    for (size_t i = 0; i < nblk0; i++) {
        const Block &b = rows0[0][i];
        const uint32_t end = i + 1 < nblk0 ? (uint32_t)(b.start + b.size) : 0xFFFFFFFFu;
        bl0.push_back({(uint32_t)b.start - bias1[b.next_k], end, b.values, __builtin_bit_cast(uint32_t, 4194304.0f + (float)b.n2)});
    }
    auto write_blocks = [&](const std::vector<std::vector<Block>> &rows, auto row_bias, auto next_bias) {
        std::vector<pvq_fast8_small_block> v;
        for (size_t k = 0; k < rows.size(); k++)
            for (const Block &b : rows[k]) {
                const uint32_t next = next_bias(b.next_k);
                v.push_back({(((uint32_t)b.start + row_bias((int)k) - next) & 0xFFFFu) | ((next + (uint32_t)b.size) << 16), b.values});
            }
        return v;
    };
    const auto bl1 = write_blocks(rows1, [&](int k) { return bias1[k]; }, [&](int k) { return bias2[k]; });
    const auto bl2 = write_blocks(rows2, [&](int k) { return bias2[k]; }, bias3);
    std::vector<float> invs((size_t)K * K / 2 + 1);
    for (int h = 0; h <= K * K / 2; h++) {
        const int n2 = 2 * h + (K & 1);
        invs[h] = n2 ? (float)(1.0 / std::sqrt((double)n2)) : 0.0f;
    }

    blob.clear();
    bool ok = append(blob, bl2) == o_bl2 && append(blob, bk0) == o_bk0 && append(blob, bk1) == o_bk1 && append(blob, bk2) == o_bk2 &&
              append(blob, t3) == o_t3;
    ok = ok && append(blob, bl0) == o_bl0 && append(blob, bl1) == o_bl1 && append(blob, invs) == o_invs;
    align16(blob);
    if (!ok || blob.size() != off) return false;

    p.blob_bytes = (uint32_t)blob.size();
    p.lds_bytes = (uint32_t)lds_bytes;
    p.n_minus_1 = (uint32_t)(N.at(8, K) - 1);
    p.bk0 = (uint32_t)o_bk0; p.bk1 = (uint32_t)o_bk1; p.bk2 = (uint32_t)o_bk2; p.t3 = (uint32_t)o_t3;
    p.bl0 = (uint32_t)o_bl0; p.bl1 = (uint32_t)o_bl1;
    p.invs = (uint32_t)o_invs - 2u * (uint32_t)(K & 1);
    p.s0 = s0; p.s1 = s1; p.s2 = s2;
    p.k2max = (uint32_t)(K * K);
    return true;
}

}  // namespace

bool pvq_fast8_build(int K, uint32_t max_bytes, std::vector<unsigned char> &blob, pvq_fast8_params &p)
{
    if (K < 1 || K > 22) return false;  // 2*K*K must stay below 2^10
    SmallTable N(K);
    if (N.at(8, K) > ((uint64_t)1 << 32)) return false;
    int bits = 0;
    while (((uint64_t)1 << bits) < N.at(8, K)) bits++;
    // Finer buckets mean fewer block-by-block steps; take the finest combination that fits.  The
    // base shifts follow the index width (for 24 bits they would be pvq_fast8_shift24's); S2 is coarsened first (its
    // blocks are the most regular), then S0, and S1 last.
    static const int steps[][3] = {{0, 0, 0}, {0, 0, 1}, {1, 0, 1}, {1, 0, 2}, {2, 0, 2}, {2, 1, 2}, {3, 1, 2}, {3, 2, 2}};
    if (bits == 24)
        return build_with_shifts(K, N, pvq_fast8_shift24(0), pvq_fast8_shift24(1), pvq_fast8_shift24(2), true, max_bytes, blob, p);
    for (const auto &st : steps) {
        const int s0 = std::min(std::max(1, bits - 13) + st[0], (int)kFast8MaxShift);
        const int s1 = std::min(std::max(1, bits - 16) + st[1], (int)kFast8MaxShift1);
        const int s2 = std::min(std::max(1, bits - 21) + st[2], 6);
        if (build_with_shifts(K, N, s0, s1, s2, false, max_bytes, blob, p)) return true;
    }
    return false;
}

// Replays the table walk on the host for indices [first, first + count) of (8, K) and compares the
// decoded point with the plain coordinate-by-coordinate walk of App. B.3.
extern "C" int pvq_fast_tables_selftest(int K, uint64_t first, uint64_t count, uint64_t *mismatches)
{
    if (!mismatches) return PVQ_E_INVALID_ARG;
    SmallTable N(K);
    const uint64_t total = N.at(8, K);
    uint64_t bad = 0;
    std::vector<unsigned char> blob;
    pvq_fast8_params p;
    if (!pvq_fast8_build(K, kFast8MaxBytes, blob, p)) return PVQ_E_UNSUPPORTED;
    for (uint64_t c = first; c < first + count && c < total; c++) {
        uint32_t cc[1] = {(uint32_t)c}, pr[1][4], nn[1];
        if (total > (1u << 23) && total <= (1u << 24)) pvq_fast8_decode<1, true>(blob.data(), p, cc, pr, nn);
        else pvq_fast8_decode<1, false>(blob.data(), p, cc, pr, nn);
        const uint32_t *pairs = pr[0];
        const uint32_t n2x2 = nn[0] - kFast8Squares;
        int y[8];
        plain_walk(N, K, c, y);
        int n2 = 0;
        bool same = true;
        for (int i = 0; i < 8; i++) {
            n2 += y[i] * y[i];
            const uint32_t h = (pairs[i / 2] >> (16 * (i & 1))) & 0xFFFFu;
            same = same && h == bf16_of_int(y[i]);
        }
        same = same && n2x2 == (uint32_t)(2 * n2);
        bad += !same;
    }
    *mismatches = bad;
    return PVQ_OK;
}
