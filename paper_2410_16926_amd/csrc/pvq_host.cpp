// Host side of libpvq: status codes, exact size tables, the choice of K, Beta quantile tables,
// the context, and argument validation in front of the kernel launchers.
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "pvq_internal.h"
#include "pvq_diagnostics.h"
#include "pvq_walk.h"

// ------------------------------------------------------------------------------------------
// status
// ------------------------------------------------------------------------------------------

static thread_local int g_last_hip_error = 0;

static int hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return PVQ_E_HIP;
}

extern "C" const char *pvq_strerror(int status)
{
    switch (status) {
    case PVQ_OK: return "ok";
    case PVQ_E_INVALID_ARG: return "invalid argument";
    case PVQ_E_UNSUPPORTED: return "unsupported configuration";
    case PVQ_E_ALIGNMENT: return "pointer or leading dimension not aligned as required";
    case PVQ_E_HIP: return "HIP runtime error (see pvq_last_hip_error)";
    case PVQ_E_NOMEM: return "out of host memory";
    default: return "unknown status";
    }
}

extern "C" int pvq_last_hip_error(void) { return g_last_hip_error; }

// ------------------------------------------------------------------------------------------
// 512-bit unsigned integers (eight 64-bit limbs) for the size tables
// ------------------------------------------------------------------------------------------

namespace {

struct U512 {
    uint64_t limb[8] = {0, 0, 0, 0, 0, 0, 0, 0};

    static U512 of(uint64_t v)
    {
        U512 r;
        r.limb[0] = v;
        return r;
    }
    // returns true when the sum left 512 bits
    bool add(const U512 &o)
    {
        unsigned __int128 carry = 0;
        for (int i = 0; i < 8; i++) {
            unsigned __int128 s = (unsigned __int128)limb[i] + o.limb[i] + carry;
            limb[i] = (uint64_t)s;
            carry = s >> 64;
        }
        return carry != 0;
    }
    void decrement()  // value > 0
    {
        for (int i = 0; i < 8; i++)
            if (limb[i]-- != 0) break;
    }
    int bit_length() const
    {
        for (int i = 7; i >= 0; i--)
            if (limb[i]) return 64 * i + 64 - __builtin_clzll(limb[i]);
        return 0;
    }
    uint32_t word(int i) const { return (uint32_t)(limb[i >> 1] >> (32 * (i & 1))); }
};

// Pyramid sizes N(d,k) for d <= D, k <= K (Sec. 2.4).  Rolling rows would do for a single count,
// but the kernels need every row, so the whole table is kept.
struct SizeTable {
    int D, K;
    int first_bad_k;      // smallest k with an entry that left 512 bits (K+1 if none); columns
                          // below it are exact, because N(d,k) only depends on columns <= k
    bool overflow;
    std::vector<U512> n;  // (D+1) x (K+1)

    SizeTable(int D_, int K_) : D(D_), K(K_), first_bad_k(K_ + 1), n((size_t)(D_ + 1) * (K_ + 1))
    {
        for (int k = 0; k <= K; k++) at(0, k) = U512::of(k == 0 ? 1 : 0);
        for (int d = 1; d <= D; d++) {
            at(d, 0) = U512::of(1);
            for (int k = 1; k <= K; k++) {
                U512 v = at(d - 1, k);
                bool bad = v.add(at(d, k - 1));
                bad |= v.add(at(d - 1, k - 1));
                if (bad && k < first_bad_k) first_bad_k = k;
                at(d, k) = v;
            }
        }
        overflow = first_bad_k <= K;
    }
    U512 &at(int d, int k) { return n[(size_t)d * (K + 1) + k]; }
    const U512 &at(int d, int k) const { return n[(size_t)d * (K + 1) + k]; }
    int index_bits() const
    {
        U512 top = at(D, K);
        top.decrement();
        return top.bit_length();
    }
};

}  // namespace

extern "C" int pvq_count(int D, int K, uint32_t *count_words, int *index_bits)
{
    if (D < 1 || D > 256 || K < 0 || K > 1024) return PVQ_E_INVALID_ARG;
    SizeTable t(D, K);
    if (t.overflow) return PVQ_E_UNSUPPORTED;
    if (count_words)
        for (int i = 0; i < 16; i++) count_words[i] = t.at(D, K).word(i);
    if (index_bits) *index_bits = t.index_bits();
    return PVQ_OK;
}

extern "C" int pvq_max_k(int D, int bit_budget, int *K)
{
    if (D < 1 || D > 256 || bit_budget < 1 || bit_budget > 511 || !K) return PVQ_E_INVALID_ARG;
    // One table with a generous K bound; N(D,k) grows with k, so the first k that does not fit
    // (or that left the 512-bit integers) ends the search.
    int kmax = 1024;
    SizeTable t(D, kmax);
    int best = 0;
    for (int k = 1; k <= kmax && k < t.first_bad_k; k++) {
        U512 top = t.at(D, k);
        top.decrement();
        if (top.bit_length() > bit_budget) break;
        best = k;
    }
    if (best < 1) return PVQ_E_UNSUPPORTED;
    *K = best;
    return PVQ_OK;
}

// ------------------------------------------------------------------------------------------
// Beta(a, b) quantiles for integer a (D even): Sec. 3.4
// ------------------------------------------------------------------------------------------

namespace {

// For integer a the upper tail of Beta(a, b) is a short sum of positive terms,
//   P[X > x] = (1-x)^b * sum_{j < a} C(b+j-1, j) x^j,
// evaluated in long double.  The lower tail is 1 minus it; the probabilities asked for are
// multiples of 2^-9 at the finest, so the subtraction costs nothing that matters at 64 mantissa bits.
long double beta_upper_tail(long double x, int a, long double b)
{
    if (x <= 0) return 1.0L;
    if (x >= 1) return 0.0L;
    long double lead = expl(b * log1pl(-x));
    long double term = 1.0L;  // C(b+j-1, j) x^j at j = 0
    long double sum = 0.0L;
    for (int j = 0; j < a; j++) {
        sum += term;
        term *= (b + j) * x / (long double)(j + 1);
    }
    return lead * sum;
}

// PPF(p) by bisection: the upper tail decreases in x.
double beta_ppf(long double p, int a, long double b)
{
    long double lo = 0.0L, hi = 1.0L;
    long double target = 1.0L - p;
    for (int it = 0; it < 400; it++) {
        long double mid = 0.5L * (lo + hi);
        if (mid == lo || mid == hi) break;
        if (beta_upper_tail(mid, a, b) > target) lo = mid; else hi = mid;
    }
    return (double)(0.5L * (lo + hi));
}

bool scale_bits_ok(int sb) { return sb == 0 || sb == 1 || sb == 2 || sb == 4 || sb == 8; }

}  // namespace

extern "C" int pvq_beta_tables(int D, int64_t G, int scale_bits, double *edges, double *centers)
{
    if (!edges || !centers || D < 2 || G < 2) return PVQ_E_INVALID_ARG;
    if ((D & 1) || !scale_bits_ok(scale_bits) || scale_bits == 0) return PVQ_E_UNSUPPORTED;
    int a = D / 2;
    long double b = (long double)D * (long double)(G - 1) / 2.0L;
    int n = 1 << scale_bits;
    for (int j = 1; j < n; j++) edges[j - 1] = beta_ppf((long double)j / n, a, b);
    for (int q = 0; q < n; q++) centers[q] = beta_ppf(((long double)q + 0.5L) / n, a, b);
    return PVQ_OK;
}

// ------------------------------------------------------------------------------------------
// tables of the coordinate-by-coordinate decoder (pvq_walk.hip)
// ------------------------------------------------------------------------------------------

namespace {

typedef unsigned __int128 u128;

u128 low128(const U512 &v) { return ((u128)v.limb[1] << 64) | v.limb[0]; }

// Lays the blob out (pvq_walk.h has the layout's formulas) and fills it.  Bucket (e, f) of a guess row with mb fraction
// bits holds the q whose float, as the decoder forms it from q | 1, lies in [2^e (1 + f / 2^mb), 2^e (1 + (f+1) / 2^mb)), in
// rows of doubles those whose q + 1/2 lies in half that range; its guess is the last threshold that is not above any of them.
template <int D, int W, int DX, int DA, int DB>
bool fill_walk_tables(const SizeTable &t, std::vector<unsigned char> &blob, pvq_walk_params &p)
{
    using namespace pvq_walk;
    const int K = p.K, entries = 2 * K + 3;
    for (int i = 0; i < 3; i++) p.part_bytes[i] = (uint32_t)((entries * (4 << i) + 15) / 16 * 16);
    uint32_t at = threshold_base(D, W, DX, DA, DB);
    blob.assign(at, 0);
    p.more = 0;
    std::vector<u128> T(entries);
    for (int dp = D - 1; dp >= 2; dp--) {
        const int words = words_of_row(dp, W, DX, DA, DB), mb = guess_bits(dp, D);
        const u128 limit = low128(t.at(dp + 1, K));                // of q
        if (t.at(dp + 1, K).bit_length() > 32 * words) return false;
        u128 even = 0;
        for (int C = 0; C <= K; C++) {
            const u128 n = low128(t.at(dp, C));
            T[2 * C] = even;
            T[2 * C + 1] = even + n;
            even += 2 * n;
        }
        T[2 * K + 2] = ~(u128)0;
        blob.resize(at + row_bytes(p, words), 0);
        const bool doubles = double_row(dp, W, DX, DA);
        if (doubles && t.at(dp + 1, K).bit_length() > 52) return false;
        for (int j = 0; doubles && j < entries; j++) {
            const double v = j < entries - 1 ? (double)(uint64_t)T[j] * kDoubleUnit : HUGE_VAL;
            memcpy(&blob[at + 8 * j], &v, 8);
        }
        for (int j = 0; !doubles && j < entries; j++)
            for (int w = 0; w < words; w++) {
                const uint32_t v = (uint32_t)(T[j] >> (32 * w));
                memcpy(&blob[words == 3 ? (w < 2 ? at + 8 * j + 4 * w : at + p.part_bytes[1] + 4 * j) : at + 4 * (words * j + w)], &v, 4);
            }
        at = (uint32_t)blob.size();
        // the buckets
        unsigned char *guess = &blob[guess_row(dp, D, W, DX, DA, DB)];
        const uint32_t n = guess_entries(dp, D, words);
        const u128 one = 1;
        auto edge = [&](uint32_t b) -> u128 {                      // the bucket's lower edge, rounded up
            const int e = (int)(b >> mb);
            const u128 f = (one << mb) + (b & ((1u << mb) - 1u));
            if (e >= 128) return ~(u128)0;
            return e >= mb ? f << (e - mb) : (f + (one << (mb - e)) - 1) >> (mb - e);
        };
        int j = 0, above = 0;                                      // thresholds: the last <= from, the last <= to
        for (uint32_t b = 0; b < n; b++) {
            // q from .. to: as floats exact below 2^23, with what the roundings may move beyond it
            u128 from = edge(b), to = edge(b + 1);
            if (doubles) {                                         // (of 2 q + 1, exact)
                from /= 2;
                to /= 2;
            } else {
                if (from >> 23) from -= from >> 21;
                if (to >> 23) to += std::min(to >> 21, ~(u128)0 - to);
                from -= from & 1;                                  // (q | 1)
            }
            to = std::min(to, limit);                              // (exclusive)
            if (from >= to) { guess[b] = (unsigned char)j; continue; }
            while (T[j + 1] <= from) j++;
            above = std::max(above, j);
            while (T[above + 1] < to) above++;
            guess[b] = (unsigned char)j;
            if (above > j + 1) p.more |= 1u << dp;
        }
    }
    p.bytes = (uint32_t)blob.size();
    return searches(D, W, DX, DA) || !p.more;
}

bool build_walk_tables(const SizeTable &t, int D, int K, int words, std::vector<unsigned char> &blob, pvq_walk_params &p)
{
    if (D > 32 || K > 127) return false;
    memset(&p, 0, sizeof p);
    int fit_3q = 0, fit_half = 0, fit_quarter = 0, fit_double = 0;
    for (int d = 1; d <= D; d++) {
        const int bits = t.at(d, K).bit_length();
        if (bits <= 52) fit_double = d;
        if (d == D) break;
        if (words >= 4 && bits <= 24 * words) fit_3q = d;
        if (words >= 2 && bits <= 16 * words) fit_half = d;
        if (words >= 4 && bits <= 8 * words) fit_quarter = d;
    }
    pvq_walk_schedule(D, words, fit_3q, fit_half, fit_quarter, fit_double, &p.dX, &p.dA, &p.dB);
    p.K = K;
    U512 last = t.at(D, K);
    last.decrement();
    for (int w = 0; w < 4; w++) p.last_index[w] = last.word(w);
#define PVQ_WALK_FILL(D_, W_, DX_, DA_, DB_) fill_walk_tables<D_, W_, DX_, DA_, DB_>(t, blob, p)
    PVQ_WALK_DISPATCH(PVQ_WALK_FILL, D, words, p.dX, p.dA, p.dB);
#undef PVQ_WALK_FILL
}

}  // namespace

// ------------------------------------------------------------------------------------------
// context
// ------------------------------------------------------------------------------------------

extern "C" int pvq_ctx_create(pvq_ctx **out, int D, int K, int scale_bits, const double *edges,
                              const double *centers)
{
    if (!out) return PVQ_E_INVALID_ARG;
    *out = nullptr;
    // groups of 64 and 128 values (the on-the-fly activation setting) go to the kernels of pvq_wide.hip:
    // tables of up to 16-word integers in device memory
    const bool wide = D == 64 || D == 128;
    if (!wide && D != 8 && D != 16 && D != 32) return PVQ_E_UNSUPPORTED;
    if (K < 1 || K > (wide ? 1023 : 127)) return PVQ_E_UNSUPPORTED;
    if (!scale_bits_ok(scale_bits) || (wide && scale_bits != 0)) return PVQ_E_UNSUPPORTED;
    if (scale_bits > 0 && (!edges || !centers)) return PVQ_E_INVALID_ARG;

    SizeTable t(D, K);
    if (t.overflow) return PVQ_E_UNSUPPORTED;
    int bits = t.index_bits();
    if (bits < 1 || bits > (wide ? 512 : 128)) return PVQ_E_UNSUPPORTED;
    int words = bits <= 32 ? 1 : (bits <= 64 ? 2 : 4);
    if (wide) words = 4 * ((std::max(t.at(D, K).bit_length(), 1) + 127) / 128);   // N(D,K) itself is an entry
    // the decoders form N(D,K) - 1 - index in `words` words: N(D,K) must fit them (it fails to only when it
    // is exactly 2^(32 words), which no supported (D,K) gives)
    if (t.at(D, K).bit_length() > 32 * words) return PVQ_E_UNSUPPORTED;

    int n = scale_bits ? (1 << scale_bits) : 0;
    std::vector<float> e32, sc32;
    if (scale_bits) {
        for (int j = 0; j + 1 < n; j++) {
            if (!(edges[j] >= 0.0) || (j > 0 && !(edges[j] >= edges[j - 1]))) return PVQ_E_INVALID_ARG;
            e32.push_back((float)edges[j]);
        }
        for (int q = 0; q < n; q++) {
            if (!(centers[q] >= 0.0)) return PVQ_E_INVALID_ARG;
            sc32.push_back((float)std::sqrt(centers[q]));
        }
    }

    // tab_u[dp][k+1] = N(dp,0) + ... + N(dp,k), tab_u[dp][0] = 0.  Every entry is below N(D,K) (the pyramid of one
    // more dimension contains all of them), so it fits `words` words.
    std::vector<uint32_t> hu;
    size_t near_at = 0, key_at = 0, guess_at = 0;    // wide: where the other tables lie behind the thresholds, in words
    if (wide) {
        // The thresholds T_j of every row (pvq_internal.h): T_{2C} = 2 (N(dp,0) + ... + N(dp,C-1)), T_{2C+1} = T_{2C} +
        // N(dp,C); none is above N(dp+1,K).
        const int row = pvq_wide_row(K), krow = pvq_wide_key_row(K), buckets = pvq_wide_buckets(words);
        const size_t nears = (size_t)D * row + 64;    // (the decoder reads 128 at a time, and uses 64)
        near_at = (size_t)D * row * words;
        key_at = near_at + 2 * nears;
        guess_at = key_at + (size_t)D * krow;
        hu.assign(guess_at + (size_t)D * buckets / 2, 0xFFFFFFFFu);
        double *near = reinterpret_cast<double *>(&hu[near_at]);
        uint16_t *guess = reinterpret_cast<uint16_t *>(&hu[guess_at]);
        std::fill(near, near + nears, (double)INFINITY);
        for (int dp = 0; dp < D; dp++) {
            uint32_t *key = &hu[key_at + (size_t)dp * krow];
            U512 even;                           // T_{2C}
            for (int C = 0; C <= K; C++) {
                const U512 &n = t.at(dp, C);
                U512 odd = even;
                odd.add(n);
                for (int h = 0; h < 2; h++) {
                    const U512 &v = h ? odd : even;
                    uint32_t *out = &hu[((size_t)dp * row + 2 * C + h) * words];
                    for (int w = 0; w < words; w++) out[w] = v.word(w);
                    key[2 * C + h] = pvq_wide_key(out, words);
                    near[(size_t)dp * row + 2 * C + h] = pvq_wide_double(out, words);
                }
                even = odd;
                even.add(n);
            }
            // A bucket's guess: the last threshold whose key lies below every key of the bucket (bucket 8 is the first
            // with a key above 0).
            for (int j = 0, from = 0; j < 2 * K + 2; j++) {
                const int to = j + 1 == 2 * K + 2 ? buckets : std::max(8, (int)(key[j + 1] >> 22) * 8 + (int)(key[j + 1] >> 18 & 7) + 1);
                if (to > from) std::fill(guess + (size_t)dp * buckets + from, guess + (size_t)dp * buckets + to, (uint16_t)j);
                from = std::max(from, to);
            }
        }
    } else {
        hu.resize((size_t)D * (K + 2) * words);
    }
    for (int dp = 0; dp < D && !wide; dp++) {
        U512 run;  // running sum
        for (int w = 0; w < words; w++) hu[((size_t)dp * (K + 2)) * words + w] = 0;
        for (int k = 0; k <= K; k++) {
            run.add(t.at(dp, k));
            for (int w = 0; w < words; w++) hu[((size_t)dp * (K + 2) + k + 1) * words + w] = run.word(w);
        }
    }

    pvq_ctx *c = new (std::nothrow) pvq_ctx();
    if (!c) return PVQ_E_NOMEM;
    c->D = D; c->K = K; c->index_bits = bits; c->words = words; c->scale_bits = scale_bits; c->wide = wide ? 1 : 0;
    c->tab_u = nullptr; c->tab_key = nullptr; c->tab_near = nullptr; c->tab_guess = nullptr;
    c->edges = c->sqrtc = nullptr; c->fast8_blob = nullptr; c->enc8_offs = nullptr; c->amplitude = PVQ_AMP_NORM;
    U512 last = t.at(D, K);
    last.decrement();
    for (int w = 0; w < 16; w++) c->last_index[w] = last.word(w);

    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess) e = hipMalloc((void **)&c->tab_u, hu.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(c->tab_u, hu.data(), hu.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess && wide) {
        c->tab_near = reinterpret_cast<const double *>(c->tab_u + near_at);
        c->tab_key = c->tab_u + key_at;
        c->tab_guess = reinterpret_cast<const uint16_t *>(c->tab_u + guess_at);
    }
    if (e == hipSuccess && scale_bits) {
        // 2^b entries, the last of which is no edge (+inf, which no kernel reads)
        e32.push_back(INFINITY);
        e = hipMalloc((void **)&c->edges, sizeof(float) * n);
        if (e == hipSuccess) e = hipMalloc((void **)&c->sqrtc, sizeof(float) * n);
        if (e == hipSuccess) e = hipMemcpy(c->edges, e32.data(), sizeof(float) * n, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(c->sqrtc, sc32.data(), sizeof(float) * n, hipMemcpyHostToDevice);
    }
    if (e == hipSuccess && D == 8 && words == 1) {
        std::vector<unsigned char> blob;
        if (pvq_fast8_build(K, kFast8MaxBytes, blob, c->fast8)) {
            e = pvq_fast8_prepare();
            if (e == hipSuccess) e = hipMalloc((void **)&c->fast8_blob, blob.size());
            if (e == hipSuccess) e = hipMemcpy(c->fast8_blob, blob.data(), blob.size(), hipMemcpyHostToDevice);
        }
    }
    if (e == hipSuccess && !wide) {
        std::vector<unsigned char> blob;
        // the decoders of pvq_walk.hip keep these in LDS: every supported (D, K) fits
        if (!build_walk_tables(t, D, K, words, blob, c->walk)) { pvq_ctx_destroy(c); return PVQ_E_UNSUPPORTED; }
        e = hipMalloc((void **)&c->walk_blob, blob.size());
        if (e == hipSuccess) e = hipMemcpy(c->walk_blob, blob.data(), blob.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess && !pvq_walk_usable(c)) { pvq_ctx_destroy(c); return PVQ_E_UNSUPPORTED; }
    }
    if (e == hipSuccess && D == 8 && bits == 24 && K <= PVQ_ENC8_MAX_K) {
        // What coordinate i (7-i dimensions after it) adds to the index when k pulses are left and it
        // takes the value y of magnitude m (App. B.2):
        //   N(7-i,k) [m>0] + 2 sum_{j=1}^{m-1} N(7-i,k-j) + [y<0] N(7-i,k-m)
        constexpr int M = PVQ_ENC8_MAX_K;
        std::vector<uint32_t> offs((size_t)(PVQ_ENC8_WORDS + 3) / 4 * 4, 0u);
        for (int i = 0; i < 7; i++)
            for (int k = 0; k <= K; k++)
                for (int m = 1; m <= k; m++) {
                    uint64_t v = t.at(7 - i, k).limb[0];
                    for (int j = 1; j < m; j++) v += 2 * t.at(7 - i, k - j).limb[0];
                    uint32_t *zero = &offs[((size_t)i * (M + 1) + k) * (2 * M + 1) + M];
                    zero[m] = (uint32_t)v;
                    zero[-m] = (uint32_t)(v + t.at(7 - i, k - m).limb[0]);
                }
        e = hipMalloc((void **)&c->enc8_offs, offs.size() * 4);
        if (e == hipSuccess) e = hipMemcpy(c->enc8_offs, offs.data(), offs.size() * 4, hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        pvq_ctx_destroy(c);
        return hip_fail(e);
    }
    *out = c;
    return PVQ_OK;
}

extern "C" int pvq_ctx_destroy(pvq_ctx *c)
{
    if (!c) return PVQ_OK;
    hipError_t first = hipSuccess;
    void *ptrs[6] = {c->tab_u, c->edges, c->sqrtc, c->fast8_blob, c->walk_blob, c->enc8_offs};
    for (void *p : ptrs) {
        if (!p) continue;
        hipError_t e = hipFree(p);
        if (first == hipSuccess) first = e;
    }
    delete c;
    return first == hipSuccess ? PVQ_OK : hip_fail(first);
}

extern "C" int pvq_ctx_info(const pvq_ctx *c, int *D, int *K, int *index_bits, int *scale_bits)
{
    if (!c) return PVQ_E_INVALID_ARG;
    if (D) *D = c->D;
    if (K) *K = c->K;
    if (index_bits) *index_bits = c->index_bits;
    if (scale_bits) *scale_bits = c->scale_bits;
    return PVQ_OK;
}

extern "C" int pvq_size_table_device(int D, int K, int words, uint32_t *table, uint32_t *overflow, void *stream)
{
    if (D < 0 || K < 0 || words < 1 || !table || !overflow) return PVQ_E_INVALID_ARG;
    if (D > 1024 || K > 1023 || words > 16) return PVQ_E_UNSUPPORTED;
    const hipError_t e = pvq_launch_size_table(D, K, words, table, overflow, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_hadamard(const void *X, int dtype, int64_t rows, int64_t cols, int64_t ldx, int block,
                            const uint8_t *signs, int inverse, void *Y, int out_dtype, int64_t ldy, void *stream)
{
    if (rows < 0 || cols < 0 || ldx < cols || ldy < cols) return PVQ_E_INVALID_ARG;
    if ((dtype != PVQ_F32 && dtype != PVQ_BF16) || (out_dtype != PVQ_F32 && out_dtype != PVQ_BF16))
        return PVQ_E_UNSUPPORTED;
    if (block < 8 || block > 8192 || (block & (block - 1)) || cols % block) return PVQ_E_UNSUPPORTED;
    if (rows == 0 || cols == 0) return PVQ_OK;
    if (!X || !Y) return PVQ_E_INVALID_ARG;
    const int64_t isz = dtype == PVQ_F32 ? 4 : 2, osz = out_dtype == PVQ_F32 ? 4 : 2;
    if (((uintptr_t)X & 15) || ((uintptr_t)Y & 15) || (ldx * isz) % 16 || (ldy * osz) % 16 || ((uintptr_t)signs & 7))
        return PVQ_E_ALIGNMENT;
    if (rows * ((cols + 511) / 512) > 0x7FFFFFFF) return PVQ_E_UNSUPPORTED;
    const hipError_t e = pvq_launch_hadamard(X, dtype, rows, cols, ldx, block, signs, inverse ? 1 : 0, Y, out_dtype,
                                             ldy, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_ctx_set_amplitude(pvq_ctx *c, int amplitude)
{
    if (!c || (amplitude != PVQ_AMP_NORM && amplitude != PVQ_AMP_LS)) return PVQ_E_INVALID_ARG;
    c->amplitude = amplitude;
    return PVQ_OK;
}

static int64_t stream_words(int64_t groups, int bits) { return (groups * bits + 31) / 32; }

static int check_shape(const pvq_ctx *c, int64_t rows, int64_t cols)
{
    if (!c || rows < 0 || cols < 0) return PVQ_E_INVALID_ARG;
    if (cols % c->D) return PVQ_E_UNSUPPORTED;
    // 32-bit bit offsets inside a row and 31-bit element counts per launch dimension
    if (cols > (int64_t)1 << 24 || rows > (int64_t)1 << 30) return PVQ_E_UNSUPPORTED;
    return PVQ_OK;
}

extern "C" int pvq_packed_sizes(const pvq_ctx *c, int64_t rows, int64_t cols, size_t *index_bytes,
                                size_t *scale_bytes, size_t *rownorm_bytes)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    int64_t G = cols / c->D;
    if (index_bytes) *index_bytes = (size_t)(rows * stream_words(G, c->index_bits) * 4);
    if (scale_bytes)
        *scale_bytes = (size_t)(c->scale_bits ? rows * stream_words(G, c->scale_bits) * 4 : rows * G * 4);
    if (rownorm_bytes) *rownorm_bytes = (size_t)(rows * 4);
    return PVQ_OK;
}

// ------------------------------------------------------------------------------------------
// the hot path: validation, then launch
// ------------------------------------------------------------------------------------------

static bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

static int check_device(const pvq_ctx *c)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    return dev == c->device ? PVQ_OK : PVQ_E_INVALID_ARG;
}

extern "C" int pvq_encode(const pvq_ctx *c, const void *W, int dtype, int64_t rows, int64_t cols,
                          int64_t ldw, uint32_t *index_out, void *scale_out, float *rownorm_out,
                          int8_t *pulses_out, void *stream)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    if (dtype != PVQ_F32 && dtype != PVQ_BF16) return PVQ_E_INVALID_ARG;
    if (rows == 0 || cols == 0) return PVQ_OK;
    if (!W || !index_out || !scale_out || ldw < cols) return PVQ_E_INVALID_ARG;
    if (c->scale_bits > 0 && !rownorm_out) return PVQ_E_INVALID_ARG;
    size_t esz = dtype == PVQ_F32 ? 4 : 2;
    if (!aligned(W, 16) || (ldw * esz) % 16 || !aligned(index_out, 4) || !aligned(scale_out, 4) ||
        (rownorm_out && !aligned(rownorm_out, 4)) || (pulses_out && !aligned(pulses_out, 16)))
        return PVQ_E_ALIGNMENT;
    if ((rc = check_device(c))) return rc;

    pvq_encode_args a;
    a.ls_amplitude = c->amplitude == PVQ_AMP_LS ? 1 : 0;
    a.W = W; a.rows = rows; a.cols = cols; a.ldw = ldw; a.groups = cols / c->D;
    a.index_out = index_out; a.scale_out = scale_out; a.rownorm_out = rownorm_out;
    a.pulses_out = pulses_out;
    a.index_row_words = stream_words(a.groups, c->index_bits);
    a.scale_row_words = c->scale_bits ? stream_words(a.groups, c->scale_bits) : 0;
    if (c->wide && pulses_out && c->K > 127) return PVQ_E_UNSUPPORTED;   // int8 cannot hold such pulses
    if (!c->wide && !pvq_encode8_usable(c, a) && !pvq_encode_fits(c, a)) return PVQ_E_UNSUPPORTED;   // rows too long for LDS
    hipError_t e = c->wide ? pvq_wide_launch_encode(c, a, dtype, (hipStream_t)stream)
                   : pvq_encode8_usable(c, a) ? pvq_encode8_launch(c, a, dtype, (hipStream_t)stream)
                                              : pvq_launch_encode(c, a, dtype, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_rotate_encode(const pvq_ctx *c, const void *X, int dtype, int64_t rows, int64_t cols,
                                 int64_t ldx, int block, const uint8_t *signs, uint32_t *index_out,
                                 void *scale_out, float *rownorm_out, void *stream)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    if (dtype != PVQ_F32 && dtype != PVQ_BF16) return PVQ_E_INVALID_ARG;
    const bool long_groups = c->wide && c->D == 128 && c->words <= 12;
    const bool groups_of_8 = !c->wide && c->D == 8 && c->index_bits == 24;
    if (!long_groups && !groups_of_8) return PVQ_E_UNSUPPORTED;
    if (block < (long_groups ? 128 : 8) || block > 8192 || (block & (block - 1)) || cols % block) return PVQ_E_UNSUPPORTED;
    const int lanes = std::min(1024, std::max(256, block / 8));   // of a workgroup: whole blocks of the rotation
    if (long_groups) {
        // a workgroup's groups must fill whole words of the index plane
        if (((int64_t)(lanes / 16) * c->index_bits) % 32) return PVQ_E_UNSUPPORTED;
    }
    pvq_encode_args a;
    a.ls_amplitude = c->amplitude == PVQ_AMP_LS ? 1 : 0;
    a.W = X; a.rows = rows; a.cols = cols; a.ldw = ldx; a.groups = cols / c->D;
    a.index_out = index_out; a.scale_out = scale_out; a.rownorm_out = rownorm_out; a.pulses_out = nullptr;
    a.index_row_words = stream_words(a.groups, c->index_bits);
    a.scale_row_words = c->scale_bits ? stream_words(a.groups, c->scale_bits) : 0;
    // groups of 8: rows of whole chunks of `lanes` groups, at most 4096 groups
    if (groups_of_8 && cols > 0 && !pvq_rotate_encode8_usable(c, a, block)) return PVQ_E_UNSUPPORTED;
    if (rows == 0 || cols == 0) return PVQ_OK;
    if (!X || !index_out || !scale_out || ldx < cols) return PVQ_E_INVALID_ARG;
    if (c->scale_bits > 0 && !rownorm_out) return PVQ_E_INVALID_ARG;
    const size_t esz = dtype == PVQ_F32 ? 4 : 2;
    if (!aligned(X, 16) || (ldx * esz) % 16 || !aligned(index_out, 4) || !aligned(scale_out, 4) || !aligned(signs, 8) ||
        (rownorm_out && !aligned(rownorm_out, 4)))
        return PVQ_E_ALIGNMENT;
    if ((rc = check_device(c))) return rc;
    const hipError_t e = long_groups ? pvq_wide_launch_rotate_encode(c, a, dtype, block, signs, (hipStream_t)stream)
                                     : pvq_rotate_encode8_launch(c, a, dtype, block, signs, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_correct_work_bytes(int64_t rows, size_t *bytes)
{
    if (rows < 0 || rows > (int64_t)1 << 30 || !bytes) return PVQ_E_INVALID_ARG;
    *bytes = (size_t)rows * 256 * sizeof(float);   // two buffers of 128 t values per row, used in turn
    return PVQ_OK;
}

// what pvq_correct and pvq_correct_static check alike; *nothing_to_do for an empty matrix
static int check_correct_args(const pvq_ctx *c, const float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                              int64_t ldu, bool *nothing_to_do)
{
    *nothing_to_do = false;
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    // (a limit of the entry point: at most 2^15 panels of 128 columns, a launch each)
    if (c->wide || (c->D != 8 && c->D != 16 && c->D != 32) || cols % 64 || cols > (int64_t)1 << 22) return PVQ_E_UNSUPPORTED;
    if (rows == 0 || cols == 0) { *nothing_to_do = true; return PVQ_OK; }
    if (!W || !U || ldw < cols || ldu < cols) return PVQ_E_INVALID_ARG;
    if (!aligned(W, 16) || ldw % 4 || !aligned(U, 16) || ldu % 4) return PVQ_E_ALIGNMENT;
    return PVQ_OK;
}

extern "C" int pvq_correct(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                           int64_t ldu, void *work, size_t work_bytes, void *stream)
{
    bool empty;
    int rc = check_correct_args(c, W, rows, cols, ldw, U, ldu, &empty);
    if (rc || empty) return rc;
    if (!work || work_bytes < (size_t)rows * 256 * sizeof(float)) return PVQ_E_INVALID_ARG;
    if (!aligned(work, 16)) return PVQ_E_ALIGNMENT;
    if ((rc = check_device(c))) return rc;
    const bool twice = work_bytes / 2 >= (size_t)rows * 256 * sizeof(float);
    const auto launch = twice ? pvq_launch_correct_two_panels : pvq_launch_correct;
    const hipError_t e = launch(c, W, rows, cols, ldw, U, ldu, (float *)work, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_correct_set_front_tiles(int64_t tiles, int64_t *previous)
{
    // (kept for callers that set and restore it; no launch depends on it)
    static std::atomic<int64_t> value{1536};
    if (tiles < 0) return PVQ_E_INVALID_ARG;
    const int64_t old = value.exchange(tiles);
    if (previous) *previous = old;
    return PVQ_OK;
}

extern "C" int pvq_correct_static_max_rows(int64_t *rows)
{
    if (!rows) return PVQ_E_INVALID_ARG;
    *rows = pvq_correct_static_max_rows();
    return PVQ_OK;
}

extern "C" int pvq_correct_static(const pvq_ctx *c, float *W, int64_t rows, int64_t cols, int64_t ldw, const float *U,
                                  int64_t ldu, void *stream)
{
    bool empty;
    int rc = check_correct_args(c, W, rows, cols, ldw, U, ldu, &empty);
    if (rc || empty) return rc;
    if (rows > pvq_correct_static_max_rows()) return PVQ_E_UNSUPPORTED;   // more rows than the static buffer holds
    if ((rc = check_device(c))) return rc;
    const hipError_t e = pvq_launch_correct_static(c, W, rows, cols, ldw, U, ldu, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

static int fill_decode_args(const pvq_ctx *c, pvq_decode_args &a, const uint32_t *index,
                            const void *scale, const float *rownorm, int64_t rows, int64_t cols)
{
    if (!index || !scale) return PVQ_E_INVALID_ARG;
    if (c->scale_bits > 0 && !rownorm) return PVQ_E_INVALID_ARG;
    if (!aligned(index, 4) || !aligned(scale, 4) || (rownorm && !aligned(rownorm, 4))) return PVQ_E_ALIGNMENT;
    memset(&a, 0, sizeof a);
    a.index = index; a.scale = scale; a.rownorm = rownorm;
    a.rows = rows; a.cols = cols; a.groups = cols / c->D;
    a.index_row_words = stream_words(a.groups, c->index_bits);
    a.scale_row_words = c->scale_bits ? stream_words(a.groups, c->scale_bits) : 0;
    return PVQ_OK;
}

// The table decoder for groups of 8 copies 155 KB of tables into every unit's LDS before its first group; the
// coordinate-by-coordinate decoder starts with 7 KB.  Launches in a row, K = 16, 2-bit codes, table / walk, us:
//                512 x 512    1024 x 8192   2048 x 8192   3072 x 8192   4096 x 8192   8192 x 8192   28672 x 8192
//   to bf16      23.8 /  3.2   19.7 / 10.2   20.9 / 14.9   20.7 / 18.7   21.3 / 22.7   34.0 / 38.9   126 / 143
//   to float16   24.2 /  3.2   21.3 / 10.7   22.6 / 16.3   22.6 / 20.1   23.3 / 24.6   38.0 / 41.8   131 / 149
//   to float32   26.1 /  3.3   21.9 / 11.3   22.2 / 16.9   23.5 / 22.5   29.2 / 28.4   62.9 / 64.7   247 / 263
// The line (1.5 M groups, which a test states) was drawn with an earlier walk, from 1024 x 8192 and 2048 x 8192: by these
// times it would lie at 4 M groups, whatever the type.  (K = 13 would be the walk's up to the largest matrix: 28672 x 8192 to
// bf16 184 / 139, to float32 281 / 259.)
static std::atomic<int64_t> g_table_decoder_min_groups{1572864};

static bool table_decoder_pays(const pvq_ctx *c, const pvq_decode_args &a)
{
    return pvq_fast8_decode_usable(c, a) && a.rows * a.groups >= g_table_decoder_min_groups.load(std::memory_order_relaxed);
}

extern "C" int pvq_decode_set_table_decoder_min_groups(int64_t groups, int64_t *previous)
{
    if (groups < 0) return PVQ_E_INVALID_ARG;
    const int64_t old = g_table_decoder_min_groups.exchange(groups);
    if (previous) *previous = old;
    return PVQ_OK;
}

extern "C" int pvq_decode(const pvq_ctx *c, const uint32_t *index, const void *scale,
                          const float *rownorm, int64_t rows, int64_t cols, void *W_out,
                          int out_dtype, int64_t ldw, void *stream)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    if (out_dtype != PVQ_F32 && out_dtype != PVQ_F16 && out_dtype != PVQ_BF16) return PVQ_E_INVALID_ARG;
    if (rows == 0 || cols == 0) return PVQ_OK;
    if (!W_out || ldw < cols) return PVQ_E_INVALID_ARG;
    size_t esz = out_dtype == PVQ_F32 ? 4 : 2;
    if (!aligned(W_out, 16) || (ldw * esz) % 16) return PVQ_E_ALIGNMENT;
    pvq_decode_args a;
    if ((rc = fill_decode_args(c, a, index, scale, rownorm, rows, cols))) return rc;
    if ((rc = check_device(c))) return rc;
    a.W_out = W_out; a.ldw = ldw;
    hipError_t e = c->wide ? pvq_wide_launch_decode(c, a, out_dtype, (hipStream_t)stream)
                   : table_decoder_pays(c, a) ? pvq_fast8_launch_decode(c, a, out_dtype, (hipStream_t)stream)
                                              : pvq_walk_launch_decode(c, a, out_dtype, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

static int decode_gemv(const pvq_ctx *c, const uint32_t *index, const void *scale, const float *rownorm, int64_t rows,
                       int64_t cols, const void *x, int batch, int64_t ldx, float *y, int64_t ldy, void *stream, int decoder,
                       int tile_rows)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    if (batch < 0) return PVQ_E_INVALID_ARG;
    if (batch > 16 || (c && c->wide)) return PVQ_E_UNSUPPORTED;
    if (rows == 0 || batch == 0) return PVQ_OK;
    if (!y || ldy < rows) return PVQ_E_INVALID_ARG;
    if (!aligned(y, 4)) return PVQ_E_ALIGNMENT;
    pvq_decode_args a;
    if (cols == 0) {
        // an empty sum: y = 0
        hipError_t e = hipSuccess;
        for (int b = 0; b < batch && e == hipSuccess; b++)
            e = pvq_launch_fill_zero(y + (int64_t)b * ldy, rows, (hipStream_t)stream);
        return e == hipSuccess ? PVQ_OK : hip_fail(e);
    }
    if (!x || ldx < cols) return PVQ_E_INVALID_ARG;
    if (!aligned(x, 16) || ldx % 8) return PVQ_E_ALIGNMENT;
    if ((rc = fill_decode_args(c, a, index, scale, rownorm, rows, cols))) return rc;
    if ((rc = check_device(c))) return rc;
    a.x = x; a.batch = batch; a.ldx = ldx; a.y = y; a.ldy = ldy;
    if (decoder == PVQ_PRODUCT_TABLE && !pvq_fast8_gemv_usable(c, a)) return PVQ_E_UNSUPPORTED;
    const bool table = decoder == PVQ_PRODUCT_TABLE || (decoder == PVQ_PRODUCT_BY_RULE && pvq_fast8_gemv_pays(c, a));
    hipError_t e = table ? pvq_fast8_launch_gemv(c, a, (hipStream_t)stream)
                         : pvq_walk_launch_gemv(c, a, tile_rows, (hipStream_t)stream);
    return e == hipSuccess ? PVQ_OK : hip_fail(e);
}

extern "C" int pvq_decode_gemv(const pvq_ctx *c, const uint32_t *index, const void *scale,
                               const float *rownorm, int64_t rows, int64_t cols, const void *x,
                               int batch, int64_t ldx, float *y, int64_t ldy, void *stream)
{
    return decode_gemv(c, index, scale, rownorm, rows, cols, x, batch, ldx, y, ldy, stream, PVQ_PRODUCT_BY_RULE, 0);
}

extern "C" int pvq_decode_gemv_on(const pvq_ctx *c, const uint32_t *index, const void *scale, const float *rownorm, int64_t rows,
                                  int64_t cols, const void *x, int batch, int64_t ldx, float *y, int64_t ldy, void *stream,
                                  int decoder, int tile_rows)
{
    if (decoder != PVQ_PRODUCT_TABLE && decoder != PVQ_PRODUCT_WALK) return PVQ_E_INVALID_ARG;
    if (tile_rows != 0 && (decoder != PVQ_PRODUCT_WALK || (tile_rows != 4 && tile_rows != 16 && (tile_rows != 8 || batch > 8)))) return PVQ_E_INVALID_ARG;
    return decode_gemv(c, index, scale, rownorm, rows, cols, x, batch, ldx, y, ldy, stream, decoder, tile_rows);
}

extern "C" int pvq_decode_gemv_plan(const pvq_ctx *c, int64_t rows, int64_t cols, int batch, int *kinds, int *nvecs,
                                    int max_passes, int *passes)
{
    int rc = check_shape(c, rows, cols);
    if (rc) return rc;
    if (!kinds || !nvecs || !passes || batch < 1 || batch > 16 || max_passes < 1) return PVQ_E_INVALID_ARG;
    if (c->wide) return PVQ_E_UNSUPPORTED;
    pvq_decode_args a;
    memset(&a, 0, sizeof a);
    a.rows = rows; a.cols = cols; a.groups = cols / c->D; a.batch = batch;
    pvq_gemv_pass plan[16];
    int n = 1;
    plan[0] = {PVQ_PASS_GENERIC, batch};
    if (pvq_fast8_gemv_pays(c, a)) n = pvq_fast8_plan_gemv(c, a, plan);
    if (n > max_passes) return PVQ_E_INVALID_ARG;
    for (int i = 0; i < n; i++) { kinds[i] = plan[i].kind; nvecs[i] = plan[i].nvec; }
    *passes = n;
    return PVQ_OK;
}

// ------------------------------------------------------------------------------------------
// host replay of the coordinate-by-coordinate decoder's tables
// ------------------------------------------------------------------------------------------

namespace {

// App. B.3 as printed (with the corrections of the boundary's decode contract), in 128-bit integers
void plain_unrank(const SizeTable &t, int D, int K, u128 c, int *y)
{
    int k = K;
    u128 r = c;
    for (int i = 0; i < D - 1; i++) {
        const int dp = D - 1 - i;
        y[i] = 0;
        if (k == 0) continue;
        if (r < low128(t.at(dp, k))) continue;
        r -= low128(t.at(dp, k));
        int j = 1;
        while (j < k && r >= 2 * low128(t.at(dp, k - j))) { r -= 2 * low128(t.at(dp, k - j)); j++; }
        if (r < low128(t.at(dp, k - j))) y[i] = j; else { y[i] = -j; r -= low128(t.at(dp, k - j)); }
        k -= j;
    }
    y[D - 1] = r == 0 ? k : -k;
}

template <int D, int W, int DX, int DA, int DB>
uint64_t replay_walk(const SizeTable &t, int K, const std::vector<unsigned char> &blob, const pvq_walk_params &p,
                     uint64_t seed, uint64_t count)
{
    using T = typename pvq_walk::wide<W>::type;
    const u128 total = low128(t.at(D, K));
    uint64_t bad = 0, state = seed;
    auto next64 = [&]() {   // splitmix64
        uint64_t z = (state += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    for (uint64_t n = 0; n < count; n++) {
        u128 c;
        if (n < 4) c = n == 0 ? 0 : n == 1 ? total - 1 : n == 2 ? total / 2 : total / 3;   // ends and middles first
        else {
            c = (((u128)next64() << 64) | next64()) % total;
            // a third of the samples near the start of the range, where long runs of equal coordinates lie
            if (n % 3 == 0) c >>= (next64() % 100);
        }
        int want[D], got[D];
        plain_unrank(t, D, K, c, want);
        int n2w = 0;
        for (int i = 0; i < D; i++) n2w += want[i] * want[i];
        auto emit = [&](int i, float minus_y) { got[i] = -(int)minus_y; };
        auto equal = [&](float n2) {
            bool same = n2 == (float)n2w;
            for (int i = 0; i < D; i++) same = same && got[i] == want[i];
            return same;
        };
        // both ways to the second threshold (the kernels differ in which they take)
        bool same = equal(pvq_walk::unrank_walk<D, W, DX, DA, DB, 0>((T)c, blob.data(), p, emit));
        same = equal(pvq_walk::unrank_walk<D, W, DX, DA, DB, 1>((T)c, blob.data(), p, emit)) && same;
        bad += !same;
    }
    return bad;
}

}  // namespace

extern "C" int pvq_walk_tables_selftest(int D, int K, uint64_t seed, uint64_t count, uint64_t *mismatches,
                                        int *schedule, uint32_t *table_bytes)
{
    if (!mismatches) return PVQ_E_INVALID_ARG;
    if ((D != 8 && D != 16 && D != 32) || K < 1 || K > 127) return PVQ_E_UNSUPPORTED;
    SizeTable t(D, K);
    if (t.overflow) return PVQ_E_UNSUPPORTED;
    const int bits = t.index_bits();
    if (bits < 1 || bits > 128 || t.at(D, K).bit_length() > 128) return PVQ_E_UNSUPPORTED;
    const int words = bits <= 32 ? 1 : (bits <= 64 ? 2 : 4);
    if (t.at(D, K).bit_length() > 32 * words) return PVQ_E_UNSUPPORTED;
    std::vector<unsigned char> blob;
    pvq_walk_params p;
    if (!build_walk_tables(t, D, K, words, blob, p)) return PVQ_E_UNSUPPORTED;
    if (schedule) { schedule[0] = p.dA; schedule[1] = p.dB; }
    if (table_bytes) *table_bytes = p.bytes;
#define PVQ_WALK_REPLAY(D_, W_, DX_, DA_, DB_) (*mismatches = replay_walk<D_, W_, DX_, DA_, DB_>(t, K, blob, p, seed, count), PVQ_OK)
    PVQ_WALK_DISPATCH(PVQ_WALK_REPLAY, D, words, p.dX, p.dA, p.dB);
#undef PVQ_WALK_REPLAY
}
