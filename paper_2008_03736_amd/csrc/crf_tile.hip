// crf_tile.hip -- the chart recursions in 4 x 4 tiles of spans.
//
// The same recursions as crf_kernels.hip (inside with the outside beside it,
// and CKY), for unlabelled sentences, organised so that a step advances four
// span widths at once and a lane owns a whole tile of spans: in LDS up to 139
// words, in the workspace past that.
//
// Fence posts are cut into m = n/4 + 1 blocks of four; tile (I,J), I <= J,
// holds the spans from a post of block I to a post of block J.  Stage t
// finishes the inside of every tile of tile diagonal D = J - I = t and the
// outside of every tile of diagonal m - t: m + 1 stages and barriers where a
// step per width takes n - 1.  A lane takes one tile (or G = 2 .. 16 lanes
// share one, each with every G-th product, when a stage has few tiles):
//   - the splits in the blocks strictly between (inside) or outside I..J
//     (outside) are t - 1 products of two finished 4 x 4 tiles, 64 FMAs on
//     eight 16-byte LDS reads each, the same count for every lane of a stage;
//   - the splits inside blocks I and J, the only ones whose other part lies
//     in the tile itself, are 48 further terms in the lane's registers.
// Nothing is decoded per span, no lane reduces for a span (but for G > 1),
// and the serial chain of a stage is one lane's 7-deep chain over its tile.
//
// Storage (float32).  Two m x m squares of tiles per sentence, P and Q:
//   P[I][J], I <= J: alpha        P[J][I], I < J: O' transposed
//   Q[I][J], I <= J: O'           Q[J][I], I < J: alpha transposed
// (O' the outside score plus the span's own score, as in crf_kernels.hip).
// Every product is then acc[r][c] += X[k][r] Y[k][c] over the rows k of two
// tiles in one row of tiles K: inside X = Q[K][I], Y = P[K][J], I < K < J;
// outside X = P[K][I], Y = Q[K][J], K < I or K > J.  Until a tile is finished
// P[I][J] and Q[I][J] both hold its scores.
//
// A bundle's S sentences (equal m, any lengths) interleave sentence-minor:
// tile (K,J) of sentence sb is slot K*rp + J*S + sb, 64 bytes, its row k at
// 16-byte piece (k + (K*S + sb)/2) mod 4.  Consecutive lanes take consecutive
// f = I*S + sb, so eight lanes' pieces cover the 32 banks (rp even); X and Y
// of a product share K and sb, hence the rotation: the sum over k does not
// mind in which order a lane meets its rows, and piece p of both tiles is a
// constant offset.
//
// What bounds it: latency, in a stage's chain of address arithmetic, one LDS
// round trip, the products (a wavefront issues an independent vector
// instruction every 5 to 6 cycles, a dependent one every 9), the lanes'
// combining, the finish and the barrier: about 4,800 cycles a stage (26 stages of
// one 99-word sentence with marginals in 57 us, launch and ends included) where a
// width step took 2,000, for four widths; LDS adds 3.4 conflict cycles to an
// instruction (the lanes that share a tile), a seventh of the busy cycles; not HBM.  Measured against the one-width-a-step
// kernels (us): 5,000 mixed sentences fused 96.5 -> 70.8, 2,000 longer ones
// 130.5 -> 112.9, MBR of 1,700 134.5 -> 114.0, gold loss of 200 39.4 -> 33.6,
// 32 short ones fused 26.7 -> 23.0, CKY of one sentence of 23 words 14.8 ->
// 13.0.  Tried and dropped: 512 threads at 128 registers instead of 256 at 256
// (mixed 72.6 -> 82.8, longer 113 -> 134), a second register buffer for the
// next product's tiles (mixed 70.8 -> 72.6).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "crf_internal.h"

namespace crf {
namespace {

constexpr float LOG2E_F = 1.4426950408889634f;
constexpr double LN2_D = 0.69314718055994530942;
// "No split" and the score of a cell that is no span: far below any chart
// value, and finite, so that sums and differences of two stay finite.
constexpr float NEG = -1.0e30f;
// Linear-domain range (see inside_block_impl): a larger value, or a root
// outside [2^-100, 2^100], sends the bundle to the log domain.  So do sums
// that lost their digits, or themselves, to underflow where that matters.  A
// sum below 2^-100 that is not zero is a sign of it (zero is what spans get
// whose every tree holds a near-forbidden score); it is off by some 2^-142 (of
// at most 2^8 terms, 2^-150 each), times 2^R by the rescales that follow, and
// log Z and the marginals by that times the span's outside over Z (a lost
// outside sum: times its inside).  So where a sentence has a low sum and its
// largest value or sum, times 2^R, exceeds 2^kHarmLog2 Z, its bundle's spans are
// looked at one by one, and it is redone when that holds of the outside of a
// span whose inside sum was below 2^-100 (or lost whole), or the other way
// round, with 2^kSpanHarmLog2 and the rescales of that span: 2^-26 at most a
// span, of which a few come near it.  (The stages look at a quarter of the
// spans, the tiles' diagonals, hence the lower bound for the sentence.  The log
// domain's own error is larger than what is let through: 24 sentences of 200
// words at deviation 4, marginals 3.0e-6 off (2-norm) after a redo in 772 us,
// 1.0e-6 without in 232.  64 of 256 words at deviation 3, a twentieth of the
// spans near-forbidden: two batches in ten hold a sentence whose largest values
// call for the look, which finds nothing: fused 1,615 us with a redo, 531 so.)
// Calls without the outside redo any bundle with a low sum.
constexpr uint32_t kLinLowBits = 0x0D800000u;   // 2^-100
constexpr uint32_t kLinMaxBits = 0x71800000u;   // 2^100; infinities and NaN compare above it
constexpr float kLinMin = 0x1p-100f, kLinMax = 0x1p+100f;
constexpr uint32_t kLinTopBits = 0x4F800000u;   // 2^32: larger values and sums are noted
constexpr float kLinTopLog2 = 32.f, kHarmLog2 = 100.f, kSpanHarmLog2 = 116.f;
constexpr int kGoldMark = 0x7FBADBAD;           // a NaN bit pattern: no finite chart value has it

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
// log2 of a positive normal float: the exact exponent plus the float32 log2
// of the mantissa.
__device__ __forceinline__ double log2_split(float x) {
    return (double)__builtin_amdgcn_frexp_expf(x) + (double)fast_log2(__builtin_amdgcn_frexp_mantf(x));
}
// a / d for 0 <= a < 2^24, inv = 1.0f / d.
__device__ __forceinline__ int div_small(int a, int d, float inv) {
    int q = (int)((float)a * inv);
    q += ((q + 1) * d <= a) ? 1 : 0;
    q -= (q * d > a) ? 1 : 0;
    return q;
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __builtin_bit_cast(float, dpp_i<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = dpp_i<CTRL>((int)(uint32_t)u), hi = dpp_i<CTRL>((int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
// row_ror:n inside each 16-lane row.  Lanes sharing a tile are the ones whose
// lane numbers differ in the top lg bits of the low four, so rotations by 8,
// 4, 2, 1 in that order leave the combined value in all of them.
constexpr int kRor8 = 0x128, kRor4 = 0x124, kRor2 = 0x122, kRor1 = 0x121;

typedef float f4 __attribute__((ext_vector_type(4)));
// a 16-byte access to global memory that is only 4-byte aligned
typedef f4 f4u __attribute__((aligned(4)));

struct Tile {
    float v[4][4];
};

// (offsets unsigned: a workspace access is then a uniform base and a 32-bit
// offset, with no 64-bit address per lane)
__device__ __forceinline__ f4 ld4(const char *sm, int off) { return *reinterpret_cast<const f4 *>(sm + (uint32_t)off); }
__device__ __forceinline__ void st4(char *sm, int off, f4 v) { *reinterpret_cast<f4 *>(sm + (uint32_t)off) = v; }

// ---------------------------------------------------------------------------
// The two domains.  LIN: the chart holds exp2 of the shifted, log2-scaled
// values, sums are sums.  Otherwise it holds those values, and sums are
// log-sum-exps (only bundles that leave float32's range come here).
template <bool LIN>
struct Dom {
    static constexpr float zero = LIN ? 0.f : NEG, one = LIN ? 1.f : 0.f;
    __device__ static __forceinline__ float add(float a, float b) {
        if constexpr (LIN) return a + b;
        const float m = __builtin_fmaxf(a, b);
        return m + fast_log2(fast_exp2(a - m) + fast_exp2(b - m));
    }
    __device__ static __forceinline__ float mul(float a, float b) {
        if constexpr (LIN) return a * b;
        return a + b;
    }
    // own term of a span: its natural-unit score and its sentence's shift
    __device__ static __forceinline__ float own(float s, float d) {
        const float x = __builtin_fmaf(s, LOG2E_F, d);
        if constexpr (LIN) return fast_exp2(x);
        return x;
    }
    __device__ static __forceinline__ float log2(float x) {
        if constexpr (LIN) return fast_log2(x);
        return x;
    }
};

// A tile's sums while its terms come in.  LIN: the sums.  Otherwise a pair per
// span, its largest term and the sum of the terms relative to that (2^m s), so
// that a span's sum is rounded at the chart's magnitude once, however many
// products and lanes it takes (a log2 per product and level rounded it every
// time: 40 sentences of 60 words at deviation 8, marginals 9.6e-6 off in the
// 2-norm and 143 us; 7.4e-6 and 127 so).
template <bool LIN>
struct Acc {
    Tile v;
    __device__ __forceinline__ Acc() {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) v.v[r][c] = 0.f;
    }
    // += sum_k x[k][r] y[k][c]
    __device__ __forceinline__ void product(const f4 (&x)[4], const f4 (&y)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) v.v[r][c] = __builtin_fmaf(x[k][r], y[k][c], v.v[r][c]);
    }
    template <int CTRL>
    __device__ __forceinline__ void combine() {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) v.v[r][c] += dpp_f<CTRL>(v.v[r][c]);
    }
    __device__ __forceinline__ void set_one(int r, int c, bool yes) { v.v[r][c] = yes ? 1.f : v.v[r][c]; }
};
struct Log_pair {
    float m = NEG, s = 1.f;
    __device__ __forceinline__ void add(float x) {
        const float n = __builtin_fmaxf(m, x);
        s = s * fast_exp2(m - n) + fast_exp2(x - n);
        m = n;
    }
    template <int CTRL>
    __device__ __forceinline__ void combine() {
        const float m2 = dpp_f<CTRL>(m), s2 = dpp_f<CTRL>(s), n = __builtin_fmaxf(m, m2);
        s = s * fast_exp2(m - n) + s2 * fast_exp2(m2 - n);
        m = n;
    }
    __device__ __forceinline__ float value() const { return m + fast_log2(s); }
};
template <>
struct Acc<false> {
    Log_pair v[4][4];
    __device__ __forceinline__ void product(const f4 (&x)[4], const f4 (&y)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Log_pair &p = v[r][c];
                float n = p.m;
#pragma unroll
                for (int k = 0; k < 4; ++k) n = __builtin_fmaxf(n, x[k][r] + y[k][c]);
                float s = p.s * fast_exp2(p.m - n);
#pragma unroll
                for (int k = 0; k < 4; ++k) s += fast_exp2(x[k][r] + y[k][c] - n);
                p.m = n;
                p.s = s;
            }
    }
    template <int CTRL>
    __device__ __forceinline__ void combine() {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[r][c].template combine<CTRL>();
    }
    __device__ __forceinline__ void set_one(int r, int c, bool yes) {
        v[r][c].m = yes ? 0.f : v[r][c].m;
        v[r][c].s = yes ? 1.f : v[r][c].s;
    }
};

// One span's sum: its accumulator and up to six further terms.
template <bool LIN>
struct Span_sum {
    float t;
    __device__ __forceinline__ Span_sum(const Acc<LIN> &a, int r, int c) : t(a.v.v[r][c]) {}
    __device__ __forceinline__ void add(float x) { t += x; }
    __device__ __forceinline__ void fma(float u, float x) { t = __builtin_fmaf(u, x, t); }
    __device__ __forceinline__ float value() const { return t; }
};
template <>
struct Span_sum<false> {
    Log_pair p;
    float term[6];
    int n = 0;   // (known once the loops are unrolled)
    __device__ __forceinline__ Span_sum(const Acc<false> &a, int r, int c) : p(a.v[r][c]) {}
    __device__ __forceinline__ void add(float x) { term[n++] = x; }
    __device__ __forceinline__ void fma(float u, float x) { term[n++] = u + x; }
    __device__ __forceinline__ float value() const {
        float m = p.m;
#pragma unroll
        for (int k = 0; k < 6; ++k) m = k < n ? __builtin_fmaxf(m, term[k]) : m;
        float s = p.s * fast_exp2(p.m - m);
#pragma unroll
        for (int k = 0; k < 6; ++k) s += k < n ? fast_exp2(term[k] - m) : 0.f;
        return m + fast_log2(s);
    }
};

// A bundle's charts (byte offsets from `sm`: the workgroup's LDS, or, GLOB, a
// sentence's slot of the workspace) and tables (from tb, in LDS).  Tile (I,J)
// of sentence sb: alpha at a, O' at o, both transposed at at and ot, rows
// rs(J - I) bytes apart.  In the workspace the four are arrays of their own,
// each by diagonal and row, so that consecutive lanes, which take consecutive
// I of a diagonal, read consecutive 16-byte pieces (64 sentences of 256 words,
// inside and marginals: 466 us with whole tiles side by side, 396 so, part of
// it from the 32-bit offsets).
template <bool GLOB>
struct Io_ctx {
    static constexpr bool kGlob = GLOB;
    int m, S, rpb, qo;   // blocks, sentences, bytes per row of tiles, offset of Q (GLOB: bytes per array)
    uint32_t mag;        // div_magic(S)
    int part, partd, forced, tab;
    char *tb;
    __device__ __forceinline__ int rot(int g) const { return GLOB ? 0 : (g >> 1) & 3; }
    __device__ __forceinline__ int diag(int D) const { return 64 * (D * m - ((D * (D - 1)) >> 1)); }
    __device__ __forceinline__ int rs(int D) const { return GLOB ? 16 * (m - D) : 16; }
    __device__ __forceinline__ int a(int I, int J, int sb) const {
        return GLOB ? diag(J - I) + I * 16 : I * rpb + (J * S + sb) * 64;
    }
    __device__ __forceinline__ int at(int I, int J, int sb) const {
        return qo + (GLOB ? diag(J - I) + I * 16 : J * rpb + (I * S + sb) * 64);
    }
    __device__ __forceinline__ int o(int I, int J, int sb) const {
        return GLOB ? 2 * qo + diag(J - I) + I * 16 : qo + I * rpb + (J * S + sb) * 64;
    }
    __device__ __forceinline__ int ot(int I, int J, int sb) const {
        return GLOB ? 3 * qo + diag(J - I) + I * 16 : J * rpb + (I * S + sb) * 64;
    }
};
template <bool GLOB>
__device__ __forceinline__ Io_ctx<GLOB> io_ctx(const int32_t *rec, char *lds) {
    Io_ctx<GLOB> c;
    c.m = rec[kTrM];
    c.S = GLOB ? 1 : rec[kTrCount];
    c.rpb = rec[kTrPitch] * 64;
    c.mag = (uint32_t)rec[kTrMagic];
    c.qo = GLOB ? 32 * c.m * (c.m + 1) : c.m * c.rpb;
    c.part = GLOB ? 0 : 2 * c.qo;
    c.partd = c.part + 16 * c.m * c.S;
    c.forced = c.partd + 8 * c.m * c.S;
    c.tab = c.forced + 8 * c.S;
    c.tb = lds;
    return c;
}
// per-sentence tables: word `which` of sentence sb
// (kTabTop: the bits of the largest value or sum noted; kTabR: log2 of what
// rescales may have added to an early sum's error)
enum { kTabD = 0, kTabDl, kTabG, kTabLz, kTabId, kTabN, kTabTop, kTabR, kTabWords };
// a bundle's flags: out of range, a low sum, early values far from 1, and low
// sums that may matter
enum { kFlagOut = 0, kFlagLow, kFlagWide, kFlagHarm, kFlags };
template <typename T, typename CX>
__device__ __forceinline__ T &tab(const CX &c, int which, int sb) {
    return *reinterpret_cast<T *>(c.tb + c.tab + 4 * (which * c.S + sb));
}
static_assert(kTabWords == kTileTabWords, "tile_io_bytes counts the tables");

// Hides a value from the optimiser: what follows from it is computed where it
// is used, not hoisted out of the stage loops into registers that spill.
__device__ __forceinline__ int here(int v) {   // a uniform value
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ int here_lane(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ int this_thread() { return here_lane((int)threadIdx.x); }

// Which tile and which share of its products a lane of wavefront task w takes
// with 2^lg lanes per tile.
struct Lane_share {
    int f, q;
};
__device__ __forceinline__ Lane_share lane_share(int w, int lg) {
    const int l = this_thread() & 63, low = l & 15;
    return Lane_share{(w * (64 >> lg)) + (low & ((16 >> lg) - 1)) + ((l >> 4) << (4 - lg)), low >> (4 - lg)};
}

// Lanes per tile of a stage whose tiles take np products each: as many as
// the workgroup's wavefronts hold without a second pass (most: the lg at which
// the bundle's m S tiles, of both kinds together, fill them), while a lane's
// saved products (about 70 issue slots each) outweigh the combining levels
// (16 each).
__device__ __forceinline__ int stage_lg(int np, int cin, int cout, int nw, int most) {
    int lg = min(np >= 12 ? 4 : np >= 6 ? 3 : np >= 3 ? 2 : np >> 1, most);
    // (the two kinds start on wavefronts of their own)
    return lg > 0 && (((cin << lg) + 63) >> 6) + (((cout << lg) + 63) >> 6) > nw ? lg - 1 : lg;
}
__device__ __forceinline__ int lanes_lg(int tiles, int nw) {
    const int room = 64 * nw / tiles;
    return room >= 16 ? 4 : room >= 8 ? 3 : room >= 4 ? 2 : room >= 2 ? 1 : 0;
}

// The spans of two and three words of a diagonal tile of P (the others it
// holds are words, whose value is one): exactly the words read, so that no
// load waits for an unused register.
struct Diag3 {
    float d02, d03, d13;
};
__device__ __forceinline__ Diag3 diag3(const char *sm, int at, int rot, int rs) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 a = *reinterpret_cast<const f2 *>(sm + (uint32_t)(at + rot * rs + 8));
    return Diag3{a[0], a[1], *reinterpret_cast<const float *>(sm + (uint32_t)(at + ((1 + rot) & 3) * rs + 12))};
}

// The inside of a tile from its products, its own terms and the diagonal
// tiles of its blocks: x[r][c] = e[r][c] (acc[r][c] + the splits inside the
// blocks); sum: the bracket on the tile's diagonal.  word: the tile's lower
// left span is a word (diagonal 1).
template <bool LIN>
__device__ __forceinline__ void finish_inside(Tile &x, float (&sum)[4], const Acc<LIN> &acc, const Tile &e, const Diag3 &U,
                                              const Diag3 &V, bool word) {
    typedef Dom<LIN> Dm;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 3; r >= 0; --r) {
            Span_sum<LIN> q(acc, r, c);
            if (r < 3) q.add(x.v[r + 1][c]);
            if (r < 2) q.fma(r == 0 ? U.d02 : U.d13, x.v[r + 2][c]);
            if (r < 1) q.fma(U.d03, x.v[3][c]);
            if (c > 0) q.add(x.v[r][c - 1]);
            if (c > 1) q.fma(c == 2 ? V.d02 : V.d13, x.v[r][c - 2]);
            if (c > 2) q.fma(V.d03, x.v[r][0]);
            const float t = q.value();
            if (r == c) sum[r] = t;
            x.v[r][c] = Dm::mul(e.v[r][c], t);
            if (r == 3 && c == 0) x.v[3][0] = word ? Dm::one : x.v[3][0];   // a word
        }
}

// One wavefront's share of a stage's tiles of one kind: inside of diagonal
// D (OUT = false) or outside of diagonal D; D >= 1 for the inside (diagonal 0
// is inside_diagonal).  cnt tiles, np products each.  mark: sums below it set
// the flags.
template <bool LIN, bool OUT, typename CX>
__device__ __forceinline__ void tile_task(const CX &cx, char *sm, int D, int np, int cnt, int w, int lg, uint32_t mark,
                                          int *flags) {
    typedef Dom<LIN> Dm;
    const int m = cx.m, S = cx.S;
    const Lane_share ls = lane_share(here(w), here(lg));
    const bool act = ls.f < cnt && ls.q == 0;
    const int f = here_lane(ls.f < cnt ? ls.f : cnt - 1);
    const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * S, J = I + D;
    const int gi = f, gj = f + D * S;   // I*S + sb, J*S + sb

    // The tile's scores, its sentence's shift and the diagonal tiles of I
    // and J (their spans of two and three words).
    const int own_at = OUT ? cx.o(I, J, sb) : cx.a(I, J, sb), ri = cx.rot(gi), rj = cx.rot(gj), rs = cx.rs(D);
    f4 raw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) raw[r] = ld4(sm, own_at + ((r + ri) & 3) * rs);
    const float d = tab<float>(cx, kTabD, sb);
    const Diag3 U = diag3(sm, cx.a(I, I, sb), ri, cx.rs(0)), V = diag3(sm, cx.a(J, J, sb), rj, cx.rs(0));

    // Products, the first one's tiles in flight while the own terms are taken.
    // In the workspace, where a lane may have a hundred in a row, kSum at a time
    // into a sum of their own, which keeps the rounding of one long chain of
    // additions out of the charts (64 sentences of 256 words: 1.4e-6 off at
    // most in one chain, 1.2e-6 so, both in 527 us).
    const int iters = (np + (1 << lg) - 1) >> lg;
    constexpr int kSum = 4;
    struct Pair {
        f4 x[4], y[4];
    } pr;
    const int bx = (OUT ? 0 : cx.qo) + gi * 64, by = (OUT ? cx.qo : 0) + gj * 64;
    const int lim = m * cx.rpb, step = cx.rpb << lg, last = ((OUT ? J : I) + np) * cx.rpb;
    int off = ((OUT ? J : I) + 1 + ls.q) * cx.rpb;
    auto load_at = [&](Pair &q, int ax, int rx, int ay, int ry) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            q.x[k] = ld4(sm, ax + rx * k);
            q.y[k] = ld4(sm, ay + ry * k);
        }
    };
    auto load = [&](Pair &q, int it) {   // (a lane past its last product reads the tile's last one again)
        if constexpr (CX::kGlob) {
            const int p = min(ls.q + (it << lg), np - 1);
            if constexpr (!OUT) {
                load_at(q, cx.qo + cx.diag(p + 1) + I * 16, cx.rs(p + 1), cx.diag(D - p - 1) + (I + p + 1) * 16,
                        cx.rs(D - p - 1));
            } else {
                const int K = J + 1 + p;
                const bool right = K < m;
                const int L = K - m;   // the block left of I
                load_at(q, right ? 3 * cx.qo + cx.diag(K - I) + I * 16 : cx.diag(I - L) + L * 16, cx.rs(right ? K - I : I - L),
                        right ? cx.qo + cx.diag(K - J) + J * 16 : 2 * cx.qo + cx.diag(J - L) + L * 16,
                        cx.rs(right ? K - J : J - L));
            }
        } else {
            const int o = (int)(OUT ? tile_row_outside(off, last, lim) : tile_row_inside(off, last));
            load_at(q, bx + o, 16, by + o, 16);
            off += step;
        }
    };
    if (iters > 0) load(pr, 0);
    Acc<LIN> acc;
    Tile e;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) e.v[r][c] = Dm::own(raw[r][c], d);
    auto run = [&](Acc<LIN> &sum, int i0, int i1) {
#pragma unroll 1
        for (int it = i0; it < i1; ++it) {
            if (it > 0) load(pr, it);
            if (ls.q + (it << lg) < np) sum.product(pr.x, pr.y);
        }
    };
    if constexpr (CX::kGlob && LIN) {
#pragma unroll 1
        for (int i0 = 0; i0 < iters; i0 += kSum) {
            Acc<LIN> part;
            run(part, i0, min(iters, i0 + kSum));
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc.v.v[r][c] += part.v.v[r][c];
        }
    } else {
        run(acc, 0, iters);
    }
    if (lg >= 1) acc.template combine<kRor8>();
    if (lg >= 2) acc.template combine<kRor4>();
    if (lg >= 3) acc.template combine<kRor2>();
    if (lg >= 4) acc.template combine<kRor1>();
    if (D == m - 1) {   // the root (0, n): own term 1; outside score 1
        const int rc = tab<int>(cx, kTabN, sb) - 4 * (m - 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            e.v[0][c] = I == 0 && c == rc ? Dm::one : e.v[0][c];
            if constexpr (OUT) acc.set_one(0, c, I == 0 && c == rc);
        }
    }

    Tile t;
    float sum[4];   // on the tile's diagonal
    if constexpr (!OUT) {
        finish_inside<LIN>(t, sum, acc, e, U, V, D == 1);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 3; c >= 0; --c) {
                Span_sum<LIN> q(acc, r, c);
                if (r > 0) q.add(t.v[r - 1][c]);
                if (r > 1) q.fma(r == 2 ? U.d02 : U.d13, t.v[r - 2][c]);
                if (r > 2) q.fma(U.d03, t.v[0][c]);
                if (c < 3) q.add(t.v[r][c + 1]);
                if (c < 2) q.fma(c == 1 ? V.d13 : V.d02, t.v[r][c + 2]);
                if (c < 1) q.fma(V.d03, t.v[r][3]);
                const float v = q.value();
                if (r == c) sum[r] = v;
                t.v[r][c] = Dm::mul(e.v[r][c], v);
                if (r == 3 && c == 0) t.v[3][0] = D == 1 ? Dm::zero : t.v[3][0];   // a word: no term of any product
            }
    }
    if constexpr (LIN) {   // every value is >= 0, so their sum shows an infinity, a NaN or a value past the range
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) s += (t.v[r][0] + t.v[r][1]) + (t.v[r][2] + t.v[r][3]);
        const uint32_t sb_bits = __builtin_bit_cast(uint32_t, s);
        uint32_t low = 0xFFFFFFFFu, top = sb_bits;   // (zero wraps round to the largest)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t b = __builtin_bit_cast(uint32_t, sum[r]);
            low = min(low, b - 1u);
            top = max(top, b);
        }
        if (low < mark || top > kLinTopBits) {
            if (sb_bits > kLinMaxBits) flags[kFlagOut] = 1;
            if (low < kLinLowBits) flags[kFlagLow] = 1;
            if (mark != kLinLowBits) flags[kFlagWide] = 1;   // (written before the stage that reads it only)
            atomicMax(&tab<uint32_t>(cx, kTabTop, sb), top);
        }
    }
    if (act) {
        const int up = OUT ? cx.o(I, J, sb) : cx.a(I, J, sb), lo = OUT ? cx.ot(I, J, sb) : cx.at(I, J, sb);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            st4(sm, up + ((k + ri) & 3) * rs, f4{t.v[k][0], t.v[k][1], t.v[k][2], t.v[k][3]});
            st4(sm, lo + ((k + rj) & 3) * rs, f4{t.v[0][k], t.v[1][k], t.v[2][k], t.v[3][k]});
        }
    }
}

// Inside of tile diagonal 0: the spans of up to three words inside a block.
// A lane per tile.
template <bool LIN, typename CX>
__device__ __forceinline__ void inside_diagonal(const CX &cx, char *sm, int *flags) {
    typedef Dom<LIN> Dm;
    const int cnt = cx.m * cx.S;
    for (int f = this_thread(); f < cnt; f += (int)blockDim.x) {
        const int I = cx.S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * cx.S;
        const int at = cx.a(I, I, sb), ri = cx.rot(f), rs = cx.rs(0);
        const f4 r0 = ld4(sm, at + ri * rs), r1 = ld4(sm, at + ((1 + ri) & 3) * rs);
        const float d = tab<float>(cx, kTabD, sb);
        const int n = tab<int>(cx, kTabN, sb);
        float e02 = Dm::own(r0[2], d), e13 = Dm::own(r1[3], d), e03 = Dm::own(r0[3], d);
        if (cx.m == 1) {   // the root is in this tile
            e02 = n == 2 ? Dm::one : e02;
            e03 = n == 3 ? Dm::one : e03;
        }
        const float x03 = Dm::mul(e03, Dm::add(e13, e02));
        if constexpr (LIN)
            if (__builtin_bit_cast(uint32_t, e02 + e13 + x03) > kLinMaxBits) flags[kFlagOut] = 1;
        const float z = Dm::zero, o = Dm::one;
        st4(sm, at + ri * rs, f4{z, o, e02, x03});
        st4(sm, at + ((1 + ri) & 3) * rs, f4{z, z, o, e13});
        st4(sm, at + ((2 + ri) & 3) * rs, f4{z, z, z, o});
        st4(sm, at + ((3 + ri) & 3) * rs, f4{z, z, z, z});
    }
}

// Outside of tile diagonal 0 (stage m): the products run over every other
// block, the finish over the three spans of two and three words.
template <bool LIN, typename CX>
__device__ __forceinline__ void outside_diagonal(const CX &cx, char *sm, int w, int lg, int *flags) {
    typedef Dom<LIN> Dm;
    const int m = cx.m, S = cx.S, cnt = m * S, np = m - 1;
    const Lane_share ls = lane_share(w, lg);
    const bool act = ls.f < cnt && ls.q == 0;
    const int f = ls.f < cnt ? ls.f : cnt - 1;
    const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * S;
    const int at = cx.o(I, I, sb), ri = cx.rot(f), rs = cx.rs(0);
    const f4 r0 = ld4(sm, at + ri * rs), r1 = ld4(sm, at + ((1 + ri) & 3) * rs);
    const float d = tab<float>(cx, kTabD, sb);
    const int n = tab<int>(cx, kTabN, sb);
    typename std::conditional<LIN, float, Log_pair>::type s02{}, s13{}, s03{};
    auto term = [](auto &a, float x, float y) {
        if constexpr (LIN) a = __builtin_fmaf(x, y, a);
        else a.add(x + y);
    };
    const int bx = f * 64, by = cx.qo + f * 64, lim = m * cx.rpb, step = cx.rpb << lg;
    int off = (I + 1 + ls.q) * cx.rpb;
    typedef float f2 __attribute__((ext_vector_type(2)));
#pragma unroll 2
    for (int p = ls.q; p < np; p += 1 << lg) {
        const int o = off >= lim ? off - lim : off;
        int ax = bx + o, ay = by + o, rx = 16, ry = 16;
        if constexpr (CX::kGlob) {
            const int K = I + 1 + p, L = K - m;
            ax = K < m ? 3 * cx.qo + cx.diag(K - I) + I * 16 : cx.diag(I - L) + L * 16;
            ay = K < m ? cx.qo + cx.diag(K - I) + I * 16 : 2 * cx.qo + cx.diag(I - L) + L * 16;
            rx = ry = cx.rs(K < m ? K - I : I - L);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // columns 0, 1 of X and 2, 3 of Y
            const f2 x = *reinterpret_cast<const f2 *>(sm + (uint32_t)(ax + rx * k));
            const f2 y = *reinterpret_cast<const f2 *>(sm + (uint32_t)(ay + ry * k + 8));
            term(s02, x[0], y[0]);
            term(s13, x[1], y[1]);
            term(s03, x[0], y[1]);
        }
        off += step;
    }
    auto level = [&](auto &a, auto ctrl) {
        if constexpr (LIN) a += dpp_f<decltype(ctrl)::value>(a);
        else a.template combine<decltype(ctrl)::value>();
    };
    auto combine = [&](auto &a) -> float {
        if (lg >= 1) level(a, std::integral_constant<int, kRor8>{});
        if (lg >= 2) level(a, std::integral_constant<int, kRor4>{});
        if (lg >= 3) level(a, std::integral_constant<int, kRor2>{});
        if (lg >= 4) level(a, std::integral_constant<int, kRor1>{});
        if constexpr (LIN) return a;
        else return a.value();
    };
    float a02 = combine(s02), a13 = combine(s13), a03 = combine(s03);
    float e02 = Dm::own(r0[2], d), e13 = Dm::own(r1[3], d), e03 = Dm::own(r0[3], d);
    if (m == 1) {
        a02 = n == 2 ? Dm::one : a02;
        e02 = n == 2 ? Dm::one : e02;
        a03 = n == 3 ? Dm::one : a03;
        e03 = n == 3 ? Dm::one : e03;
    }
    const float o03 = Dm::mul(e03, a03);
    a02 = Dm::add(a02, o03);
    a13 = Dm::add(a13, o03);
    const float o02 = Dm::mul(e02, a02), o13 = Dm::mul(e13, a13);
    if constexpr (LIN) {
        const uint32_t s = __builtin_bit_cast(uint32_t, o02 + o13 + o03);
        const uint32_t top = max(max(s, __builtin_bit_cast(uint32_t, a03)),
                                 max(__builtin_bit_cast(uint32_t, a02), __builtin_bit_cast(uint32_t, a13)));
        if (top > kLinTopBits) {
            if (s > kLinMaxBits) flags[kFlagOut] = 1;
            atomicMax(&tab<uint32_t>(cx, kTabTop, sb), top);
        }
    }
    if (act) {
        st4(sm, at + ri * rs, f4{Dm::zero, Dm::zero, o02, o03});
        st4(sm, at + ((1 + ri) & 3) * rs, f4{Dm::zero, Dm::zero, Dm::zero, o13});
        if constexpr (CX::kGlob)   // (where gold spans are marked; in LDS the alpha tile's lower half)
#pragma unroll
            for (int k = 0; k < 4; ++k) st4(sm, cx.ot(I, I, sb) + rs * k, f4{0.f, 0.f, 0.f, 0.f});
    }
}

// Stages after which the chart is rescaled, the first >= lo, or 0.  The seed
// (tile_seed) comes from the scores alone: independent scores grow less than
// it says, by 0.4 log2 units a node at deviation 1 and 3 at 5 (30 words), so
// that sentences of 16 to 43 words, whose range holds at deviation 2, need one
// rescale where the scores spread further.  They take it only when a value or
// sum of the stages before lies outside [2^-36, 2^32] (kFlagWide): it costs 3 us
// (40 words: 38 and 41), a redo in the log domain 40 (deviation 3, 76 us).
// The log domain, which never leaves the range, rescales once, a quarter of the
// way, to keep the values and so their rounding small.
constexpr int kWideBlocks = 12;   // fewer blocks: only if flagged
constexpr uint32_t kLinWideBits = 0x2D800000u;   // 2^-36
template <bool LIN>
__device__ __forceinline__ int tile_rescale_after(int lo, int m) {
    if (!LIN) return m >= 5 && m / 4 >= lo ? m / 4 : 0;
    if (m >= kWideBlocks && lo <= 4) return 4;
    if (m >= 5 && m < kWideBlocks && lo <= 2) return m >= 7 ? 3 : 2;
    if (m > 32 && lo <= 12) return 12;
    if (m > 64 && m / 4 >= lo) return m / 4;
    if (m > 24 && m / 2 >= lo) return m / 2;
    return 0;
}

// Sums over the 16 lanes of a row, left in all of them.
__device__ __forceinline__ float row_sum(float v) {
    v += dpp_f<kRor8>(v);
    v += dpp_f<kRor4>(v);
    v += dpp_f<kRor2>(v);
    return v + dpp_f<kRor1>(v);
}
__device__ __forceinline__ float row_max(float v) {
    v = __builtin_fmaxf(v, dpp_f<kRor8>(v));
    v = __builtin_fmaxf(v, dpp_f<kRor4>(v));
    v = __builtin_fmaxf(v, dpp_f<kRor2>(v));
    return __builtin_fmaxf(v, dpp_f<kRor1>(v));
}
__device__ __forceinline__ double row_sum(double v) {
    v += dpp_d<kRor8>(v);
    v += dpp_d<kRor4>(v);
    v += dpp_d<kRor2>(v);
    return v + dpp_d<kRor1>(v);
}

// Growth of log2 alpha per node over a tile's spans (diagonal D >= 1): the
// largest, the sum and the number of log2(x) / (w-1).  Linear domain: spans of
// no value left out.  Log domain: those more than kShiftBand below the tile's
// largest, as growth_shift leaves out whole tiles: they hold near-forbidden
// scores, whose share per node falls with the width (-1e4 in a span of 88
// words is -166, and 5% of such spans moved the shift by 8 a node: marginals
// of 350 words 1e-3 off, 1e-4 without them).
constexpr float kShiftBand = 30.0f;
struct Growth {
    float mx = NEG, sum = 0.f, cnt = 0.f;
};
template <bool LIN>
__device__ __forceinline__ Growth tile_growth(const Tile &x, int D) {
    Growth g;
    auto each = [&](auto &&f) {
#pragma unroll
        for (int j = -3; j <= 3; ++j) {
            const int w = 4 * D + j;
            const float inv = __builtin_amdgcn_rcpf((float)(w > 1 ? w - 1 : 1));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = r + j;
                if (c < 0 || c > 3) continue;
                f(Dom<LIN>::log2(x.v[r][c]) * inv, w >= 2);
            }
        }
    };
    float floor_v = -200.f;
    if constexpr (!LIN) {
        each([&](float v, bool ok) { g.mx = ok ? __builtin_fmaxf(g.mx, v) : g.mx; });
        floor_v = g.mx - kShiftBand;
    }
    each([&](float v, bool ok) {
        const bool in = ok && v > floor_v && (!LIN || v < 200.f);
        if constexpr (LIN) g.mx = in ? __builtin_fmaxf(g.mx, v) : g.mx;
        g.sum += in ? v : 0.f;
        g.cnt += in ? 1.f : 0.f;
    });
    return g;
}
// The shift that a sentence's growth partials (part[I*S + sb], I < blocks)
// call for: linear domain, minus the midpoint of the mean and the largest,
// which keeps the largest values further from float32's limit; log domain,
// minus the mean.  Left in table `which`; add: on top of what it holds.
template <bool LIN, typename CX>
__device__ __forceinline__ void growth_shift(const CX &cx, int blocks, int which) {
    const int gl = this_thread() & 15, S = cx.S;
    for (int sb = this_thread() >> 4; sb < S; sb += (int)blockDim.x >> 4) {
        float mx = NEG, sum = 0.f, c = 0.f;
        if constexpr (!LIN) {
            for (int I = gl; I < blocks; I += 16) mx = __builtin_fmaxf(mx, ld4(cx.tb, cx.part + 16 * (I * S + sb))[0]);
            mx = row_max(mx);
        }
        for (int I = gl; I < blocks; I += 16) {
            const f4 p = ld4(cx.tb, cx.part + 16 * (I * S + sb));
            if constexpr (!LIN) {
                if (!(p[0] > mx - kShiftBand)) continue;   // a tile of near-forbidden spans
            } else {
                mx = __builtin_fmaxf(mx, p[0]);
            }
            sum += p[1];
            c += p[2];
        }
        if constexpr (LIN) mx = row_max(mx);
        sum = row_sum(sum);
        c = row_sum(c);
        if (gl == 0)
            tab<float>(cx, which, sb) = c > 0.f ? (LIN ? -0.5f * (mx + sum / c) : -sum / c) : 0.f;
    }
}

// Score shift (see rescale_chart in crf_kernels.hip): after stage t0 the
// growth per node of each sentence is estimated from its tiles of diagonal
// t0, and the finished values move to the problem with every non-forced score
// shifted by delta.
template <bool LIN, bool REV, typename CX>
__device__ void tile_rescale(const CX &cx, char *sm, int t0) {
    typedef Dom<LIN> Dm;
    const int m = cx.m, S = cx.S, tid = this_thread(), NT = (int)blockDim.x;
    for (int f = tid; f < (m - t0) * S; f += NT) {
        const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, at = cx.a(I, I + t0, f - I * S), rt = cx.rot(f);
        Tile x;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f4 v = ld4(sm, at + ((r + rt) & 3) * cx.rs(t0));
#pragma unroll
            for (int c = 0; c < 4; ++c) x.v[r][c] = v[c];
        }
        const Growth g = tile_growth<LIN>(x, t0);
        st4(cx.tb, cx.part + 16 * f, f4{g.mx, g.sum, g.cnt, 0.f});
    }
    __syncthreads();
    growth_shift<LIN>(cx, m - t0, kTabDl);
    __syncthreads();
    auto move_tile = [&](int at, int rt, int at2, int rt2, int rs, float dl, float base, float dir) {
        // row r, column c of the tile at `at` moves by dl (base + dir (c - r)); copied transposed to at2
        Tile x;
        float fac[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const float k = dl * (base + dir * (float)(j - 3));
            fac[j] = LIN ? fast_exp2(k) : k;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const f4 v = ld4(sm, at + ((r + rt) & 3) * rs);
#pragma unroll
            for (int c = 0; c < 4; ++c) x.v[r][c] = Dm::mul(v[c], fac[c - r + 3]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            st4(sm, at + ((k + rt) & 3) * rs, f4{x.v[k][0], x.v[k][1], x.v[k][2], x.v[k][3]});
            if (at2 >= 0) st4(sm, at2 + ((k + rt2) & 3) * rs, f4{x.v[0][k], x.v[1][k], x.v[2][k], x.v[3][k]});
        }
    };
    // a wavefront per tile diagonal
    const int nw = NT >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    for (int D = wave; D <= t0; D += nw) {
        const int cnt = (m - D) * S;
        for (int f = lane; f < cnt; f += 64) {
            const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * S, J = I + D, gj = f + D * S;
            const float dl = tab<float>(cx, kTabDl, sb);
            move_tile(cx.a(I, J, sb), cx.rot(f), D > 0 ? cx.at(I, J, sb) : -1, cx.rot(gj), cx.rs(D), dl,
                      (float)(4 * D - 1), 1.f);
        }
    }
    if constexpr (REV)
        for (int D = m - t0 + wave; D < m; D += nw) {
            const int cnt = (m - D) * S;
            for (int f = lane; f < cnt; f += 64) {
                const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * S, J = I + D, gj = f + D * S;
                const float dl = tab<float>(cx, kTabDl, sb);
                const int n = tab<int>(cx, kTabN, sb);
                // (cells past the sentence hold zero; their factor may be anything finite)
                move_tile(cx.o(I, J, sb), cx.rot(f), cx.ot(I, J, sb), cx.rot(gj), cx.rs(D), dl,
                          (float)(n - 4 * D), -1.f);
            }
        }
    for (int sb = tid; sb < S; sb += NT) {
        const float dl = tab<float>(cx, kTabDl, sb);
        tab<float>(cx, kTabD, sb) += dl;
        tab<float>(cx, kTabR, sb) += __builtin_fmaxf(dl, 0.f) * (float)(4 * t0 + 2);   // the widest span moved
    }
    __syncthreads();
}

// Forced sums (float64) and the seed of each sentence's shift.  A node of a
// tree adds about log2(4 mean(2^s)) to log2 alpha (four the growth of the
// number of trees), the mean over the scores near it: block I's figure is
// over the spans of tile (I,I+1), near-forbidden scores left out, words and
// the root too; the sentence's shift takes away their mean.
template <typename CX>
__device__ void tile_seed(const CX &cx, char *sm) {
    const int m = cx.m, S = cx.S, tid = this_thread(), NT = (int)blockDim.x;
    for (int f = tid; f < m * S; f += NT) {
        const int I = S > 1 ? (int)__umulhi((uint32_t)f, cx.mag) : f, sb = f - I * S;
        const int n = tab<int>(cx, kTabN, sb), ri = cx.rot(f), rc = n - 4 * (m - 1);
        const int at = cx.a(I, I, sb), at1 = I + 1 < m ? cx.a(I, I + 1, sb) : at;
        const int rs0 = cx.rs(0), rs1 = I + 1 < m ? cx.rs(1) : rs0;
        f4 a[4], b[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            a[r] = ld4(sm, at + ((r + ri) & 3) * rs0);
            b[r] = ld4(sm, at1 + ((r + ri) & 3) * rs1);
        }
        const f4 z = ld4(sm, cx.a(0, m - 1, sb) + cx.rot(sb) * cx.rs(m - 1));   // (row 0 of the root's tile, for I = 0)
        double fs = 4 * I + 1 <= n ? (double)a[0][1] : 0.0;
        fs += 4 * I + 2 <= n ? (double)a[1][2] : 0.0;
        fs += 4 * I + 3 <= n ? (double)a[2][3] : 0.0;
        fs += I + 1 < m ? (double)b[3][0] : 0.0;
        fs += I == 0 && n >= 2 ? (double)(rc == 0 ? z[0] : rc == 1 ? z[1] : rc == 2 ? z[2] : z[3]) : 0.0;
        *reinterpret_cast<double *>(cx.tb + cx.partd + 8 * f) = fs;
        b[3][0] = NEG;
        if (m <= 2 && I == 0)   // the root
#pragma unroll
            for (int c = 0; c < 4; ++c) b[0][c] = c == rc ? NEG : b[0][c];
        if (m == 1) {   // (the tile itself: two spans at most that are neither)
            b[0][1] = b[1][2] = b[2][3] = NEG;
        }
        float mx = NEG;
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = __builtin_fmaxf(mx, __builtin_fmaxf(__builtin_fmaxf(b[r][0], b[r][1]), __builtin_fmaxf(b[r][2], b[r][3])));
        float sum = 0.f, cnt = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                sum += fast_exp2((b[r][c] - mx) * LOG2E_F);
                cnt += b[r][c] > -700.f ? 1.f : 0.f;
            }
        const bool some = cnt > 0.f && (m == 1 || I + 1 < m);
        st4(cx.tb, cx.part + 16 * f, f4{0.f, some ? mx * LOG2E_F + fast_log2(sum) - fast_log2(cnt) + 2.f : 0.f, some ? 1.f : 0.f, 0.f});
    }
    __syncthreads();
    growth_shift<false>(cx, m, kTabD);
    for (int sb = tid >> 4; sb < S; sb += NT >> 4) {   // a 16-lane row per sentence, in a fixed order
        double fs = 0.0;
        for (int I = tid & 15; I < m; I += 16) fs += *reinterpret_cast<const double *>(cx.tb + cx.partd + 8 * (I * S + sb));
        fs = row_sum(fs);
        if ((tid & 15) == 0) *reinterpret_cast<double *>(cx.tb + cx.forced + 8 * sb) = fs;
    }
    __syncthreads();
}

// The walk over a bundle's tile rows in the order of the score rows: rows of
// blocks I and m-1-I share one folded row of m+1 tiles, so consecutive
// threads take consecutive 16-byte pieces of a score row.
struct Row_walk {
    int m, W, per, total;
    float inv_per, inv_w;
    __device__ Row_walk(int m_, int S) : m(m_), W(m_ + 1) {
        per = ((m + 1) / 2) * 4 * W;
        total = per * S;
        inv_per = 1.0f / (float)per;
        inv_w = 1.0f / (float)W;
    }
    struct At {
        int sb, I, J, r;
        bool ok;
    };
    __device__ __forceinline__ At at(int c) const {
        At e;
        const int cc = c < total ? c : 0;
        e.sb = div_small(cc, per, inv_per);
        const int rem = cc - e.sb * per;
        const int u = div_small(rem, W, inv_w), v = rem - u * W, h = u >> 2;
        e.r = u & 3;
        e.I = v < m - h ? h : m - 1 - h;
        e.J = e.I + (v < m - h ? v : v - (m - h));
        e.ok = c < total && (v < m - h || e.I > h);   // odd m: the middle row of tiles is not folded twice
        return e;
    }
};
// The scores (i, 4J .. 4J+3) of a row: in bounds for every row i < n (rows
// from n on, which hold no span, read row n-1): the last ones run into row n,
// which the padded block has, since N1 > n.
__device__ __forceinline__ f4 load_row(const float *sent, int N1, int i, int J, int n) {
    return *reinterpret_cast<const f4u *>(sent + (size_t)min(i, n - 1) * N1 + 4 * J);
}

// Inside (+ marginals) of a bundle: the tile form of inside_block_impl, same
// outputs.  Returns false, having written no output, when a linear-domain
// value leaves float32's range.
template <bool LIN, bool REV, bool GOLD, bool GLOB>
__device__ __forceinline__ bool tile_inside_impl(const KernelPlan &p, const int32_t *rec, char *sm, char *lds,
                                                 const float *__restrict__ scores, const float *__restrict__ grad,
                                                 float *__restrict__ logZ, float *__restrict__ marg,
                                                 const int32_t *__restrict__ gold, float *__restrict__ loss) {
    typedef Dom<LIN> Dm;
    __shared__ int flags[kFlags];
    const int tid = this_thread(), NT = (int)blockDim.x, N1 = p.n1;
    const Io_ctx<GLOB> cx = io_ctx<GLOB>(rec, lds);
    const int m = cx.m, S = cx.S;
    for (int sb = tid; sb < S; sb += NT) {
        const int id = rec[kTrHeader + 2 * sb];
        tab<int>(cx, kTabId, sb) = id;
        tab<int>(cx, kTabN, sb) = rec[kTrHeader + 2 * sb + 1];
        tab<float>(cx, kTabG, sb) = grad ? grad[id] : 1.0f;
        tab<uint32_t>(cx, kTabTop, sb) = 0u;
        tab<float>(cx, kTabR, sb) = 0.f;
    }
    if (tid < kFlags) flags[tid] = 0;
    __syncthreads();

    // Prologue: the score rows into P and Q, at most kTilePieces pieces a
    // thread (the plan's limit), all in flight together.
    const Row_walk rw(m, S);
    const size_t sent_stride = (size_t)N1 * N1;
    f4 piece[kTilePieces];
    // Where a thread has one piece at most, the epilogue stops after the first
    // (a uniform test): the walk is some 40 instructions a piece in the chain
    // of a small bundle (one sentence of 4 words with marginals 9.2 -> 7.9 us,
    // 7.8 on the width-step kernels).  A test before every piece, or in the
    // prologue, costs large batches more than it saves (2,000 of 28 words with
    // marginals 23.2 -> 23.8, inside 14.9 -> 15.5).
    auto none_left = [&](int u) { return !GLOB && u == 1 && rw.total <= NT; };
    auto load_pieces = [&](int t0, bool skip) {
#pragma unroll
        for (int u = 0; u < kTilePieces; ++u) {
            if (skip && none_left(u)) break;
            const typename Row_walk::At a = rw.at(t0 + u * NT);
            piece[u] = load_row(scores + (size_t)tab<int>(cx, kTabId, a.sb) * sent_stride, N1, 4 * a.I + a.r, a.J,
                                tab<int>(cx, kTabN, a.sb));
        }
    };
    for (int c0 = tid; c0 < rw.total; c0 += NT * kTilePieces) {   // (one round in LDS)
    load_pieces(c0, false);
#pragma unroll
    for (int u = 0; u < kTilePieces; ++u) {
        const typename Row_walk::At a = rw.at(c0 + u * NT);
        const int n = tab<int>(cx, kTabN, a.sb), i = 4 * a.I + a.r, j0 = 4 * a.J, g = a.I * S + a.sb;
        f4 x;
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = j0 + c > i && j0 + c <= n ? piece[u][c] : NEG;
        const int rr = ((a.r + cx.rot(g)) & 3) * cx.rs(a.J - a.I);
        if (a.ok) {
            st4(sm, cx.a(a.I, a.J, a.sb) + rr, x);
            if constexpr (REV) st4(sm, cx.o(a.I, a.J, a.sb) + rr, x);
        }
    }
    }
    __syncthreads();
    tile_seed(cx, sm);
    // What the q-th rescale moved a sentence's shift by (in place of the forced
    // sums' partials; a rescale needs 5 blocks, and there are 4 at most).
    auto rescale_of = [&](int q, int sb) -> float & {
        return *reinterpret_cast<float *>(cx.tb + cx.partd + 8 * (q * S + sb));
    };
    int rescales = 0;

    // The stages.
    const int nw = NT >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int most = lanes_lg(m * S, nw);
    inside_diagonal<LIN>(cx, sm, flags);
    __syncthreads();
    int tr = tile_rescale_after<LIN>(1, m);
    for (int t = 1; t < (REV ? m + 1 : m); ++t) {
        const int cin = (m - t) * S, cout = REV ? t * S : 0;
        const int lg = stage_lg(t - 1, cin, cout, nw, most);
        const int win = ((cin << lg) + 63) >> 6, wout = ((cout << lg) + 63) >> 6;
        const uint32_t mark = LIN && m < kWideBlocks && t <= tr ? kLinWideBits : kLinLowBits;
        for (int w = wave; w < win + wout; w += nw) {
            if (w < win)
                tile_task<LIN, false>(cx, sm, t, t - 1, cin, w, lg, mark, flags);
            else if (REV && t < m)
                tile_task<LIN, true>(cx, sm, m - t, t - 1, cout, w - win, lg, mark, flags);
            else if (REV)
                outside_diagonal<LIN>(cx, sm, w - win, lg, flags);
        }
        __syncthreads();
        if (t == tr) {
            // (the flag is uniform: no later stage writes it)
            if (!LIN || m >= kWideBlocks || flags[kFlagWide] != 0) {
                tile_rescale<LIN, REV>(cx, sm, t);
                if constexpr (LIN && REV)
                    for (int sb = tid; sb < S; sb += NT) rescale_of(rescales, sb) = tab<float>(cx, kTabDl, sb);
            }
            ++rescales;
            tr = tile_rescale_after<LIN>(t + 1, m);
        }
    }

    // The scores again, for the epilogue: in flight during the roots' sums.
    const int tid_e = here_lane(tid);   // (the walk again too, not kept across the sweep)
    if constexpr (REV && !GLOB) load_pieces(tid_e, true);

    // The roots.
    auto root_of = [&](int sb) {
        const int rc = tab<int>(cx, kTabN, sb) - 4 * (m - 1);
        return *reinterpret_cast<const float *>(sm + cx.a(0, m - 1, sb) + cx.rot(sb) * cx.rs(m - 1) + 4 * rc);
    };
    for (int sb = tid; sb < S; sb += NT) {
        const float r = root_of(sb);
        const float lz = Dm::log2(r);
        if constexpr (LIN) {
            bool bad = !(r >= kLinMin) || !(r <= kLinMax);
            if (flags[kFlagLow] != 0) {
                const float top = __builtin_fmaxf(kLinTopLog2, fast_log2(tab<float>(cx, kTabTop, sb)));
                if constexpr (!REV) bad = true;
                else if (top + tab<float>(cx, kTabR, sb) > lz + kHarmLog2) flags[kFlagHarm] = 1;
            }
            if (bad) flags[kFlagOut] = 1;
        }
        tab<float>(cx, kTabLz, sb) = LIN ? 1.0f / r : lz;
    }
    __syncthreads();
    int redo = LIN ? flags[kFlagOut] : 0;
    if constexpr (LIN && REV) {
        const int harm = flags[kFlagHarm];
        if (harm != 0 && redo == 0) {   // (uniform: both are written before the barrier)
            __syncthreads();
            const bool moved = m >= kWideBlocks || flags[kFlagWide] != 0;
            for (int c0 = tid_e; c0 < rw.total; c0 += NT) {
                const typename Row_walk::At a = rw.at(c0);
                const int sb = a.sb, n = tab<int>(cx, kTabN, sb), i = 4 * a.I + a.r, j0 = 4 * a.J;
                if (!a.ok || i >= n) continue;
                const f4 s = load_row(scores + (size_t)tab<int>(cx, kTabId, sb) * sent_stride, N1, i, a.J, n);
                const int rr = ((a.r + cx.rot(a.I * S + sb)) & 3) * cx.rs(a.J - a.I);
                const f4 al = ld4(sm, cx.a(a.I, a.J, sb) + rr), ou = ld4(sm, cx.o(a.I, a.J, sb) + rr);
                // The rescales since the tile was finished, per node: its sums
                // have moved by that (w - 2 nodes inside a span's sum, n - w - 1
                // outside), and so have their errors.
                float di = 0.f, dout = 0.f;
                int q = 0;
                for (int t = tile_rescale_after<LIN>(1, m); t > 0; t = tile_rescale_after<LIN>(t + 1, m), ++q) {
                    const float dl = moved ? rescale_of(q, sb) : 0.f;
                    di += a.J - a.I <= t ? dl : 0.f;
                    dout += a.J - a.I >= m - t ? dl : 0.f;
                }
                float x = NEG;   // log2 of the largest partner of a low sum, times how its error grew
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = j0 + c, w = j - i;
                    const float e = __builtin_fmaf(s[c], LOG2E_F, tab<float>(cx, kTabD, sb));
                    const float la = fast_log2(al[c]), lo = fast_log2(ou[c]);
                    const float gi = di * (float)(w - 2), go = dout * (float)(n - w - 1);
                    float y = la - e - gi < -100.f ? lo + gi : NEG;
                    y = lo - e - go < -100.f ? __builtin_fmaxf(y, la + go) : y;
                    x = w > 1 && j <= n && !(i == 0 && j == n) ? __builtin_fmaxf(x, y) : x;
                }
                if (x + fast_log2(tab<float>(cx, kTabLz, sb)) > kSpanHarmLog2) flags[kFlagOut] = 1;
            }
            __syncthreads();
            redo = flags[kFlagOut];
        }
    }
    if constexpr (LIN)
        if (redo != 0) return false;
    auto log_z = [&](int sb) {
        const int n = tab<int>(cx, kTabN, sb);
        const float r = root_of(sb);
        const double lr = LIN ? log2_split(r) : (double)r;
        return (lr - (double)tab<float>(cx, kTabD, sb) * (n >= 2 ? n - 2 : 0)) * LN2_D +
               *reinterpret_cast<const double *>(cx.tb + cx.forced + 8 * sb);
    };
    if (logZ != nullptr)
        for (int sb = tid; sb < S; sb += NT) logZ[tab<int>(cx, kTabId, sb)] = (float)log_z(sb);
    if constexpr (!REV) return true;

    if constexpr (GOLD) {
        // The gold spans' scores summed in float64 (a fixed order) and marked
        // in the transposed outside tiles, which nothing reads any more
        // (diagonal tiles: below their diagonal).  A wavefront per sentence, or
        // 16 lanes where the bundle has more sentences than wavefronts: each
        // has kAhead rows' two round trips to memory in flight (4,000 of up to
        // 60 words, mean 8: loss 65 us with a wavefront each and a row a lane,
        // 51 on the width-step kernels, 45 so).
        const int R = 2 * (N1 - 1) - 1, per = S > nw ? 16 : 64, lane = tid & (per - 1);
        for (int sb = S > nw ? tid >> 4 : wave; sb < S; sb += NT / per) {
            const int id = tab<int>(cx, kTabId, sb), n = tab<int>(cx, kTabN, sb);
            const int32_t *g2 = gold + (size_t)id * R * 2;
            double acc = 0.0;
            const int rows = 2 * n - 1;
            constexpr int kAhead = 4;   // rows a lane has in flight
            for (int r0 = lane; r0 < rows; r0 += kAhead * per) {
                int gi[kAhead], gj[kAhead];
                float v[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int r = min(r0 + u * per, rows - 1);
                    gi[u] = g2[2 * r];
                    gj[u] = r0 + u * per < rows ? g2[2 * r + 1] : -1;
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    if (!(0 <= gi[u] && gi[u] < gj[u] && gj[u] <= n)) gi[u] = -1, gj[u] = 0;
                    v[u] = gi[u] >= 0 ? scores[(size_t)id * sent_stride + (size_t)gi[u] * N1 + gj[u]] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int i = gi[u], j = gj[u], g = (j >> 2) * S + sb;
                    acc += (double)v[u];
                    if (i >= 0)
                        *reinterpret_cast<int *>(sm + cx.ot(i >> 2, j >> 2, sb) +
                                                 ((j + cx.rot(g)) & 3) * cx.rs((j >> 2) - (i >> 2)) + 4 * (i & 3)) = kGoldMark;
                }
            }
            acc = row_sum(acc);
            if (per == 64) {
                acc += __shfl_xor(acc, 16, 64);
                acc += __shfl_xor(acc, 32, 64);
            }
            if (lane == 0) loss[id] = (float)(log_z(sb) - acc);
        }
        __syncthreads();
    }

    // Epilogue: the marginals row piece by row piece,
    //   mu(i,j) = g exp2(alpha~(i,j) + O'(i,j) - (s(i,j) + d) - alpha~(0,n)),
    // and exactly g on forced spans.  Linear domain: as the product
    // alpha (O' / e) / Z of the chart's own values, e = exp2(s + d) halved
    // between the two so that neither leaves float32's range (their product is
    // p Z); their logarithms, of values up to 2^100, would carry 10 to 50 times
    // float32's rounding (20 to 40 words at deviation 2: marginals 3.6e-7 off
    // that way, 1.0e-7 so).
    for (int c0 = tid_e; c0 < rw.total; c0 += NT * kTilePieces) {
    if constexpr (GLOB) load_pieces(c0, false);
#pragma unroll
    for (int u = 0; u < kTilePieces; ++u) {
        if (none_left(u)) break;
        const typename Row_walk::At a = rw.at(c0 + u * NT);
        const int sb = a.sb, n = tab<int>(cx, kTabN, sb), id = tab<int>(cx, kTabId, sb);
        const int i = 4 * a.I + a.r, j0 = 4 * a.J, gi = a.I * S + sb;
        if (!a.ok || i >= n) continue;
        const int rr = ((a.r + cx.rot(gi)) & 3) * cx.rs(a.J - a.I);
        const f4 al = ld4(sm, cx.a(a.I, a.J, sb) + rr), ou = ld4(sm, cx.o(a.I, a.J, sb) + rr);
        const float d = tab<float>(cx, kTabD, sb), g = tab<float>(cx, kTabG, sb);
        const float lz = tab<float>(cx, kTabLz, sb);   // (LIN: 1 / Z)
        f4 mu;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = j0 + c;
            const bool forced = j == i + 1 || (i == 0 && j == n);
            float x = __builtin_fmaf(piece[u][c], LOG2E_F, d);
            if constexpr (LIN) {
                const float h = fast_exp2(__builtin_fminf(-0.5f * x, 64.f));   // (e = 0 below 2^-126: both values are 0)
                x = ((al[c] * h) * (ou[c] * h)) * lz;
            } else {
                x = fast_exp2(((al[c] - lz) + ou[c]) - x);
            }
            mu[c] = forced ? g : g * x;
            if constexpr (GOLD) {
                const int gj = a.J * S + sb;
                const int mk = *reinterpret_cast<const int *>(sm + cx.ot(a.I, a.J, sb) +
                                                              ((c + cx.rot(gj)) & 3) * cx.rs(a.J - a.I) + 4 * a.r);
                if (mk == kGoldMark && j > i) mu[c] -= g;
            }
        }
        float *out = marg + (size_t)id * sent_stride + (size_t)i * N1 + j0;
        if (j0 > i && j0 + 3 <= n) {
            *reinterpret_cast<f4u *>(out) = mu;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (j0 + c > i && j0 + c <= n) out[c] = mu[c];
        }
    }
    }
    return true;
}

template <bool REV, bool GOLD = false, bool GLOB = false>
__device__ __forceinline__ void tile_inside(const KernelPlan &p, const int32_t *rec, char *sm, char *lds,
                                            const float *__restrict__ scores, const float *__restrict__ grad,
                                            float *__restrict__ logZ, float *__restrict__ marg,
                                            const int32_t *__restrict__ gold = nullptr,
                                            float *__restrict__ loss = nullptr) {
    if (tile_inside_impl<true, REV, GOLD, GLOB>(p, rec, sm, lds, scores, grad, logZ, marg, gold, loss)) return;
    __syncthreads();   // every thread has left the linear attempt
    tile_inside_impl<false, REV, GOLD, GLOB>(p, rec, sm, lds, scores, grad, logZ, marg, gold, loss);
}

// ---------------------------------------------------------------------------
// CKY in tiles.  Float64 max-plus, beta(i,j) = (max_k fl(beta(i,k) +
// beta(k,j))) + s(i,j), the same sums and the same lowest-split rule as
// cky_block.  A stage finishes one tile diagonal.  When a stage has few tiles
// four lanes share one, a row each (no combining over lanes, but for the
// splits when 8 or 16 share it), and pass their rows round before the finish.
//
// Storage: the upper tiles by diagonal, each diagonal as eight planes of
// 16-byte pieces (row r, columns 0-1 and 2-3), entry f = I*S + sb, so that
// consecutive lanes read consecutive pieces; then 16 bytes of splits
// (k - 4 I) per tile.
// GLOB: the chart in the workspace, one sentence, splits in 16 bits each.
template <bool GLOB>
struct Ck_ctx {
    static constexpr bool kGlob = GLOB;
    static constexpr int kSplitTile = GLOB ? 32 : 16, kNone = GLOB ? 0xFFFF : 0xFF;
    int m, S, split, tab;
    uint32_t mag;
    __device__ __forceinline__ int cnt(int D) const { return (m - D) * S; }
    // tiles of the diagonals before D
    __device__ __forceinline__ int before(int D) const { return S * (D * m - ((D * (D - 1)) >> 1)); }
    __device__ __forceinline__ int plane0(int D, int f) const { return before(D) * 128 + f * 16; }
    __device__ __forceinline__ int stride(int D) const { return cnt(D) * 16; }
};
template <bool GLOB>
__device__ __forceinline__ Ck_ctx<GLOB> ck_ctx(const int32_t *rec) {
    Ck_ctx<GLOB> c;
    c.m = rec[kTrM];
    c.S = GLOB ? 1 : rec[kTrCount];
    c.mag = (uint32_t)rec[kTrMagic];
    c.split = c.before(c.m) * 128;
    c.tab = GLOB ? 0 : c.before(c.m) * 144;
    return c;
}

typedef double d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ d2 ldd(const char *sm, int off) { return *reinterpret_cast<const d2 *>(sm + (uint32_t)off); }
__device__ __forceinline__ void std2(char *sm, int off, d2 v) { *reinterpret_cast<d2 *>(sm + (uint32_t)off) = v; }

// Running maximum of a span's splits and the first split (from 4 I) at it.
// The choice of the split goes through the sign of a difference (exact in
// its sign) and a bit select: five vector operations, where a compare and a
// conditional move, which pass a mask through the scalar registers, issue at
// half rate each and slow each other down across a CU's wavefronts.
struct Best {
    double v;
    int k;
};
__device__ __forceinline__ int neg_mask(double x) {   // all ones when x < 0
    return (int)(__builtin_bit_cast(uint64_t, x) >> 32) >> 31;
}
__device__ __forceinline__ int bit_select(int mask, int a, int b) {   // mask ? a : b, bit by bit
    int r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ void take(Best &b, double t, int k) {   // t > b.v: t and k
    b.k = bit_select(neg_mask(b.v - t), k, b.k);
    b.v = fmax(b.v, t);
}
__device__ __forceinline__ void take_first(Best &b, double t, int k) {   // t >= b.v
    b.k = bit_select(neg_mask(t - b.v), b.k, k);
    b.v = fmax(b.v, t);
}
// Below any chart value, finite (differences of two stay finite).
constexpr double kNoSplit = -1.0e300;
// Over lanes with different splits of one span: the higher value, the lower
// split among equals.
template <int CTRL, int NONE>
__device__ __forceinline__ void best_level(Best (&b)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double v = dpp_d<CTRL>(b[c].v);
        const int k = dpp_i<CTRL>(b[c].k);
        const double m = fmax(b[c].v, v);
        b[c].k = min(b[c].k | (neg_mask(b[c].v - m) & NONE), k | (neg_mask(v - m) & NONE));
        b[c].v = m;
    }
}
// The same across the rows of 16 lanes (WIDE: the 32-lane halves): the swap of
// a value with itself leaves one row's value in one result, the other's in the
// other.
template <bool WIDE, int NONE>
__device__ __forceinline__ void best_swap(Best (&b)[4]) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    auto swap = [](uint32_t v) -> u2 {
        if constexpr (WIDE) return __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(v, v, false, false));
        else return __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(v, v, false, false));
    };
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint64_t u = __builtin_bit_cast(uint64_t, b[c].v);
        const u2 lo = swap((uint32_t)u), hi = swap((uint32_t)(u >> 32)), k = swap((uint32_t)b[c].k);
        const double v0 = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
        const double v1 = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
        const double m = fmax(v0, v1);
        b[c].k = min((int)k[0] | (neg_mask(v0 - m) & NONE), (int)k[1] | (neg_mask(v1 - m) & NONE));
        b[c].v = m;
    }
}
// Lanes per tile of a CKY stage (2^lg, lg of 0, 2 .. 6): one pass of the
// workgroup's wavefronts, and no more lanes than products.
__device__ __forceinline__ int cky_stage_lg(int np, int cnt, int nw) {
    const int room = 64 * nw / cnt;
    const int fit = room >= 64 ? 6 : room >= 32 ? 5 : room >= 16 ? 4 : room >= 8 ? 3 : room >= 4 ? 2 : 0;
    return min(np >= 12 ? 6 : np >= 6 ? 5 : np >= 3 ? 4 : np >= 2 ? 3 : np >= 1 ? 2 : 0, fit);
}

// One row of a tile's products: row r of tiles (I,K) with the four rows of
// (K,J), splits in increasing order.
__device__ __forceinline__ void cky_row(Best (&b)[4], const d2 (&L)[2], const d2 (&R)[4][2], int k0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int kv = here_lane(k0 + k);
#pragma unroll
        for (int c = 0; c < 4; ++c) take(b[c], L[k >> 1][k & 1] + R[k][c >> 1][c & 1], kv);
    }
}

template <typename CX>
__device__ __forceinline__ void cky_tile_task(const CX &cx, char *sm, int D, int w, int lg) {
    D = here(D);
    w = here(w);
    lg = here(lg);
    const int S = cx.S, cnt = cx.cnt(D), np = D - 1, l = this_thread() & 63;
    int f = w * (64 >> lg) + l, row = 0, q = 0;
    if (lg > 0) {
        row = l & 3;
        q = lg == 2 ? 0 : lg == 3 ? (l >> 3) & 1 : (l >> 2) & ((1 << (lg - 2)) - 1);
        f = w * (64 >> lg) + (lg == 3 ? ((l >> 2) & 1) + 2 * (l >> 4) : l >> lg);
    }
    const bool act = f < cnt && row == 0 && q == 0;
    f = min(f, cnt - 1);
    const int at = cx.plane0(D, f), st = cx.stride(D), u = f * 16, v = (f + D * S) * 16, s0 = cx.stride(0);

    Best best[4][4];
    auto load_l = [&](d2 (&L)[2], int kk, int r) {
        const int la = cx.plane0(kk, f), lst = cx.stride(kk);
#pragma unroll
        for (int h = 0; h < 2; ++h) L[h] = ldd(sm, la + (2 * r + h) * lst);
    };
    auto load_r = [&](d2 (&R)[4][2], int kk) {
        const int ra = cx.plane0(D - kk, f + kk * S), rst = cx.stride(D - kk);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) R[k][h] = ldd(sm, ra + (2 * k + h) * rst);
    };
    if (lg == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) best[r][c] = Best{kNoSplit, 0};
#pragma unroll 1
        for (int kk = 1; kk <= np; ++kk) {
            d2 R[4][2], L[2], N[2];   // (the next row of L in flight)
            load_r(R, kk);
            load_l(N, kk, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                __builtin_amdgcn_sched_barrier(0);
                L[0] = N[0];
                L[1] = N[1];
                if (r < 3) load_l(N, kk, r + 1);
                cky_row(best[r], L, R, 4 * kk);
            }
        }
    } else {
        // one row's products, the next tiles in flight during each
        const Best none{kNoSplit, 0};
        Best b[4] = {none, none, none, none};
        constexpr int kAhead = 2;
        struct Ops {
            d2 L[2], R[4][2];
        } op[kAhead];
        const int g = lg - 2, iters = (np + (1 << g) - 1) >> g;   // 2^g lanes per row
        auto load = [&](Ops &o, int it) {
            const int kk = min(1 + q + (it << g), np);
            load_l(o.L, kk, row);
            load_r(o.R, kk);
        };
#pragma unroll
        for (int j = 0; j < kAhead; ++j)
            if (j < iters) load(op[j], j);
#pragma unroll 1
        for (int i0 = 0; i0 < iters; i0 += kAhead)
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const int it = i0 + j, kk = 1 + q + (it << g);
                if (it >= iters) break;
                if (kk <= np) cky_row(b, op[j].L, op[j].R, 4 * kk);
                if (it + kAhead < iters) load(op[j], it + kAhead);
            }
        if (g >= 1) best_level<kRor8, CX::kNone>(b);
        if (g >= 2) best_level<kRor4, CX::kNone>(b);
        if (g >= 3) best_swap<false, CX::kNone>(b);
        if (g >= 4) best_swap<true, CX::kNone>(b);
        auto rows = [&](auto rr) {   // row rr from the lane of each four that holds it
            constexpr int R = decltype(rr)::value, ctrl = R * 0x55;
#pragma unroll
            for (int c = 0; c < 4; ++c) best[R][c] = Best{dpp_d<ctrl>(b[c].v), dpp_i<ctrl>(b[c].k)};
        };
        rows(std::integral_constant<int, 0>{});
        rows(std::integral_constant<int, 1>{});
        rows(std::integral_constant<int, 2>{});
        rows(std::integral_constant<int, 3>{});
    }

    __builtin_amdgcn_sched_barrier(0);   // (the loads below stay out of the products' registers)
    d2 s[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) s[r][h] = ldd(sm, at + (2 * r + h) * st);
    double U[4][4], V[4][4];   // above the diagonal
    auto diag = [&](double (&T)[4][4], int a) {
        const d2 a1 = ldd(sm, a + s0), b1 = ldd(sm, a + 3 * s0);
        T[0][1] = *reinterpret_cast<const double *>(sm + (uint32_t)(a + 8));
        T[0][2] = a1[0];
        T[0][3] = a1[1];
        T[1][2] = b1[0];
        T[1][3] = b1[1];
        T[2][3] = *reinterpret_cast<const double *>(sm + (uint32_t)(a + 5 * s0 + 8));
    };
    diag(U, u);
    diag(V, v);
    // Splits in block I (the lowest), in the blocks between, in block J.  By
    // antidiagonals of the tile; the two splits whose other part the last
    // antidiagonal finished come last (the lower one first at equal sums).
    double x[4][4];
#pragma unroll
    for (int a = 0; a < 7; ++a) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int r = c + 3 - a;
            if (r < 0 || r > 3) continue;
            Best b = best[r][c];
            if (r < 2) {
                Best lo{U[r][r + 2] + x[r + 2][c], r + 2};
                if (r < 1) take(lo, U[0][3] + x[3][c], 3);
                take(lo, b.v, b.k);
                b = lo;
            }
#pragma unroll
            for (int q2 = 0; q2 + 1 < c; ++q2) take(b, x[r][q2] + V[q2][c], 4 * D + q2);
            if (r < 3) {
                const double t = U[r][r + 1] + x[r + 1][c];
                take_first(b, t, r + 1);
            }
            if (c > 0) take(b, x[r][c - 1] + V[c - 1][c], 4 * D + c - 1);
            const double sv = s[r][c >> 1][c & 1];
            x[r][c] = b.v + sv;
            best[r][c].k = b.k;
            if (r == 3 && c == 0) x[3][0] = D == 1 ? sv : x[3][0];   // a word
        }
    }
    if (act) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) std2(sm, at + (2 * r + h) * st, d2{x[r][2 * h], x[r][2 * h + 1]});
        uint32_t pk[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const Best(&q)[4] = best[r];
            if constexpr (CX::kGlob) {
                pk[2 * r] = (uint32_t)q[0].k | (uint32_t)q[1].k << 16;
                pk[2 * r + 1] = (uint32_t)q[2].k | (uint32_t)q[3].k << 16;
            } else {
                pk[r] = (uint32_t)q[0].k | (uint32_t)q[1].k << 8 | (uint32_t)q[2].k << 16 | (uint32_t)q[3].k << 24;
            }
        }
        uint4 *const out = reinterpret_cast<uint4 *>(sm + cx.split + (cx.before(D) + f) * CX::kSplitTile);
        out[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        if constexpr (CX::kGlob) out[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
    }
}

// The split of span (i, j), two words or more, of sentence sb.
template <typename CX>
__device__ __forceinline__ int tile_split(const CX &cx, const char *sm, int sb, int i, int j) {
    const int I = i >> 2, D = (j >> 2) - I;
    const int t = cx.before(D) + I * cx.S + sb;
    typedef typename std::conditional<CX::kGlob, uint16_t, uint8_t>::type SP;
    const int k = 4 * I + (int)reinterpret_cast<const SP *>(sm + cx.split + t * CX::kSplitTile)[4 * (i & 3) + (j & 3)];
    return max(i + 1, min(k, j - 1));   // (already so, unless a score was not finite)
}

template <bool GLOB = false>
__device__ __forceinline__ void tile_cky(const KernelPlan &p, const int32_t *rec, char *sm, char *lds,
                                         const float *__restrict__ scores, int32_t *__restrict__ spans,
                                         float *__restrict__ best) {
    const int tid = this_thread(), NT = (int)blockDim.x, N1 = p.n1;
    const Ck_ctx<GLOB> cx = ck_ctx<GLOB>(rec);
    const int m = cx.m, S = cx.S;
    int *const ids = reinterpret_cast<int *>(lds + cx.tab), *const ns = ids + S;
    for (int sb = tid; sb < S; sb += NT) {
        ids[sb] = rec[kTrHeader + 2 * sb];
        ns[sb] = rec[kTrHeader + 2 * sb + 1];
    }
    __syncthreads();
    const Row_walk rw(m, S);
    const size_t sent_stride = (size_t)N1 * N1;
    constexpr int kU = 6;
    for (int c0 = tid; c0 < rw.total; c0 += NT * kU) {
        typename Row_walk::At a[kU];
        f4 v[kU];
        int n[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            a[u] = rw.at(c0 + u * NT);
            n[u] = ns[a[u].sb];
            v[u] = load_row(scores + (size_t)ids[a[u].sb] * sent_stride, N1, 4 * a[u].I + a[u].r, a[u].J, n[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (!a[u].ok) continue;
            const int i = 4 * a[u].I + a[u].r, j0 = 4 * a[u].J, D = a[u].J - a[u].I;
            double x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = (double)(j0 + c > i && j0 + c <= n[u] ? v[u][c] : NEG);
            const int st = cx.stride(D), at = cx.plane0(D, a[u].I * S + a[u].sb) + 2 * a[u].r * st;
            std2(sm, at, d2{x[0], x[1]});
            std2(sm, at + st, d2{x[2], x[3]});
        }
    }
    __syncthreads();
    for (int f = tid; f < m * S; f += NT) {   // diagonal 0: spans of two and three words
        const int s0 = cx.stride(0), at = f * 16;
        const d2 a0 = ldd(sm, at), a1 = ldd(sm, at + s0), b1 = ldd(sm, at + 3 * s0), c1 = ldd(sm, at + 5 * s0);
        const double x02 = (a0[1] + b1[0]) + a1[0], x13 = (b1[0] + c1[1]) + b1[1];
        Best b{a0[1] + x13, 1};
        take(b, x02 + c1[1], 2);
        const double x03 = b.v + a1[1];
        uint4 *const out = reinterpret_cast<uint4 *>(sm + cx.split + f * Ck_ctx<GLOB>::kSplitTile);
        if constexpr (GLOB) out[0] = make_uint4(0u, 1u | (uint32_t)b.k << 16, 0u, 2u << 16);
        else out[0] = make_uint4(1u << 16 | (uint32_t)b.k << 24, 2u << 24, 0u, 0u);
        std2(sm, at + s0, d2{x02, x03});
        std2(sm, at + 3 * s0, d2{b1[0], x13});
    }
    __syncthreads();
    const int nw = NT >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int D = 1; D < m; ++D) {
        const int cnt = cx.cnt(D), lg = cky_stage_lg(D - 1, cnt, nw), wn = ((cnt << lg) + 63) >> 6;
        for (int w = wave; w < wn; w += nw) cky_tile_task(cx, sm, D, w, lg);
        __syncthreads();
    }

    const int R = 2 * (N1 - 1) - 1;
    for (int sb = wave; sb < S; sb += nw) {   // rows past each tree are -1
        int2 *const out = reinterpret_cast<int2 *>(spans + (size_t)ids[sb] * R * 2);
        for (int r = 2 * ns[sb] - 1 + (tid & 63); r < R; r += 64) out[r] = make_int2(-1, -1);
    }
    if (best != nullptr)
        for (int sb = tid; sb < S; sb += NT) {
            const int n = ns[sb], D = n >> 2, c = n & 3;
            best[ids[sb]] = (float)*reinterpret_cast<const double *>(sm + cx.plane0(D, sb) + (c >> 1) * cx.stride(D) +
                                                                     8 * (c & 1));
        }
    // The trees, one lane per word (see walk_trees).
    const int per = 4 * m - 1, total = S * per;
    const float inv_per = 1.0f / (float)per;
    for (int t = tid; t < total; t += NT) {
        const int sb = div_small(t, per, inv_per), w = t - sb * per, n = ns[sb];
        if (w >= n) continue;
        int2 *const out = reinterpret_cast<int2 *>(spans + (size_t)ids[sb] * R * 2);
        int i = 0, j = n, row = 0;
        for (int it = 0; i < w && it < n; ++it) {   // (the bounds only guard against a corrupt table)
            const int k = tile_split(cx, sm, sb, i, j);
            if (w < k) {
                ++row;
                j = k;
            } else {
                row += 2 * (k - i);
                i = k;
            }
        }
        for (int it = 0; it < n; ++it) {
            out[row] = make_int2(i, j);
            if (j - i < 2) break;
            j = tile_split(cx, sm, sb, i, j);
            ++row;
        }
    }
}

// ---------------------------------------------------------------------------
// Kernels: a workgroup per bundle, the longest predicted first (the plan's
// order); the dispatcher hands a workgroup to each slot that frees up.
#define CRF_TILE_KERNEL \
    __global__ __launch_bounds__(kTileThreadsMax) __attribute__((amdgpu_waves_per_eu(2, 2))) void

template <bool REV>
CRF_TILE_KERNEL tile_inside_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                   float *__restrict__ logZ, float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    tile_inside<REV>(p, p.tile_io.recs + (size_t)blockIdx.x * p.tile_stride, smem_raw, smem_raw, scores, grad, logZ, marg);
}

CRF_TILE_KERNEL tile_loss_kernel(KernelPlan p, const float *__restrict__ scores, const int32_t *__restrict__ gold,
                                 const float *__restrict__ grad, float *__restrict__ loss, float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    tile_inside<true, true>(p, p.tile_io.recs + (size_t)blockIdx.x * p.tile_stride, smem_raw, smem_raw, scores, grad, nullptr,
                            marg, gold, loss);
}

CRF_TILE_KERNEL tile_cky_kernel(KernelPlan p, const float *__restrict__ scores, int32_t *__restrict__ spans,
                                float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    tile_cky(p, p.tile_ck.recs + (size_t)blockIdx.x * p.tile_stride, smem_raw, smem_raw, scores, spans, best);
}

// Inside with the marginals and CKY in one launch, bundles of both merged.
CRF_TILE_KERNEL tile_parse_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                  float *__restrict__ logZ, float *__restrict__ marg, int32_t *__restrict__ spans,
                                  float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = p.tile_mix.recs + (size_t)blockIdx.x * p.tile_stride;
    if (rec[kTrKind] == kKindInside) tile_inside<true>(p, rec, smem_raw, smem_raw, scores, grad, logZ, marg);
    else tile_cky(p, rec, smem_raw, smem_raw, scores, spans, best);
}

// MBR decoding: a bundle's marginals, then CKY over them (read back by the
// workgroup that wrote them) in the same LDS.
CRF_TILE_KERNEL tile_mbr_kernel(KernelPlan p, const float *__restrict__ scores, float *__restrict__ logZ, float *marg,
                                int32_t *__restrict__ spans, float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = p.tile_io.recs + (size_t)blockIdx.x * p.tile_stride;
    tile_inside<true>(p, rec, smem_raw, smem_raw, scores, nullptr, logZ, marg);
    __syncthreads();   // the marginals are written and the charts are free
    tile_cky(p, rec, smem_raw, smem_raw, marg, spans, best);
}

#define CRF_TILE_WS_KERNEL __global__ __launch_bounds__(kTileThreadsWs) void

// The same on charts in the workspace, for sentences past LDS: a workgroup per
// sentence and pass, record 2 b of the b-th longest sentence its inside pass,
// 2 b + 1 its CKY (their charts are disjoint, so that the fused launch runs
// both side by side).  Bound by the stages' products, whose tiles come from L2
// (a sentence's charts are 0.9 MB at 256 words): 64 sentences of 256 words
// fused 1,709 -> 540 us, a lone one 1,095 -> 493 (the kernels that take a width a
// step, on teams of 16 workgroups).  1,024 threads were slower (635 us), and so
// were three products' loads in flight instead of one or two.
__device__ __forceinline__ const int32_t *ws_record(const KernelPlan &p, int b) {
    return p.tile_ws.recs + (size_t)b * (kTrHeader + 2);
}
__device__ __forceinline__ char *ws_chart(const KernelPlan &p, const int32_t *rec) {
    return p.ws + (size_t)rec[kTrPitch] * 256;
}

template <bool REV>
CRF_TILE_WS_KERNEL tile_ws_inside_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                      float *__restrict__ logZ, float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = ws_record(p, 2 * (int)blockIdx.x);
    tile_inside<REV, false, true>(p, rec, ws_chart(p, rec), smem_raw, scores, grad, logZ, marg);
}

CRF_TILE_WS_KERNEL tile_ws_loss_kernel(KernelPlan p, const float *__restrict__ scores, const int32_t *__restrict__ gold,
                                    const float *__restrict__ grad, float *__restrict__ loss,
                                    float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = ws_record(p, 2 * (int)blockIdx.x);
    tile_inside<true, true, true>(p, rec, ws_chart(p, rec), smem_raw, scores, grad, nullptr, marg, gold, loss);
}

CRF_TILE_WS_KERNEL tile_ws_cky_kernel(KernelPlan p, const float *__restrict__ scores, int32_t *__restrict__ spans,
                                   float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = ws_record(p, 2 * (int)blockIdx.x + 1);
    tile_cky<true>(p, rec, ws_chart(p, rec), smem_raw, scores, spans, best);
}

CRF_TILE_WS_KERNEL tile_ws_parse_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                     float *__restrict__ logZ, float *__restrict__ marg, int32_t *__restrict__ spans,
                                     float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = ws_record(p, (int)blockIdx.x);
    if (rec[kTrKind] == kKindInside) tile_inside<true, false, true>(p, rec, ws_chart(p, rec), smem_raw, scores, grad, logZ, marg);
    else tile_cky<true>(p, rec, ws_chart(p, rec), smem_raw, scores, spans, best);
}

CRF_TILE_WS_KERNEL tile_ws_mbr_kernel(KernelPlan p, const float *__restrict__ scores, float *__restrict__ logZ, float *marg,
                                      int32_t *__restrict__ spans, float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const int32_t *rec = ws_record(p, 2 * (int)blockIdx.x);
    tile_inside<true, false, true>(p, rec, ws_chart(p, rec), smem_raw, scores, nullptr, logZ, marg);
    __syncthreads();   // the marginals are written (each row piece by the thread that reads it back)
    rec += kTrHeader + 2;
    tile_cky<true>(p, rec, ws_chart(p, rec), smem_raw, marg, spans, best);
}

// Batches with sentences on both sides of LDS, in one launch: the workspace
// sentences' passes first (they are the longest), then the bundles, all of 512
// threads, so that a bundle does not wait for the last long sentence.  As two
// launches the times added up, and a batch clipped at 140 words (a block past
// LDS, where a width a step still fits) lost to the width-step kernels.  1,000
// sentences of up to 140 words, us (a width a step, two launches, one):
// inside 96.5, 141, 78; with marginals 175.5, 218, 123; fused 177, 295, 163;
// MBR 304, 510, 286; loss 189, 249, 151.  64 of 256 words and 4,000 of up to 99,
// fused: 1,811, 609, 522.
// A workgroup's record, and whether its charts are in the workspace.  per:
// passes of a workspace sentence in the launch.  (The charts' address is taken
// on each side of the branch: a pointer that may be either would be a generic
// one: 16 of 20 to 200 words fused 316 us that way, 286 so.)
struct Both_work {
    const int32_t *rec;
    bool glob;
};
__device__ __forceinline__ Both_work both_work(const KernelPlan &p, const TileSchedule &lds, int per, int pass) {
    const int b = (int)blockIdx.x, n_ws = per * p.tile_ws.n;
    if (b >= n_ws) return Both_work{lds.recs + (size_t)(b - n_ws) * p.tile_stride, false};
    return Both_work{ws_record(p, per == 2 ? b : 2 * b + pass), true};
}

template <bool REV>
CRF_TILE_KERNEL tile_both_inside_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                        float *__restrict__ logZ, float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    const Both_work k = both_work(p, p.tile_io, 1, 0);
    if (k.glob) tile_inside<REV, false, true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, grad, logZ, marg);
    else tile_inside<REV>(p, k.rec, smem_raw, smem_raw, scores, grad, logZ, marg);
}

CRF_TILE_KERNEL tile_both_loss_kernel(KernelPlan p, const float *__restrict__ scores, const int32_t *__restrict__ gold,
                                      const float *__restrict__ grad, float *__restrict__ loss,
                                      float *__restrict__ marg) {
    extern __shared__ __align__(16) char smem_raw[];
    const Both_work k = both_work(p, p.tile_io, 1, 0);
    if (k.glob) tile_inside<true, true, true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, grad, nullptr, marg, gold, loss);
    else tile_inside<true, true>(p, k.rec, smem_raw, smem_raw, scores, grad, nullptr, marg, gold, loss);
}

CRF_TILE_KERNEL tile_both_cky_kernel(KernelPlan p, const float *__restrict__ scores, int32_t *__restrict__ spans,
                                     float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const Both_work k = both_work(p, p.tile_ck, 1, 1);
    if (k.glob) tile_cky<true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, spans, best);
    else tile_cky(p, k.rec, smem_raw, smem_raw, scores, spans, best);
}

CRF_TILE_KERNEL tile_both_parse_kernel(KernelPlan p, const float *__restrict__ scores, const float *__restrict__ grad,
                                       float *__restrict__ logZ, float *__restrict__ marg, int32_t *__restrict__ spans,
                                       float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const Both_work k = both_work(p, p.tile_mix, 2, 0);
    const bool inside = k.rec[kTrKind] == kKindInside;
    if (k.glob) {
        if (inside) tile_inside<true, false, true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, grad, logZ, marg);
        else tile_cky<true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, spans, best);
    } else {
        if (inside) tile_inside<true>(p, k.rec, smem_raw, smem_raw, scores, grad, logZ, marg);
        else tile_cky(p, k.rec, smem_raw, smem_raw, scores, spans, best);
    }
}

// (a workspace sentence too: its inside record is followed by its CKY record)
CRF_TILE_KERNEL tile_both_mbr_kernel(KernelPlan p, const float *__restrict__ scores, float *__restrict__ logZ, float *marg,
                                     int32_t *__restrict__ spans, float *__restrict__ best) {
    extern __shared__ __align__(16) char smem_raw[];
    const Both_work k = both_work(p, p.tile_io, 1, 0);
    if (k.glob) {
        tile_inside<true, false, true>(p, k.rec, ws_chart(p, k.rec), smem_raw, scores, nullptr, logZ, marg);
        __syncthreads();
        const int32_t *rec = k.rec + kTrHeader + 2;
        tile_cky<true>(p, rec, ws_chart(p, rec), smem_raw, marg, spans, best);
    } else {
        tile_inside<true>(p, k.rec, smem_raw, smem_raw, scores, nullptr, logZ, marg);
        __syncthreads();
        tile_cky(p, k.rec, smem_raw, smem_raw, marg, spans, best);
    }
}

}  // namespace

hipError_t set_tile_attributes(int max_lds_bytes) {
    const void *fns[] = {(const void *)tile_inside_kernel<false>, (const void *)tile_inside_kernel<true>,
                         (const void *)tile_loss_kernel, (const void *)tile_cky_kernel, (const void *)tile_parse_kernel,
                         (const void *)tile_mbr_kernel, (const void *)tile_both_inside_kernel<false>,
                         (const void *)tile_both_inside_kernel<true>, (const void *)tile_both_loss_kernel,
                         (const void *)tile_both_cky_kernel, (const void *)tile_both_parse_kernel,
                         (const void *)tile_both_mbr_kernel};
    for (const void *f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// A plan's workspace sentences (ws), bundles (lds), or both in one launch:
// `per` passes a workspace sentence.
template <typename... KA, typename... A>
static hipError_t launch_tile(const KernelPlan &p, const TileSchedule &lds, int per, hipStream_t stream,
                              void (*k_ws)(KernelPlan, KA...), void (*k_lds)(KernelPlan, KA...),
                              void (*k_both)(KernelPlan, KA...), A... args) {
    const int n_ws = per * p.tile_ws.n;
    const size_t ws_bytes = (size_t)p.tile_ws.lds_bytes, lds_bytes = (size_t)lds.lds_bytes;
    if (n_ws > 0 && lds.n > 0)
        hipLaunchKernelGGL(k_both, dim3(n_ws + lds.n), dim3(kTileThreadsMax), ws_bytes > lds_bytes ? ws_bytes : lds_bytes,
                           stream, p, args...);
    else if (n_ws > 0)
        hipLaunchKernelGGL(k_ws, dim3(n_ws), dim3(kTileThreadsWs), ws_bytes, stream, p, args...);
    else if (lds.n > 0)
        hipLaunchKernelGGL(k_lds, dim3(lds.n), dim3(p.tile_threads), lds_bytes, stream, p, args...);
    else
        return hipSuccess;
    return hipGetLastError();
}

hipError_t launch_tile_inside(const KernelPlan &p, const float *scores, const float *grad, float *logZ, float *marg,
                              hipStream_t stream) {
    if (marg != nullptr)
        return launch_tile(p, p.tile_io, 1, stream, tile_ws_inside_kernel<true>, tile_inside_kernel<true>,
                           tile_both_inside_kernel<true>, scores, grad, logZ, marg);
    return launch_tile(p, p.tile_io, 1, stream, tile_ws_inside_kernel<false>, tile_inside_kernel<false>,
                       tile_both_inside_kernel<false>, scores, grad, logZ, marg);
}
hipError_t launch_tile_loss(const KernelPlan &p, const float *scores, const int32_t *gold, const float *grad,
                            float *loss, float *grad_scores, hipStream_t stream) {
    return launch_tile(p, p.tile_io, 1, stream, tile_ws_loss_kernel, tile_loss_kernel, tile_both_loss_kernel, scores, gold,
                       grad, loss, grad_scores);
}
hipError_t launch_tile_cky(const KernelPlan &p, const float *scores, int32_t *spans, float *best, hipStream_t stream) {
    return launch_tile(p, p.tile_ck, 1, stream, tile_ws_cky_kernel, tile_cky_kernel, tile_both_cky_kernel, scores, spans, best);
}
hipError_t launch_tile_parse(const KernelPlan &p, const float *scores, const float *grad, float *logZ, float *marg,
                             int32_t *spans, float *best, hipStream_t stream) {
    return launch_tile(p, p.tile_mix, 2, stream, tile_ws_parse_kernel, tile_parse_kernel, tile_both_parse_kernel, scores,
                       grad, logZ, marg, spans, best);
}
hipError_t launch_tile_mbr(const KernelPlan &p, const float *scores, float *logZ, float *marg, int32_t *spans,
                           float *best, hipStream_t stream) {
    return launch_tile(p, p.tile_io, 1, stream, tile_ws_mbr_kernel, tile_mbr_kernel, tile_both_mbr_kernel, scores, logZ,
                       marg, spans, best);
}

}  // namespace crf
