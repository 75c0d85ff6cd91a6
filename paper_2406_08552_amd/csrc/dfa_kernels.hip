// Attention kernels of the DiTFastAttn hot path for gfx950 (CDNA4).
//
// One kernel template covers the three attention operations of the method:
//   MODE_FULL     O = softmax(Q K^T / sqrt(d)) V                 (Sec. 3.2, Eq. 1 first line)
//   MODE_REFRESH  O = full attention, R = O - window attention    (Sec. 3.2, Eq. 1), R in fp32
//   MODE_WINDOW   O = window attention (+ R when given)           (Sec. 3.2, Eq. 2)
//   MODE_WINDOW_FINE  the same for bands of at most 31 keys, with split probabilities
// The window is the band |i - j| <= w over the flattened token index.
//
// Work decomposition
//   A workgroup is 4 wavefronts and owns 128 consecutive queries of one
//   (batch, head); each wavefront owns 32 of them (two 16-query MFMA blocks,
//   QB = 2).  Launches whose tile walk is short (small L or a narrow band)
//   use QB = 1 instead: 64-query workgroups, four wavefronts per SIMD.
//   The workgroup walks key tiles of BK = 64 keys, staged in LDS with double
//   buffering (global loads of the next tile are in flight while the current
//   one is used).  A whole tile is copied from a uniform tile base plus
//   per-lane offsets that do not depend on the tile, so the copies take the
//   scalar-base addressing form and cost the softmax no VALU work; only the
//   ragged last tile clamps its rows.  Three workgroups share a CU (three wavefronts per SIMD), so
//   the MFMA work of one overlaps the softmax arithmetic of the others.
//
// MFMA mapping (v_mfma_f32_16x16x32_bf16, fp32 accumulation)
//   Scores are formed transposed, S^T = K Q^T: A = 16 keys x 32 dims from LDS,
//   B = 32 dims x 16 queries held in registers for the whole kernel.  The
//   result leaves every lane with a single query (lane % 16) and four keys
//   per 16-key block, so softmax statistics are per-lane values reduced over
//   the four 16-lane rows only (two permlane swaps).  The same registers,
//   rounded to bf16, are directly the B operand of the second product
//   O^T = V^T P^T, whose A operand is read from a transposed copy of the V
//   tile in LDS.  The output accumulator keeps the one-query-per-lane
//   layout, so the online-softmax rescale needs no data movement.
//   Head dim 72 = 2 x 32 + 8: the last 8 dims go through one more 16x16x32
//   MFMA with k zero-padded (on gfx950 the k=16 form costs about as much);
//   PV pads the 72 output dims to 5 blocks of 16.  The
//   padding row 72 of V^T is set to 1.0, so the PV product also yields the
//   softmax row sum (the sum of the same bf16 probabilities that weight V).
//   Head dim 64 has no padding row: the lanes sum the rounded probabilities
//   themselves, so both head dims normalise exactly the weights they apply.
//
// Online softmax
//   Per query a running max m (log2 domain) and accumulator (O, l).  The max
//   is updated lazily: the accumulator is rescaled only when a tile's max
//   exceeds m by more than 8 (so probabilities stay below 2^8 and the
//   rescale is almost never taken after the first tiles).  Once every query
//   of a wavefront has a running max, a tile's probabilities are formed
//   without its maxima, scaled by 2^-7 so that the margin is the top bit of
//   their bf16 exponents, and one OR over the packed words tests it; a tile
//   that reaches the margin is scored again and takes the exact form, which
//   forms the maxima across lanes and rescales.
//
// Narrow bands
//   A bf16 probability is off by up to 2^-8 of itself.  Over many keys these
//   errors average out; over a band of a few keys they do not, and the output
//   moves by up to 2^-8 max|v - o| on top of its own bf16 rounding.  Bands of
//   at most 31 keys per query therefore apply each probability twice: as its
//   bf16 value and as the bf16 rounding of its residual p - bf16(p), in two PV
//   products, so each weight is applied to about 2^-16 relative.  The refresh
//   does the same in its in-band phase, which forms W.
//
// Tile walk and band handling
//   The key tiles a workgroup visits are split into segments so that the hot
//   loop carries no mask: tiles where every score counts (PLAIN), the ragged
//   last tile (KEYS: j < L), and the tiles at the band edges, where each
//   wavefront classifies the tile against its own queries (inside the band,
//   outside, or straddling it with an element mask).
//   The window kernel visits only the tiles that intersect the workgroup's
//   band.  In long sequences the refresh kernel runs ONE accumulator over two
//   phases: first the in-band scores of the band tiles (after which the
//   accumulator, normalised, is the window attention W; it is parked in the R
//   buffer), then every out-of-band score, which turns the same accumulator
//   into full attention.  R = O - W is formed in the epilogue.  Every score is
//   used exactly once, only the few band-edge tiles are visited twice, and no
//   second accumulator occupies registers.  In shorter ones, where band-edge
//   tiles are a large part of the walk (one_pass_refresh), and in launches of
//   few workgroups, which take key groups, the refresh instead keeps two
//   accumulators and visits every tile once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfa_internal.h"

namespace dfa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NWAVES = 4;
constexpr int NTHREADS = NWAVES * 64;
constexpr int BK = 64;                    // keys per tile
constexpr int NKB = BK / 16;              // 16-key blocks per tile
// A wavefront owns QB 16-query blocks (QB = 1 or 2), a workgroup bq<QB>() queries.
template <int QB>
constexpr int bq() { return NWAVES * QB * 16; }
constexpr float RESCALE_THRESH = 8.0f;    // lazy rescale margin (log2 units)
// Probabilities are formed as 2^(x - m - P_SHIFT): a probability at the rescale
// margin is then exactly 2, the smallest value whose bf16 form has the top
// exponent bit set, so one OR over the packed probabilities tests the margin.
// The power-of-two factor cancels in O / l.  The shifted exponent argument is
// rounded at a larger magnitude, which moves any probability of at least 2^-8
// of the running max by at most about 2^-21 of itself, far below its bf16
// rounding.
constexpr float P_SHIFT = RESCALE_THRESH - 1.0f;
constexpr uint32_t P_MARGIN_BITS = 0x40004000u;   // top exponent bit of both packed bf16 values
constexpr int FINE_MAX_HALF_WIDTH = 15;   // window half-widths applied with split probabilities
constexpr float NEG_INF = -__builtin_inff();

enum {
    MODE_FULL = 0, MODE_REFRESH = 1, MODE_WINDOW = 2, MODE_ASC = 3, MODE_REFRESH_SPLIT = 4, MODE_WINDOW_FINE = 5,
    MODE_REFRESH_FINE = 6
};
// MODE_ASC computes exactly what MODE_FULL computes (on the conditional half of
// the batch, storing every tile to both halves); it is a separate
// instantiation only so that profiles report it apart from full attention.
// MODE_REFRESH_SPLIT computes what MODE_REFRESH computes, in one pass with two
// accumulators instead of two phases with one (short sequences).
// MODE_REFRESH_FINE is the two-phase refresh for bands of at most 31 keys: its
// in-band phase (the window attention W) applies split probabilities, like
// MODE_WINDOW_FINE; the out-of-band phase, over all other keys, plain ones.
enum { MASK_NONE = 0, MASK_KEYS = 1, MASK_BAND_IN = 2, MASK_BAND_OUT = 3 };
enum { TILE_INSIDE = 0, TILE_OUTSIDE = 1, TILE_BOUNDARY = 2 };
// segment kinds of the tile walk
enum { SEG_PLAIN = 0, SEG_KEYS = 1, SEG_BAND_IN = 2, SEG_BAND_OUT = 3 };

// Geometry derived from the head dim.
//   LDS tiles are row-major, one key per row, filled by 16-byte direct
//   global->LDS copies (lane l of a copy lands at base + 16 l, so chunk c of a
//   tile sits at 16 c bytes).  K rows take KPC chunks (pitch 144 B for d = 64
//   and 72: 16-byte reads by 16 consecutive rows hit distinct 4-bank groups).
//   V rows take VPC chunks; for d = 72 the tenth chunk holds (1, 0, ..., 0),
//   a constant "dim 72 = 1" column that makes the PV product emit the row
//   sum.  Chunks at or beyond NCH are never copied into.
template <int D>
struct Geo {
    static_assert(D % 8 == 0 && D <= 72, "head dim must be a multiple of 8, at most 72");
    static_assert(D % 32 == 0 || D % 32 == 8 || D % 32 == 16, "unsupported head dim remainder");
    static constexpr int NC32 = D / 32;              // k=32 chunks of the score product
    static constexpr int D32 = NC32 * 32;
    static constexpr int TAIL = D - D32;             // dims left for one zero-padded k=32 chunk (0, 8, 16)
    static constexpr int NDB = (D + 15) / 16;        // 16-dim output blocks of PV
    static constexpr bool ONES = (D % 16) != 0;      // the padding column D of V carries ones
    static constexpr int NCH = D / 8;                // 16-byte chunks of data per row
    static constexpr int KPC = 9;                    // K row pitch in chunks (144 B)
    static constexpr int VPC = ONES ? NCH + 1 : 9;   // V row pitch in chunks (160 B for d = 72)
    static constexpr int KP = KPC * 8;               // pitches in elements
    static constexpr int VP = VPC * 8;
    static constexpr int KS_ELEMS = BK * KP;
    static constexpr int VS_ELEMS = BK * VP;
    static constexpr int STAGE_ELEMS = KS_ELEMS + VS_ELEMS;
    static constexpr int KROUNDS = (BK * KPC + NTHREADS - 1) / NTHREADS;
    static constexpr int VROUNDS = (BK * VPC + NTHREADS - 1) / NTHREADS;
    static_assert(NDB * 16 <= VP, "PV reads the padded dims of each V row");
    static_assert((KP / 2) % 32 == 4, "K pitch");
};

struct Params {
    const uint16_t* Q;
    const uint16_t* K;
    const uint16_t* V;
    const float* Rin;         // MODE_WINDOW: fp32 residual added to the output (or null)
    float* Rout;              // MODE_REFRESH: fp32 residual output (also parks W)
    uint16_t* dst[4];         // every destination receives the same output tile
    int ndst;
    int H, L, w;
    int n_qt;                 // query tiles per (batch, head)
    int nblocks;
    float c;                  // log2(e) / sqrt(d)
    int nout;                 // the first nout of dst[] are O, the others the output cache
};

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Two floats -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}

// acc + the two bf16 values packed in w (one dot2 with (1, 1)): the row sum
// is taken over the same rounded probabilities that weight V, so each output
// row is a convex combination of V rows (exact for a one-hot row).
__device__ __forceinline__ float pair_acc(uint32_t w, float acc) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, acc, false);
}

// The rounding residuals lo - bf16(lo) and hi - bf16(hi) of a pair packed by
// pack_bf16x2 (exact in fp32), themselves packed to bf16.
__device__ __forceinline__ uint32_t pack_residual(float lo, float hi, uint32_t packed) {
    return pack_bf16x2(lo - __builtin_bit_cast(float, packed << 16), hi - __builtin_bit_cast(float, packed & 0xFFFF0000u));
}

// s_waitcnt vmcnt(0): every global access of this wavefront has completed.
// The tile stores sit in branches that whole wavefronts skip; without this
// the compiler cannot prove at the loop head that the Q fragments have
// arrived and waits for the just-issued prefetch before the first MFMA.
__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Reductions over the four 16-lane rows that hold the same query.
// v_permlane16_swap exchanges rows 1 and 3 of its first operand with rows 0
// and 2 of its second; v_permlane32_swap exchanges the upper half of the
// first with the lower half of the second.  Applied to two copies of x they
// leave each lane with its own and its partner row's value (rows r^1, then
// halves r^2).  Issued as inline assembly: the compiler's folding of the
// builtin's paired result has been seen to drop the second value.  The
// leading s_nop covers the VALU-write -> permlane-read hazard.
__device__ __forceinline__ void xchg16(uint32_t& a, uint32_t& b) {
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void xchg32(uint32_t& a, uint32_t& b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

__device__ __forceinline__ float group_max(float x) {
    uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
    xchg16(a, b);
    a = __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)));
    b = a;
    xchg32(a, b);
    return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}

__device__ __forceinline__ float group_sum(float x) {
    uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
    xchg16(a, b);
    a = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b));
    b = a;
    xchg32(a, b);
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// One score tile, passed by value where a masked private copy is needed.
template <int QB>
struct Tile {
    f32x4 s[QB][NKB];
};

template <int D, int QB>
struct Acc {
    f32x4 o[QB][Geo<D>::NDB];   // O^T: lane holds dims 16*m + 4*g + i of query lane%16
    // The running max m (log2 domain) is kept in two derived forms:
    float negm[QB];             // -m - P_SHIFT, or -P_SHIFT while the query has seen no finite score
    float thr[QB];              // (m + RESCALE_THRESH) / c in raw score units (-inf: no m yet)
    float l[QB];                // lane-partial sum of the bf16 probabilities (unused when a ones row is present)
    bool fresh;                 // some query of the wavefront has no running max yet (wave-uniform)

    __device__ __forceinline__ void init() {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int mb = 0; mb < Geo<D>::NDB; ++mb) o[qb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            negm[qb] = -P_SHIFT;
            thr[qb] = NEG_INF;
            l[qb] = 0.f;
        }
        fresh = true;
    }
    // m of query block qb (-inf before its first finite score)
    __device__ __forceinline__ float running_max(int qb) const { return thr[qb] == NEG_INF ? NEG_INF : -(negm[qb] + P_SHIFT); }
};

template <int D, int QB>
struct QFrag {
    bf16x8 a[QB][Geo<D>::NC32 > 0 ? Geo<D>::NC32 : 1];
    bf16x8 t[QB];   // dims D32.. in lane rows g < TAIL/8, zero elsewhere
};

// Q fragments (B operand of S^T = K Q^T), zero beyond L and beyond d
template <int D, int QB>
__device__ __forceinline__ void load_q(QFrag<D, QB>& q, const uint16_t* __restrict__ Qbh, int qw0, int L, int r, int g) {
    using G = Geo<D>;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qrow = qw0 + 16 * qb + r;
        const bool ok = qrow < L;
        const uint16_t* qp = Qbh + (size_t)(ok ? qrow : 0) * D;
#pragma unroll
        for (int c = 0; c < G::NC32; ++c)
            q.a[qb][c] = as_bf16x8(ok ? *(const u32x4*)(qp + 32 * c + 8 * g) : u32x4{0u, 0u, 0u, 0u});
        q.t[qb] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
        if constexpr (G::TAIL > 0) {
            if (ok && 8 * g < G::TAIL) q.t[qb] = as_bf16x8(*(const u32x4*)(qp + G::D32 + 8 * g));
        }
    }
}

// Score tile S^T for the wavefront's 16 * QB queries against the 64 keys of one LDS
// stage: S[qb][kb][i] is the score of query (16*qb + lane%16) and key
// (16*kb + 4*(lane/16) + i) of the tile.
template <int D, int QB>
__device__ __forceinline__ void score_tile(const uint16_t* __restrict__ Ks, const QFrag<D, QB>& q, Tile<QB>& S, int r, int g) {
    using G = Geo<D>;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        const uint16_t* krow = Ks + (16 * kb + r) * G::KP;
        bf16x8 ka[G::NC32 > 0 ? G::NC32 : 1];
#pragma unroll
        for (int c = 0; c < G::NC32; ++c) ka[c] = as_bf16x8(*(const u32x4*)(krow + 32 * c + 8 * g));
        // tail dims: lane rows g >= TAIL/8 re-read the row's first tail chunk;
        // their Q tail fragment is zero, so those products vanish (the values
        // read belong to the same key row, so no other row's data enters)
        u32x4 kt = u32x4{0u, 0u, 0u, 0u};
        if constexpr (G::TAIL > 0) kt = *(const u32x4*)(krow + G::D32 + (8 * g < G::TAIL ? 8 * g : 0));
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < G::NC32; ++c) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[c], q.a[qb][c], s, 0, 0, 0);
            if constexpr (G::TAIL > 0) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kt), q.t[qb], s, 0, 0, 0);
            S.s[qb][kb] = s;
        }
    }
}

// Offsets [lo, lo + span] of a lane's in-band keys from its first, for query
// qi: the band |qi - j| <= w cut to [0, L - 1]; a query beyond L whose band
// holds no key gets an offset that no key has.
__device__ __forceinline__ void band_range(int qi, int jbase, int L, int w, int& lo, uint32_t& span) {
    const int a = (qi > w ? qi - w : 0) - jbase;
    const uint32_t qpw = (uint32_t)qi + (uint32_t)w;    // < 2^32: qi < 2^31, w < 2^31
    const int b = (int)(qpw < (uint32_t)(L - 1) ? qpw : (uint32_t)(L - 1)) - jbase;
    lo = b < a ? (1 << 30) : a;
    span = b < a ? 0u : (uint32_t)(b - a);
}

// Masks a score tile for one of the band or key masks (MASK_NONE: no-op).
template <int MASK, int QB>
__device__ __forceinline__ void mask_tile(Tile<QB>& S, int r, int g, int qrow0, int k0, int L, int w) {
    if constexpr (MASK != MASK_NONE) {
        // The lane's scores are the keys jbase + o, o = 16 kb + i.  Valid keys
        // (j < L) are the offsets o <= lim.  For the in-band mask the band
        // |qi - j| <= w, cut to [0, L - 1], is the offset range [a, b], tested
        // as one unsigned compare (o - a <= b - a); a query row beyond L whose
        // band holds no key gets an empty range.  The out-of-band mask keeps
        // the direct distance test: the range form's two extra live values per
        // query block cost the refresh kernel spills and time.
        const int jbase = k0 + 4 * g;
        const int lim = L - 1 - jbase;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            int lo = 0;
            uint32_t span = 0u;
            if constexpr (MASK == MASK_BAND_IN) {
                band_range(qrow0 + 16 * qb + r, jbase, L, w, lo, span);
            }
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int o = 16 * kb + i;
                    bool ok;
                    if constexpr (MASK == MASK_KEYS) ok = o <= lim;
                    else if constexpr (MASK == MASK_BAND_IN) ok = (uint32_t)(o - lo) <= span;
                    else {
                        const int j = jbase + o, qi = qrow0 + 16 * qb + r;
                        ok = j < L && (qi > j ? qi - j : j - qi) > w;
                    }
                    S.s[qb][kb][i] = ok ? S.s[qb][kb][i] : NEG_INF;
                }
            }
        }
    }
}

// Splits a score tile by the band: S keeps the in-band scores, X gets the
// others (of keys < L if S was masked so); -inf elsewhere.
template <int QB>
__device__ __forceinline__ void split_tile(Tile<QB>& S, Tile<QB>& X, int r, int g, int qrow0, int k0, int L, int w) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        int lo;
        uint32_t span;
        band_range(qrow0 + 16 * qb + r, k0 + 4 * g, L, w, lo, span);
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = (uint32_t)(16 * kb + i - lo) <= span;
                const float s = S.s[qb][kb][i];
                S.s[qb][kb][i] = in ? s : NEG_INF;
                X.s[qb][kb][i] = in ? NEG_INF : s;
            }
    }
}

// Probabilities of one score tile against the running maxima, packed to bf16
// as the B operand of PV.  FINE adds a second operand, the rounding residual
// p - bf16(p) rounded to bf16, so that the two PV products apply each weight
// to about 2^-16 relative: rows with few keys do not average the bf16
// rounding of their weights.  psum: the lane-partial sums of what is applied
// (head dims without a ones row).
template <int D, int QB, bool FINE>
struct Probs {
    bf16x8 pb[QB][BK / 32];
    bf16x8 pl[FINE ? QB : 1][BK / 32];
    float psum[QB];
};

template <int D, int QB, bool FINE>
__device__ __forceinline__ void form_probs(const Acc<D, QB>& acc, const Tile<QB>& S, float c, Probs<D, QB, FINE>& P) {
    using G = Geo<D>;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float negm = acc.negm[qb];
        float psum = 0.f;
#pragma unroll
        for (int h = 0; h < BK / 32; ++h) {
            uint32_t wds[4], rws[4];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const f32x4 s = S.s[qb][2 * h + half];
                const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0], c, negm));
                const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[1], c, negm));
                const float p2 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2], c, negm));
                const float p3 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[3], c, negm));
                wds[2 * half + 0] = pack_bf16x2(p0, p1);
                wds[2 * half + 1] = pack_bf16x2(p2, p3);
                if constexpr (FINE) {
                    rws[2 * half + 0] = pack_residual(p0, p1, wds[2 * half + 0]);
                    rws[2 * half + 1] = pack_residual(p2, p3, wds[2 * half + 1]);
                }
                if constexpr (!G::ONES) {
                    psum = pair_acc(wds[2 * half + 1], pair_acc(wds[2 * half], psum));
                    if constexpr (FINE) psum = pair_acc(rws[2 * half + 1], pair_acc(rws[2 * half], psum));
                }
            }
            P.pb[qb][h] = as_bf16x8(u32x4{wds[0], wds[1], wds[2], wds[3]});
            if constexpr (FINE) P.pl[qb][h] = as_bf16x8(u32x4{rws[0], rws[1], rws[2], rws[3]});
        }
        P.psum[qb] = psum;
    }
}

// A operand of O^T += V^T P^T, dims 16 mb.. x keys 32 h.., from the row-major V
// tile through transposing reads: within each 16-lane row, lane 4m+q addresses
// dims 16mb+4q..+3 of key k+m, and every lane receives its own dim of keys
// k..k+3.
template <int D>
__device__ __forceinline__ bf16x8 read_v(const uint16_t* Vs, int h, int mb, int r, int g) {
    using G = Geo<D>;
    const uint16_t* src = Vs + (32 * h + 4 * g + (r >> 2)) * G::VP + 16 * mb + 4 * (r & 3);
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + 16 * G::VP));
    return __builtin_bit_cast(bf16x8, s16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]});
}

// O^T += V^T P^T.
template <int D, int QB, bool FINE>
__device__ __forceinline__ void apply_probs(Acc<D, QB>& acc, const Probs<D, QB, FINE>& P, const uint16_t* Vs, int r,
                                            int g) {
    using G = Geo<D>;
    if constexpr (!G::ONES) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) acc.l[qb] += P.psum[qb];
    }
#pragma unroll
    for (int h = 0; h < BK / 32; ++h) {
#pragma unroll
        for (int mb = 0; mb < G::NDB; ++mb) {
            const bf16x8 va = read_v<D>(Vs, h, mb, r, g);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                acc.o[qb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, P.pb[qb][h], acc.o[qb][mb], 0, 0, 0);
                if constexpr (FINE)
                    acc.o[qb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, P.pl[qb][h], acc.o[qb][mb], 0, 0, 0);
            }
        }
    }
}

// The same for two accumulators with probabilities of their own, each V
// fragment read once.
template <int D, int QB>
__device__ __forceinline__ void apply_probs2(Acc<D, QB>& acc, const Probs<D, QB, false>& P, Acc<D, QB>& ax,
                                             const Probs<D, QB, false>& PX, const uint16_t* Vs, int r, int g) {
    using G = Geo<D>;
    if constexpr (!G::ONES) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            acc.l[qb] += P.psum[qb];
            ax.l[qb] += PX.psum[qb];
        }
    }
#pragma unroll
    for (int h = 0; h < BK / 32; ++h) {
#pragma unroll
        for (int mb = 0; mb < G::NDB; ++mb) {
            const bf16x8 va = read_v<D>(Vs, h, mb, r, g);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                acc.o[qb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, P.pb[qb][h], acc.o[qb][mb], 0, 0, 0);
                ax.o[qb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, PX.pb[qb][h], ax.o[qb][mb], 0, 0, 0);
            }
        }
    }
}

// Online-softmax probabilities of one score tile, with the lazy rescale of the
// accumulator.  S is taken by value: the mask is applied to a private copy.
template <int D, int MASK, int QB, bool FINE>
__device__ __forceinline__ void exact_probs(Acc<D, QB>& acc, Tile<QB> S, int r, int g, int qrow0, int k0, int L, int w,
                                            float c, Probs<D, QB, FINE>& P) {
    using G = Geo<D>;
    mask_tile<MASK>(S, r, g, qrow0, k0, L, w);
    // Lazy rescale.  Each lane compares the largest of its own scores with
    // its query's threshold (m + RESCALE_THRESH) / c; only when some lane of
    // the wavefront exceeds it (one wave-uniform branch) are the exact tile
    // maxima formed over the four lanes that share a query, and the queries
    // whose maximum grew by more than the margin are rescaled.  Otherwise
    // every probability is below 2^8 (2 after the shift).
    float v[QB];
    bool hot = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        v[qb] = NEG_INF;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[qb] = fmaxf(v[qb], S.s[qb][kb][i]);
        hot = hot || v[qb] > acc.thr[qb];
    }
    if (__any(hot)) {
        bool unset = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mx = group_max(v[qb]) * c;
            const float m = acc.running_max(qb);
            if (mx > m + RESCALE_THRESH) {
                const float alpha = __builtin_amdgcn_exp2f(m - mx);
#pragma unroll
                for (int mb = 0; mb < G::NDB; ++mb) acc.o[qb][mb] *= alpha;
                acc.l[qb] *= alpha;
                acc.negm[qb] = -mx - P_SHIFT;
                acc.thr[qb] = (mx + RESCALE_THRESH) / c;
            }
            unset = unset || acc.thr[qb] == NEG_INF;
        }
        acc.fresh = __any(unset);
    }
    form_probs(acc, S, c, P);
}

// The probabilities without the maxima, for a wavefront whose queries all have
// a running max: they are formed first, and one OR over their packed bf16
// words tests whether any reached the rescale margin.  Returns false if one
// did (rare after the first tiles); the caller then scores the tile again and
// takes exact_probs(), which rescales.
template <int D, int MASK, int QB, bool FINE>
__device__ __forceinline__ bool fast_probs(const Acc<D, QB>& acc, Tile<QB> S, int r, int g, int qrow0, int k0, int L,
                                           int w, float c, Probs<D, QB, FINE>& P) {
    mask_tile<MASK>(S, r, g, qrow0, k0, L, w);
    form_probs(acc, S, c, P);
    uint32_t bits = 0u;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int h = 0; h < BK / 32; ++h) {
            const u32x4 wv = __builtin_bit_cast(u32x4, P.pb[qb][h]);
            bits |= wv[0] | wv[1] | wv[2] | wv[3];
        }
    return !__any((bits & P_MARGIN_BITS) != 0u);
}

// Online-softmax update of the accumulator with one score tile, then PV.
template <int D, int MASK, int QB, bool FINE = false>
__device__ __forceinline__ void accumulate(Acc<D, QB>& acc, const Tile<QB>& S, const uint16_t* Vs, int r, int g,
                                           int qrow0, int k0, int L, int w, float c) {
    Probs<D, QB, FINE> P;
    exact_probs<D, MASK>(acc, S, r, g, qrow0, k0, L, w, c, P);
    apply_probs(acc, P, Vs, r, g);
}

// Row sum of one query block, broadcast to every lane of that query.
template <int D, int QB>
__device__ __forceinline__ float row_sum(const Acc<D, QB>& acc, int qb, int r) {
    using G = Geo<D>;
    if constexpr (G::ONES) {
        constexpr int MB = D / 16, GS = (D % 16) / 4, IS = (D % 16) % 4;
        return __shfl(acc.o[qb][MB][IS], r + 16 * GS);
    } else {
        return group_sum(acc.l[qb]);
    }
}

// Direct global -> LDS copy of one K/V tile (no staging registers).  Rows
// beyond L copy row L-1 instead: their scores are masked and their
// probabilities are zero, so any finite value will do.
template <int D>
__device__ __forceinline__ void issue_tile(const uint16_t* __restrict__ Kbh, const uint16_t* __restrict__ Vbh, int k0,
                                           int L, int tid, uint16_t* Ks, uint16_t* Vs) {
    using G = Geo<D>;
    // first chunk of this wavefront in a round: uniform, kept in a scalar
    // register so the LDS destination (M0) needs no per-copy lane read
    const int wave_chunk0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    if (k0 + BK <= L) {
        // whole tile: a uniform tile base plus a per-lane offset that does not
        // depend on the tile (loop-invariant, so no address arithmetic per copy)
        const uint16_t* kb = Kbh + (size_t)k0 * D;
        const uint16_t* vb = Vbh + (size_t)k0 * D;
#pragma unroll
        for (int it = 0; it < G::KROUNDS; ++it) {
            const int c = it * NTHREADS + tid;
            const int row = c / G::KPC, ch = c % G::KPC;
            if (row < BK && ch < G::NCH)
                __builtin_amdgcn_global_load_lds((const void*)(kb + (uint32_t)(row * D + ch * 8)),
                                                 (__attribute__((address_space(3))) void*)(Ks + (it * NTHREADS + wave_chunk0) * 8),
                                                 16, 0, 0);
        }
#pragma unroll
        for (int it = 0; it < G::VROUNDS; ++it) {
            const int c = it * NTHREADS + tid;
            const int row = c / G::VPC, ch = c % G::VPC;
            if (row < BK && ch < G::NCH)
                __builtin_amdgcn_global_load_lds((const void*)(vb + (uint32_t)(row * D + ch * 8)),
                                                 (__attribute__((address_space(3))) void*)(Vs + (it * NTHREADS + wave_chunk0) * 8),
                                                 16, 0, 0);
        }
        return;
    }
#pragma unroll
    for (int it = 0; it < G::KROUNDS; ++it) {
        const int c = it * NTHREADS + tid;
        const int row = c / G::KPC, ch = c % G::KPC;
        if (row < BK && ch < G::NCH) {
            const int krow = min(k0 + row, L - 1);
            __builtin_amdgcn_global_load_lds((const void*)(Kbh + (size_t)krow * D + ch * 8),
                                             (__attribute__((address_space(3))) void*)(Ks + (it * NTHREADS + wave_chunk0) * 8),
                                             16, 0, 0);
        }
    }
#pragma unroll
    for (int it = 0; it < G::VROUNDS; ++it) {
        const int c = it * NTHREADS + tid;
        const int row = c / G::VPC, ch = c % G::VPC;
        if (row < BK && ch < G::NCH) {
            const int vrow = min(k0 + row, L - 1);
            __builtin_amdgcn_global_load_lds((const void*)(Vbh + (size_t)vrow * D + ch * 8),
                                             (__attribute__((address_space(3))) void*)(Vs + (it * NTHREADS + wave_chunk0) * 8),
                                             16, 0, 0);
        }
    }
}

// Direct global -> LDS copy of n16 16-byte chunks starting at src (the
// residual rows of a workgroup, at most NR chunks), chunk c landing at byte
// 16 c of dst.  Addressed as a uniform base plus a 32-bit lane offset formed
// here, so that no address stays live across the tile loop.
template <int NR>
__device__ __forceinline__ void issue_rows(const float* __restrict__ src, int n16, int tid, uint16_t* dst) {
    const int wave_chunk0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    uint32_t off = (uint32_t)tid * 16u;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int it = 0; it < (NR + NTHREADS - 1) / NTHREADS; ++it) {
        if (it * NTHREADS + tid < n16)
            __builtin_amdgcn_global_load_lds((const void*)((const char*)src + off + (uint32_t)(it * NTHREADS * 16)),
                                             (__attribute__((address_space(3))) void*)(dst + 8 * (it * NTHREADS + wave_chunk0)),
                                             16, 0, 0);
    }
}

// Per-workgroup state of the tile walk.  FAST: the tiles of PLAIN segments
// take the fast form of the softmax update (a band segment's unmasked tiles
// keep the exact form: both forms beside the masks exceed the register budget).
template <int D, int QB, bool FAST = false>
struct Walk {
    using G = Geo<D>;
    const uint16_t* Kbh;
    const uint16_t* Vbh;
    uint16_t* smem;
    int tid, r, g, L, w, qw0, qhi_w;
    bool wave_active;
    float c;
    int stage;
    // Residual rows copied into the free LDS stage while the last tile is
    // used, so that the epilogue does not wait on their global read (null:
    // none); rpre_n16 16-byte chunks.
    const float* rpre;
    int rpre_n16;

    // Visit tiles [t0, t1) with one segment kind; `next_after` is the first
    // tile of the next non-empty segment (-1: none), prefetched while the
    // last tile of this segment is used.
    template <int KIND, bool FINE = false>
    __device__ __forceinline__ void run(Acc<D, QB>& acc, const QFrag<D, QB>& q, int t0, int t1, int next_after) {
        // the walk's last tile is peeled when residual rows are to be copied
        const int tl = (next_after < 0 && rpre) ? t1 - 1 : t1;
        for (int t = t0; t < tl; ++t) {
            const uint16_t* Ks = smem + stage * G::STAGE_ELEMS;
            const uint16_t* Vs = Ks + G::KS_ELEMS;
            const int next = (t + 1 < t1) ? t + 1 : next_after;
            if (next >= 0) {
                uint16_t* Kn = smem + (stage ^ 1) * G::STAGE_ELEMS;
                issue_tile<D>(Kbh, Vbh, next * BK, L, tid, Kn, Kn + G::KS_ELEMS);
            }
            if (wave_active) tile<KIND, FINE>(acc, q, Ks, Vs, t * BK);
            wait_vm_all();
            __syncthreads();
            stage ^= 1;
        }
        if (tl < t1 && t0 < t1) {
            const uint16_t* Ks = smem + stage * G::STAGE_ELEMS;
            const uint16_t* Vs = Ks + G::KS_ELEMS;
            issue_rows<bq<QB>() * D / 4>(rpre, rpre_n16, tid, smem + (stage ^ 1) * G::STAGE_ELEMS);
            if (wave_active) tile<KIND, FINE>(acc, q, Ks, Vs, tl * BK);
            wait_vm_all();
            __syncthreads();
            stage ^= 1;
        }
    }

    // Single pass over tiles [t0, t1) with two accumulators: the in-band
    // scores of each tile go to aw, the out-of-band ones to ax.  A tile that
    // is inside or outside the band for all of the wavefront's queries feeds
    // one of them; a band-edge tile is scored once and feeds both.
    __device__ __forceinline__ void run_split(Acc<D, QB>& aw, Acc<D, QB>& ax, const QFrag<D, QB>& q, int t0, int t1) {
        for (int t = t0; t < t1; ++t) {
            const uint16_t* Ks = smem + stage * G::STAGE_ELEMS;
            const uint16_t* Vs = Ks + G::KS_ELEMS;
            if (t + 1 < t1) {
                uint16_t* Kn = smem + (stage ^ 1) * G::STAGE_ELEMS;
                issue_tile<D>(Kbh, Vbh, (t + 1) * BK, L, tid, Kn, Kn + G::KS_ELEMS);
            }
            if (wave_active) tile_split(aw, ax, q, Ks, Vs, t * BK);
            wait_vm_all();
            __syncthreads();
            stage ^= 1;
        }
    }

    __device__ __forceinline__ int classify(int k0) const {
        const int khi = min(k0 + BK - 1, L - 1);
        const int mind = khi < qw0 ? qw0 - khi : (k0 > qhi_w ? k0 - qhi_w : 0);
        const int maxd = max(qhi_w - k0, khi - qw0);
        return maxd <= w ? TILE_INSIDE : (mind > w ? TILE_OUTSIDE : TILE_BOUNDARY);
    }

    __device__ __forceinline__ void tile_split(Acc<D, QB>& aw, Acc<D, QB>& ax, const QFrag<D, QB>& q,
                                               const uint16_t* Ks, const uint16_t* Vs, int k0) {
        const bool ragged = k0 + BK > L;
        const int cls = classify(k0);
        Tile<QB> S;
        score_tile<D>(Ks, q, S, r, g);
        if (cls == TILE_BOUNDARY) {
            // One band test per score deals it to one of the two, and each V
            // fragment is read once for both: against a mask and a PV pass of
            // its own for each, 79.1 -> 75 us at (32, 16, 405, 72), 28.9 ->
            // 24.1 us at (8, 16, 500, 64), where registers also fell from 154
            // to 127 and a fourth wavefront per SIMD fits.
            Tile<QB> X;
            if (ragged) mask_tile<MASK_KEYS>(S, r, g, qw0, k0, L, w);
            split_tile(S, X, r, g, qw0, k0, L, w);
            Probs<D, QB, false> P, PX;
            exact_probs<D, MASK_NONE>(aw, S, r, g, qw0, k0, L, w, c, P);
            exact_probs<D, MASK_NONE>(ax, X, r, g, qw0, k0, L, w, c, PX);
            apply_probs2(aw, P, ax, PX, Vs, r, g);
        } else if (cls == TILE_INSIDE) {
            if (ragged) accumulate<D, MASK_KEYS>(aw, S, Vs, r, g, qw0, k0, L, w, c);
            else accumulate<D, MASK_NONE>(aw, S, Vs, r, g, qw0, k0, L, w, c);
        } else {
            if (ragged) accumulate<D, MASK_KEYS>(ax, S, Vs, r, g, qw0, k0, L, w, c);
            else accumulate<D, MASK_NONE>(ax, S, Vs, r, g, qw0, k0, L, w, c);
        }
    }

    // A tile of a window walk in two forms, masked (which also cuts keys beyond
    // L) and plain: fewer registers than the three of a band segment.
    __device__ __forceinline__ void tile_window(Acc<D, QB>& acc, const QFrag<D, QB>& q, const uint16_t* Ks,
                                                const uint16_t* Vs, int k0) {
        const int cls = classify(k0);
        if (cls == TILE_OUTSIDE) return;
        Tile<QB> S;
        score_tile<D>(Ks, q, S, r, g);
        if (cls == TILE_BOUNDARY || k0 + BK > L) accumulate<D, MASK_BAND_IN>(acc, S, Vs, r, g, qw0, k0, L, w, c);
        else accumulate<D, MASK_NONE>(acc, S, Vs, r, g, qw0, k0, L, w, c);
    }

    // One update with the score tile S of the tile at k0.  With F, an unmasked
    // tile takes the fast form once every query of the wavefront has a running
    // max, and the exact form before that and when the fast form finds a
    // probability at the rescale margin (the tile is then scored again, so
    // that no second score tile stays live across the fast form).
    template <int MASK, bool FINE, bool F = FAST>
    __device__ __forceinline__ void update(Acc<D, QB>& acc, const QFrag<D, QB>& q, Tile<QB>& S, const uint16_t* Ks,
                                           const uint16_t* Vs, int k0) {
        Probs<D, QB, FINE> P;
        if constexpr (F && MASK == MASK_NONE) {
            if (acc.fresh || !fast_probs<D, MASK>(acc, S, r, g, qw0, k0, L, w, c, P)) {
                if (!acc.fresh) {
                    // a compiler barrier: the tile is read and scored again, not kept
                    asm volatile("" ::: "memory");
                    score_tile<D>(Ks, q, S, r, g);
                }
                exact_probs<D, MASK>(acc, S, r, g, qw0, k0, L, w, c, P);
            }
        } else {
            exact_probs<D, MASK>(acc, S, r, g, qw0, k0, L, w, c, P);
        }
        apply_probs(acc, P, Vs, r, g);
    }

    template <int KIND, bool FINE>
    __device__ __forceinline__ void tile(Acc<D, QB>& acc, const QFrag<D, QB>& q, const uint16_t* Ks, const uint16_t* Vs,
                                         int k0) {
        if constexpr (KIND == SEG_PLAIN) {
            Tile<QB> S;
            score_tile<D>(Ks, q, S, r, g);
            update<MASK_NONE, FINE>(acc, q, S, Ks, Vs, k0);
        } else if constexpr (KIND == SEG_KEYS) {
            Tile<QB> S;
            score_tile<D>(Ks, q, S, r, g);
            update<MASK_KEYS, FINE>(acc, q, S, Ks, Vs, k0);
        } else {
            // classify the tile against this wavefront's queries
            const bool ragged = k0 + BK > L;
            const int cls = classify(k0);
            constexpr int SKIP = (KIND == SEG_BAND_IN) ? TILE_OUTSIDE : TILE_INSIDE;
            if (cls == SKIP) return;
            Tile<QB> S;
            score_tile<D>(Ks, q, S, r, g);
            if (cls == TILE_BOUNDARY)
                update<KIND == SEG_BAND_IN ? MASK_BAND_IN : MASK_BAND_OUT, FINE>(acc, q, S, Ks, Vs, k0);
            else if (ragged)
                update<MASK_KEYS, FINE>(acc, q, S, Ks, Vs, k0);
            else
                update<MASK_NONE, FINE, false>(acc, q, S, Ks, Vs, k0);
        }
    }
};

template <int KMODE>
constexpr bool split_refresh() { return KMODE == MODE_REFRESH_SPLIT; }

// Orders a wavefront's LDS accesses before and after it (its lanes hand values
// to each other; a wavefront's LDS accesses complete in order).
__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Pitch, in elements, of 16 output rows on their way through LDS: rows of bf16
// and of fp32 spread over the banks for both head dims.
constexpr int OUT_PITCH = 72;
constexpr int OUT_ELEMS = 16 * OUT_PITCH;   // bf16 elements of a wavefront's rows; fp32 rows take twice that

// Stores the 16 rows of a query block to every destination, the first `rows`
// of them, from row offset `at`.  A lane holds 4 dims of one query, so stores
// straight from it write 32-byte (bf16) or 64-byte (fp32) pieces of 16 rows;
// passed through LDS `Wl` (the wavefront's own), they leave as whole lines in
// row order.  O is allocated in the caches, since a caller's next launch (the
// output projection) reads it; its cache and R, which a later step reads, are
// not.  O without allocation takes 1-2 us off the call and puts 6-7 on the
// projection behind it, us of the call, then of both, without and with: full
// (810, 16, 16, 72) 23.4, 24.8 and 72.5, 65.6; (32, 16, 405, 72) 46.8, 47.9
// and 97.4, 90.2; reuse (8, 16, 1024, 72) 33.0, 33.8 and 67.6, 61.1; from
// 75 MB of O on the pairs are level.  R in whole lines without allocation,
// against direct stores: refresh (8, 16, 1024, 72) 82.9 -> 76.7.
template <int D>
__device__ __forceinline__ void store_rows(const Params& p, const u32x2 (&o)[Geo<D>::NDB], uint16_t* Wl, size_t at, int rows,
                                           int lane) {
    using G = Geo<D>;
    const int r = lane & 15, g = lane >> 4;
    lds_fence();
#pragma unroll
    for (int mb = 0; mb < G::NDB; ++mb)
        if (16 * mb + 4 * g < D) *(u32x2*)(Wl + r * OUT_PITCH + 16 * mb + 4 * g) = o[mb];
    lds_fence();
    constexpr int NIT = (16 * G::NCH + 63) / 64;
    u32x4 v[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int idx = it * 64 + lane, row = idx / G::NCH, ch = idx - row * G::NCH;
        v[it] = u32x4{0u, 0u, 0u, 0u};
        if (idx < 16 * G::NCH) v[it] = *(const u32x4*)(Wl + row * OUT_PITCH + 8 * ch);
    }
    for (int di = 0; di < p.nout; ++di) {
        u32x4* out = (u32x4*)(p.dst[di] + at);
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            if (it * 64 + lane < rows * G::NCH) out[it * 64 + lane] = v[it];
    }
    for (int di = p.nout; di < p.ndst; ++di) {
        u32x4* out = (u32x4*)(p.dst[di] + at);
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            if (it * 64 + lane < rows * G::NCH) __builtin_nontemporal_store(v[it], out + it * 64 + lane);
    }
}

// The same for the residual, fp32, without allocation.
template <int D>
__device__ __forceinline__ void store_residual(const Params& p, const f32x4 (&o)[Geo<D>::NDB], uint16_t* Wl, size_t at,
                                               int rows, int lane) {
    using G = Geo<D>;
    const int r = lane & 15, g = lane >> 4;
    float* Wf = (float*)Wl;
    lds_fence();
#pragma unroll
    for (int mb = 0; mb < G::NDB; ++mb)
        if (16 * mb + 4 * g < D) *(f32x4*)(Wf + r * OUT_PITCH + 16 * mb + 4 * g) = o[mb];
    lds_fence();
    constexpr int N4 = D / 4;
#pragma unroll
    for (int it = 0; it < (16 * N4 + 63) / 64; ++it) {
        const int idx = it * 64 + lane, row = idx / N4, c4 = idx - row * N4;
        if (idx < rows * N4) __builtin_nontemporal_store(*(const f32x4*)(Wf + row * OUT_PITCH + 4 * c4), (f32x4*)(p.Rout + at) + idx);
    }
}

// Epilogue of a two-accumulator refresh: W = aw / lw, O from both, each scaled
// from its own running max to the larger one, R = O - W.
template <int D, int QB, bool ROWS>
__device__ __forceinline__ void store_split(const Params& p, const Acc<D, QB>& aw, const Acc<D, QB>& ax, size_t head_off,
                                            int qw0, int L, int w, uint16_t* Wl, int lane) {
    using G = Geo<D>;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q0 = qw0 + 16 * qb;
        // row sums first: they exchange values across lanes
        const float lw = row_sum<D>(aw, qb, lane & 15), lx = row_sum<D>(ax, qb, lane & 15);
        // whether the query has keys outside its band (not whether ax has a
        // maximum: it has none if all of their scores are NaN)
        const int qi = q0 + (lane & 15);
        const bool has_x = qi > w || qi < L - 1 - w;
        const float mw = aw.running_max(qb);
        const float mx = ax.running_max(qb);
        const float mm = fmaxf(mw, mx);
        const float sw = has_x ? __builtin_amdgcn_exp2f(mw - mm) : 1.f;
        const float sx = has_x ? __builtin_amdgcn_exp2f(mx - mm) : 0.f;
        const float invw = 1.f / lw;
        const float inv = 1.f / (lw * sw + lx * sx);
        const size_t at = head_off + (size_t)q0 * D;
        const int rows = min(16, L - q0);
        f32x4 res[G::NDB];
        u32x2 ob[G::NDB];
#pragma unroll
        for (int mb = 0; mb < G::NDB; ++mb) {
#pragma clang fp contract(off)
            const f32x4 wv = aw.o[qb][mb] * invw;
            const f32x4 o = has_x ? (aw.o[qb][mb] * sw + ax.o[qb][mb] * sx) * inv : wv;
            res[mb] = o - wv;
            ob[mb] = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
        }
        if constexpr (ROWS) {
            store_residual<D>(p, res, Wl, at, rows, lane);
            store_rows<D>(p, ob, Wl, at, rows, lane);
        } else if (qi < L) {
#pragma unroll
            for (int mb = 0; mb < G::NDB; ++mb) {
                const int col = 16 * mb + 4 * (lane >> 4);
                if (col >= D) continue;
                const size_t off = head_off + (size_t)qi * D + col;
                *(f32x4*)(p.Rout + off) = res[mb];
                for (int di = 0; di < p.ndst; ++di) *(u32x2*)(p.dst[di] + off) = ob[mb];
            }
        }
    }
}

// Refresh in one pass (Sec. 3.2, Eq. 1), for short sequences: W = aw / lw from the in-band scores
// alone; O combines both accumulators, each scaled from its own running max
// to the larger one.  A query whose band covers every key has no
// out-of-band score, and its O is then formed exactly as W, so R == 0.
template <int D, int QB, bool ROWS>
__device__ __forceinline__ void refresh_split(const Params& p, uint16_t* smem, Walk<D, QB, false>& wk, const QFrag<D, QB>& q,
                                              size_t head_off, int ntiles) {
    using G = Geo<D>;
    Acc<D, QB> aw, ax;
    aw.init();
    ax.init();
    issue_tile<D>(wk.Kbh, wk.Vbh, 0, wk.L, wk.tid, smem, smem + G::KS_ELEMS);
    wait_vm_all();
    __syncthreads();
    wk.run_split(aw, ax, q, 0, ntiles);
    if (wk.wave_active) store_split<D, QB, ROWS>(p, aw, ax, head_off, wk.qw0, wk.L, wk.w, smem + (wk.tid >> 6) * 2 * OUT_ELEMS, wk.tid & 63);
}

template <int D, int KMODE, int QB, bool ROWS>
__device__ __forceinline__ void attn_body(const Params& p, uint16_t* smem) {
    using G = Geo<D>;
    constexpr int MODE = KMODE == MODE_ASC             ? MODE_FULL
                         : KMODE == MODE_REFRESH_SPLIT ? MODE_REFRESH
                         : KMODE == MODE_REFRESH_FINE  ? MODE_REFRESH
                         : KMODE == MODE_WINDOW_FINE   ? MODE_WINDOW
                                                       : KMODE;
    // split probabilities in the in-band segments (the window attention)
    constexpr bool FINE = KMODE == MODE_WINDOW_FINE || KMODE == MODE_REFRESH_FINE;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int r = lane & 15;
    const int g = lane >> 4;

    // XCD-aware block order: workgroups are dealt to the 8 XCDs round-robin,
    // so give each XCD a contiguous range of (head, query-tile) work and the
    // workgroups sharing an XCD's L2 read the same K/V.
    int blk = blockIdx.x;
    if ((p.nblocks & 7) == 0) blk = (blk & 7) * (p.nblocks >> 3) + (blk >> 3);
    const int bh = blk / p.n_qt;
    const int qt = blk % p.n_qt;
    const int L = p.L, w = p.w;
    const size_t head_off = (size_t)bh * L * D;
    const uint16_t* __restrict__ Qbh = p.Q + head_off;

    const int q0 = qt * bq<QB>();                 // workgroup's first query
    const int qw0 = q0 + wave * (QB * 16);       // wavefront's first query
    const int qhi_wg = min(q0 + bq<QB>() - 1, L - 1);
    const int qhi_w = min(qw0 + QB * 16 - 1, L - 1);

    // constant V padding chunk of every row in both stages: (1, 0, ..., 0) for
    // the row-sum column, never overwritten by the tile copies
    if constexpr (G::ONES) {
        for (int idx = tid; idx < 2 * BK * 8; idx += NTHREADS) {
            const int st = idx / (BK * 8), row = (idx / 8) % BK, e = idx % 8;
            smem[st * G::STAGE_ELEMS + G::KS_ELEMS + row * G::VP + D + e] = (e == 0) ? (uint16_t)0x3F80u : (uint16_t)0u;
        }
    }

    // Q fragments, zero beyond L and beyond d.  load_q in line: called, the window
    // walk of 512 workgroups at (8, 16, 256, 72) takes 9.28 us, in line 9.25 (31
    // rounds in turn, twice; 9.06 and 9.01 on another card).
    QFrag<D, QB> q;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qrow = qw0 + 16 * qb + r;
        const bool ok = qrow < L;
        const uint16_t* qp = Qbh + (size_t)(ok ? qrow : 0) * D;
#pragma unroll
        for (int c = 0; c < G::NC32; ++c)
            q.a[qb][c] = as_bf16x8(ok ? *(const u32x4*)(qp + 32 * c + 8 * g) : u32x4{0u, 0u, 0u, 0u});
        q.t[qb] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
        if constexpr (G::TAIL > 0) {
            if (ok && 8 * g < G::TAIL) q.t[qb] = as_bf16x8(*(const u32x4*)(qp + G::D32 + 8 * g));
        }
    }

    // the fast update measured 1-2% faster in the long walks of two query
    // blocks per wavefront and about 1% slower in the short walks of one
    Walk<D, QB, QB == 2 && !split_refresh<KMODE>()> wk;
    wk.Kbh = p.K + head_off;
    wk.Vbh = p.V + head_off;
    wk.smem = smem;
    wk.tid = tid;
    wk.r = r;
    wk.g = g;
    wk.L = L;
    wk.w = w;
    wk.qw0 = qw0;
    wk.qhi_w = qhi_w;
    wk.wave_active = qw0 < L;
    wk.c = p.c;
    wk.stage = 0;
    wk.rpre = nullptr;
    wk.rpre_n16 = 0;
    // 64-query window walks take their residual rows through the LDS stage
    // that the last tile leaves free (one stage holds 64 fp32 rows of d <= 72)
    if constexpr (MODE == MODE_WINDOW && QB == 1) {
        static_assert(bq<1>() * D * 4 <= G::STAGE_ELEMS * 2, "residual rows must fit one LDS stage");
        if (p.Rin) {
            wk.rpre = p.Rin + head_off + (size_t)q0 * D;
            wk.rpre_n16 = (min(L, q0 + bq<1>()) - q0) * D / 4;
        }
    }

    // segments of the tile walk
    const int ntiles = (L + BK - 1) / BK, nfull = L / BK;
    int tb0 = 0, tb1 = ntiles - 1, m0 = 0, m1 = 0;
    if constexpr (MODE != MODE_FULL) {
        const long long klo = max(0LL, (long long)q0 - w);
        const long long khi = min((long long)L - 1, (long long)qhi_wg + w);
        tb0 = (int)(klo / BK);
        tb1 = (int)(khi / BK);
        // tiles inside the band for every query of the workgroup and not ragged
        const long long lo_key = (long long)qhi_wg - w;                      // first key every query reaches
        const long long hi_key = min((long long)q0 + w, (long long)L - 1);  // last key every query reaches
        const long long ai0 = lo_key <= 0 ? 0 : (lo_key + BK - 1) / BK;
        const long long ai1 = hi_key - (BK - 1) < 0 ? -1 : (hi_key - (BK - 1)) / BK;
        m0 = (int)min(max(ai0, (long long)tb0), (long long)tb1 + 1);
        m1 = (int)min(max(ai1 + 1, (long long)m0), (long long)tb1 + 1);
    }
    constexpr int NSEG = MODE == MODE_FULL ? 2 : (MODE == MODE_WINDOW ? 3 : 8);
    int s0[NSEG], s1[NSEG];
    if constexpr (MODE == MODE_FULL) {
        s0[0] = 0; s1[0] = nfull;              // PLAIN
        s0[1] = nfull; s1[1] = ntiles;         // KEYS
    } else {
        s0[0] = tb0; s1[0] = m0;               // BAND_IN
        s0[1] = m0; s1[1] = m1;                // PLAIN
        s0[2] = m1; s1[2] = tb1 + 1;           // BAND_IN
        if constexpr (MODE == MODE_REFRESH) {
            const int after = max(tb1 + 1, nfull);
            s0[3] = 0; s1[3] = tb0;            // PLAIN (left of the band)
            s0[4] = tb0; s1[4] = m0;           // BAND_OUT
            s0[5] = m1; s1[5] = tb1 + 1;       // BAND_OUT
            s0[6] = tb1 + 1; s1[6] = after;    // PLAIN (right of the band)
            s0[7] = after; s1[7] = ntiles;     // KEYS (ragged tile right of the band)
        }
    }
    // first tile of the first non-empty segment at or after each position
    int nxt[NSEG + 1];
    nxt[NSEG] = -1;
#pragma unroll
    for (int i = NSEG - 1; i >= 0; --i) nxt[i] = s0[i] < s1[i] ? s0[i] : nxt[i + 1];

    if constexpr (split_refresh<KMODE>()) {
        refresh_split<D, QB, ROWS>(p, smem, wk, q, head_off, ntiles);
        return;
    }

    Acc<D, QB> acc;
    acc.init();

    // every workgroup has at least one key tile: the window of any query
    // contains the query itself
    issue_tile<D>(wk.Kbh, wk.Vbh, nxt[0] * BK, L, tid, smem, smem + G::KS_ELEMS);
    wait_vm_all();
    __syncthreads();

    if constexpr (MODE == MODE_FULL) {
        wk.template run<SEG_PLAIN>(acc, q, s0[0], s1[0], nxt[1]);
        wk.template run<SEG_KEYS>(acc, q, s0[1], s1[1], nxt[2]);
    } else {
        wk.template run<SEG_BAND_IN, FINE>(acc, q, s0[0], s1[0], nxt[1]);
        wk.template run<SEG_PLAIN, FINE>(acc, q, s0[1], s1[1], nxt[2]);
        wk.template run<SEG_BAND_IN, FINE>(acc, q, s0[2], s1[2], nxt[3]);
    }

    if constexpr (MODE == MODE_REFRESH) {
        // the accumulator now holds the window attention of the wavefront's
        // queries: park W (fp32) in the R buffer
        if (wk.wave_active) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int qrow = qw0 + 16 * qb + r;
                const float inv = 1.f / row_sum<D>(acc, qb, r);
                if (qrow < L) {
#pragma unroll
                    for (int mb = 0; mb < G::NDB; ++mb) {
                        const int col = 16 * mb + 4 * g;
                        if (col < D) *(f32x4*)(p.Rout + head_off + (size_t)qrow * D + col) = acc.o[qb][mb] * inv;
                    }
                }
            }
        }
        wk.template run<SEG_PLAIN>(acc, q, s0[3], s1[3], nxt[4]);
        wk.template run<SEG_BAND_OUT>(acc, q, s0[4], s1[4], nxt[5]);
        wk.template run<SEG_BAND_OUT>(acc, q, s0[5], s1[5], nxt[6]);
        wk.template run<SEG_PLAIN>(acc, q, s0[6], s1[6], nxt[7]);
        wk.template run<SEG_KEYS>(acc, q, s0[7], s1[7], nxt[8]);
    }

    if (!wk.wave_active) return;

    // epilogue: normalise, form R, store bf16 to every destination, through LDS
    // as whole lines (ROWS) or straight from the registers
    static_assert(NWAVES * OUT_ELEMS <= G::STAGE_ELEMS && NWAVES * 2 * OUT_ELEMS <= 2 * G::STAGE_ELEMS, "output rows must fit");
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qrow = qw0 + 16 * qb + r;
        const float inv = 1.f / row_sum<D>(acc, qb, r);
        if (!ROWS && qrow >= L) continue;
        const size_t row_off = head_off + (size_t)qrow * D;
        f32x4 res[G::NDB];
        u32x2 ob[G::NDB];
#pragma unroll
        for (int mb = 0; mb < G::NDB; ++mb) {
            // no fma contraction: o must be rounded exactly as the parked W was
#pragma clang fp contract(off)
            const int col = 16 * mb + 4 * g;
            const bool ok = qrow < L && col < D;
            if (!ROWS && !ok) continue;
            const size_t off = row_off + col;
            const f32x4 o = acc.o[qb][mb] * inv;
            f32x4 out = o;
            if constexpr (MODE == MODE_REFRESH) {
                // R is the exact difference of the two rounded fp32 results (a
                // band covering every key gives R == 0 exactly); the window
                // result parked above is read back by the lane that wrote it.
                res[mb] = o;
                if (ok) res[mb] = o - *(const f32x4*)(p.Rout + off);
            }
            if constexpr (MODE == MODE_WINDOW) {
                if (wk.rpre) {
                    // the walk's last iteration left the rows in the stage it freed
                    const float* rl = (const float*)(smem + wk.stage * G::STAGE_ELEMS);
                    if (ok) out = o + *(const f32x4*)(rl + (qrow - q0) * D + col);
                } else if (p.Rin) {
                    if (ok) out = o + *(const f32x4*)(p.Rin + off);
                }
            }
            ob[mb] = u32x2{pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
            if constexpr (!ROWS) {
                if constexpr (MODE == MODE_REFRESH) *(f32x4*)(p.Rout + off) = res[mb];
                for (int di = 0; di < p.ndst; ++di) *(u32x2*)(p.dst[di] + off) = ob[mb];
            }
        }
        if constexpr (ROWS) {
            // through the stage that holds no residual rows (both stages are
            // free after the walk's last barrier)
            uint16_t* Wl = MODE == MODE_REFRESH ? smem + wave * 2 * OUT_ELEMS
                                                : smem + (wk.stage ^ 1) * G::STAGE_ELEMS + wave * OUT_ELEMS;
            int el = tid;   // opaque: nothing of the stores' addressing is formed before the walk
            asm volatile("" : "+v"(el));
            const size_t at = head_off + (size_t)(qw0 + 16 * qb) * D;
            const int rows = min(16, L - (qw0 + 16 * qb));
            if constexpr (MODE == MODE_REFRESH) store_residual<D>(p, res, Wl, at, rows, el & 63);
            store_rows<D>(p, ob, Wl, at, rows, el & 63);
        }
    }
}

// Three waves per SIMD with two query blocks per wavefront (register budget
// 168), four with one (budget 128): the MFMA work of one wavefront overlaps the
// softmax arithmetic of the others.  The two-accumulator refresh fits four at
// d = 64 (127 registers; 27.0 -> 23.9 us at (8, 16, 500, 64)); at d = 72 it
// needs 143, and in 128 it spills (77.4 -> 82.1 us at (32, 16, 405, 72)).
template <int D, int QB, int KMODE>
constexpr int waves_per_simd() { return QB == 1 && (D == 64 || !split_refresh<KMODE>()) ? 4 : 3; }

template <int D, int MODE, int QB, bool ROWS>
__global__ void __launch_bounds__(NTHREADS)
    __attribute__((amdgpu_waves_per_eu(waves_per_simd<D, QB, MODE>(), waves_per_simd<D, QB, MODE>()))) attn_kernel(Params p) {
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * Geo<D>::STAGE_ELEMS];
    attn_body<D, MODE, QB, ROWS>(p, smem);
}

// ---------------------------------------------------------------------------
// Launches that leave SIMDs short of wavefronts: the key tiles of a 64-query
// workgroup are dealt to KS groups of four wavefronts, each with LDS stages, a
// running maximum and accumulators of its own, and group 0 combines them.  At
// one wavefront per SIMD a tile costs its whole dependence chain (scores, exp,
// PV: 0.64 us), several times its issue time; deeper copy pipelines did not
// help there.
// ---------------------------------------------------------------------------

// Wavefronts per SIMD that its register budget allows for.
template <int KMODE, int KS>
constexpr int keysplit_waves() { return KMODE == MODE_REFRESH ? KS : 4; }

// One query block's state as a wavefront leaves it in LDS: 16 bytes per lane
// and output block, then (-m - P_SHIFT, threshold, row-sum share).
template <int D>
constexpr int state_elems() { return (Geo<D>::NDB + 1) * 64 * 8; }

template <int D>
__device__ __forceinline__ void put_state(const Acc<D, 1>& a, uint16_t* at, int lane) {
#pragma unroll
    for (int mb = 0; mb < Geo<D>::NDB; ++mb) *(f32x4*)(at + (mb * 64 + lane) * 8) = a.o[0][mb];
    *(f32x4*)(at + (Geo<D>::NDB * 64 + lane) * 8) = f32x4{a.negm[0], a.thr[0], a.l[0], 0.f};
}

// a += the state at `at`, both scaled to the larger running maximum.  A state
// without a maximum saw no key of these queries, and is zero, or only scores
// that set none (NaN, -inf): its accumulator may then hold a NaN, which a
// factor of 0 passes on, so no state is skipped.
template <int D>
__device__ __forceinline__ void add_state(Acc<D, 1>& a, const uint16_t* at, int lane, float c) {
    const f32x4 st = *(const f32x4*)(at + (Geo<D>::NDB * 64 + lane) * 8);
    const float ma = a.running_max(0), mb_ = st[1] == NEG_INF ? NEG_INF : -(st[0] + P_SHIFT);
    const float m = fmaxf(ma, mb_);
    const float sa = ma == NEG_INF ? 0.f : __builtin_amdgcn_exp2f(ma - m);
    const float sb = mb_ == NEG_INF ? 0.f : __builtin_amdgcn_exp2f(mb_ - m);
#pragma unroll
    for (int mb = 0; mb < Geo<D>::NDB; ++mb) a.o[0][mb] = a.o[0][mb] * sa + *(const f32x4*)(at + (mb * 64 + lane) * 8) * sb;
    a.l[0] = a.l[0] * sa + st[2] * sb;
    if (m != NEG_INF) {
        a.negm[0] = -m - P_SHIFT;
        a.thr[0] = (m + RESCALE_THRESH) / c;
    }
}

template <int D, int KMODE, int KS>
__global__ void __launch_bounds__(NTHREADS* KS) __attribute__((amdgpu_waves_per_eu(keysplit_waves<KMODE, KS>(), keysplit_waves<KMODE, KS>())))
attn_keysplit_kernel(Params p) {
    using G = Geo<D>;
    constexpr int MODE = KMODE == MODE_ASC ? MODE_FULL : KMODE;
    __shared__ __attribute__((aligned(16))) uint16_t smem[KS * 2 * G::STAGE_ELEMS];
    // states of groups 1 .. KS - 1: behind group 0's stages (which may hold
    // residual rows), or from the start for a refresh's two accumulators
    constexpr int NACC = MODE == MODE_REFRESH ? 2 : 1, STATE0 = MODE == MODE_REFRESH ? 0 : 2 * G::STAGE_ELEMS;
    constexpr int STATES = NWAVES * state_elems<D>();
    // a refresh's outputs leave through LDS behind the states
    constexpr int OUT = MODE == MODE_REFRESH ? NWAVES * 2 * OUT_ELEMS : 0;
    static_assert(STATE0 + (KS - 1) * NACC * STATES + OUT <= KS * 2 * G::STAGE_ELEMS, "the states must fit the stages");
    static_assert(bq<1>() * D * 4 <= G::STAGE_ELEMS * 2, "residual rows must fit one LDS stage");
    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NTHREADS);
    const int tid = threadIdx.x % NTHREADS;
    const int lane = tid & 63, wave = tid >> 6, r = lane & 15, g = lane >> 4;
    uint16_t* sg = smem + grp * 2 * G::STAGE_ELEMS;    // the group's stages

    int blk = blockIdx.x;
    if ((p.nblocks & 7) == 0) blk = (blk & 7) * (p.nblocks >> 3) + (blk >> 3);
    const int bh = blk / p.n_qt, qt = blk % p.n_qt;
    const int L = p.L, w = p.w;
    const size_t head_off = (size_t)bh * L * D;
    const int q0 = qt * bq<1>(), qw0 = q0 + wave * 16;

    if constexpr (G::ONES) {
        for (int idx = tid; idx < 2 * BK * 8; idx += NTHREADS) {
            const int st = idx / (BK * 8), row = (idx / 8) % BK, e = idx % 8;
            sg[st * G::STAGE_ELEMS + G::KS_ELEMS + row * G::VP + D + e] = (e == 0) ? (uint16_t)0x3F80u : (uint16_t)0u;
        }
    }
    Walk<D, 1> wk;
    wk.Kbh = p.K + head_off;
    wk.Vbh = p.V + head_off;
    wk.smem = sg;
    wk.tid = tid;
    wk.r = r;
    wk.g = g;
    wk.L = L;
    wk.w = w;
    wk.qw0 = qw0;
    wk.qhi_w = min(qw0 + 15, L - 1);
    wk.wave_active = qw0 < L;
    wk.c = p.c;
    wk.stage = 0;
    wk.rpre = nullptr;

    // tiles [t0, t1) of the walk, tile t0 + i KS + grp for group grp
    int t0 = 0, t1 = (L + BK - 1) / BK;
    if constexpr (MODE == MODE_WINDOW) {
        t0 = (int)(max(0LL, (long long)q0 - w) / BK);
        t1 = (int)(min((long long)L - 1, (long long)min(q0 + bq<1>() - 1, L - 1) + w) / BK) + 1;
    }
    const int iters = (t1 - t0 + KS - 1) / KS;
    t0 += grp;
    if (t0 < t1) issue_tile<D>(wk.Kbh, wk.Vbh, t0 * BK, L, tid, sg, sg + G::KS_ELEMS);

    QFrag<D, 1> q;
    load_q<D, 1>(q, p.Q + head_off, qw0, L, r, g);
    Acc<D, 1> acc, ax;
    acc.init();
    ax.init();
    wait_vm_all();
    __syncthreads();
    for (int i = 0; i < iters; ++i) {
        const int t = t0 + i * KS;
        const uint16_t* Ks = sg + (i & 1) * G::STAGE_ELEMS;
        const uint16_t* Vs = Ks + G::KS_ELEMS;
        uint16_t* nx = sg + (~i & 1) * G::STAGE_ELEMS;
        if (t + KS < t1) issue_tile<D>(wk.Kbh, wk.Vbh, (t + KS) * BK, L, tid, nx, nx + G::KS_ELEMS);
        else if (MODE == MODE_WINDOW && grp == 0 && i == iters - 1 && p.Rin)
            // the residual rows, into the stage that the last tile leaves free
            issue_rows<bq<1>() * D / 4>(p.Rin + head_off + (size_t)q0 * D, (min(L, q0 + bq<1>()) - q0) * D / 4, tid, nx);
        if (t < t1 && wk.wave_active) {
            if constexpr (MODE == MODE_REFRESH) wk.tile_split(acc, ax, q, Ks, Vs, t * BK);
            else if constexpr (MODE == MODE_WINDOW) wk.tile_window(acc, q, Ks, Vs, t * BK);
            else if (t * BK + BK <= L) wk.template tile<SEG_PLAIN, false>(acc, q, Ks, Vs, t * BK);
            // the ragged last tile (its group's last, in the last iteration) follows the loop
        }
        wait_vm_all();
        __syncthreads();
    }
    if constexpr (MODE == MODE_FULL) {
        const int i = iters - 1, t = t0 + i * KS;
        if (t < t1 && wk.wave_active && t * BK + BK > L) {
            const uint16_t* Ks = sg + (i & 1) * G::STAGE_ELEMS;
            wk.template tile<SEG_KEYS, false>(acc, q, Ks, Ks + G::KS_ELEMS, t * BK);
        }
        __syncthreads();
    }
    uint16_t* states = smem + STATE0 + wave * state_elems<D>();
    if (grp != 0) {
        put_state<D>(acc, states + (grp - 1) * NACC * STATES, lane);
        if constexpr (MODE == MODE_REFRESH) put_state<D>(ax, states + ((grp - 1) * NACC + 1) * STATES, lane);
    }
    __syncthreads();
    if (grp != 0 || !wk.wave_active) return;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k) {
        add_state<D>(acc, states + k * NACC * STATES, lane, p.c);
        if constexpr (MODE == MODE_REFRESH) add_state<D>(ax, states + (k * NACC + 1) * STATES, lane, p.c);
    }
    if constexpr (MODE == MODE_REFRESH) {
        store_split<D, 1, true>(p, acc, ax, head_off, qw0, L, w, smem + STATE0 + (KS - 1) * NACC * STATES + wave * 2 * OUT_ELEMS, lane);
    } else {
        const float inv = 1.f / row_sum<D>(acc, 0, r);
        const float* rl = (const float*)(smem + (iters & 1) * G::STAGE_ELEMS) + (wave * 16 + r) * D;
        u32x2 ob[G::NDB];
#pragma unroll
        for (int mb = 0; mb < G::NDB; ++mb) {
#pragma clang fp contract(off)
            const int col = 16 * mb + 4 * g;
            f32x4 out = acc.o[0][mb] * inv;
            if constexpr (MODE == MODE_WINDOW) {
                if (p.Rin && qw0 + r < L && col < D) out = out + *(const f32x4*)(rl + col);
            }
            ob[mb] = u32x2{pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
        }
        // through the stage of group 0 that holds no residual rows
        store_rows<D>(p, ob, smem + (~iters & 1) * G::STAGE_ELEMS + wave * OUT_ELEMS, head_off + (size_t)qw0 * D, min(16, L - qw0), lane);
    }
}

// Streaming copy of n16 16-byte units (AST output reuse).
__global__ void __launch_bounds__(256) copy16_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, size_t n16) {
    const size_t stride = (size_t)gridDim.x * 256 * 4;
    for (size_t base = (size_t)blockIdx.x * 256 * 4 + threadIdx.x; base < n16; base += stride) {
        u32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t i = base + (size_t)u * 256;
            if (i < n16) v[u] = src[i];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t i = base + (size_t)u * 256;
            if (i < n16) dst[i] = v[u];
        }
    }
}

// One query block per wavefront (64-query workgroups, four wavefronts per
// SIMD) when a workgroup's tile walk is short: the extra workgroups and
// wavefronts hide latency there.  Long walks run faster with two blocks,
// which halve the K/V tile copies per query.  The crossovers, measured at
// d = 72 with interleaved timings: full attention up to L = 256 (4 key tiles),
// window attention up to a band of 1280 keys.  A band that covers every key is
// full attention and takes full attention's choice, so that the two give
// identical results.  A refresh has one block in its one-pass form
// (one_pass_refresh), and up to L = 1024 in two phases.
template <int MODE>
bool one_query_block(const AttnLaunch& a, int B) {
    // A launch whose 128-query workgroups would number at most one per CU
    // (one wavefront per SIMD) takes 64-query workgroups whatever its length:
    // measured 11% faster at (B, H, L) = (1, 16, 2048) and (4, 16, 512).
    if ((long long)B * a.H * ((a.L + bq<2>() - 1) / bq<2>()) <= 256) return true;
    if constexpr (MODE == MODE_REFRESH) return a.L <= 1024;
    if constexpr (MODE == MODE_WINDOW) {
        if (a.w < a.L - 1) return 2LL * a.w + 1 <= 1280;
    }
    return a.L <= 256;
}

// Key groups of a launch of 64-query workgroups (1: attn_kernel).  Two
// workgroups of four wavefronts per CU are two wavefronts per SIMD; below that
// the groups fill the SIMDs.  Combining them costs about 1 us, so a walk of
// fewer than 8 tiles keeps one group (kernel times at 256 workgroups or fewer:
// full attention of 4 tiles 6.8 us in one group, 7.9 in four; of 8 tiles 10.0
// and 9.4; of 64 tiles 49.3 and 31.5; windows of 6 tiles 8.5 and 9.2, of 18
// tiles 18.6 and 15.8; at 512 workgroups full attention of 16 tiles 19.8 us in
// one, 18.9 in two).  A refresh, whose walk also carries two accumulators'
// work, gains from 2 tiles on (4 tiles 10.6 -> 9.2 us, 64 tiles 57.9 -> 44.0);
// its registers allow two groups and no more than 256 workgroups.  The groups
// change the order of a query's sums, so their number is that of the whole
// call's batch also where only its conditional half is launched: the ASC codes
// then give the conditional half of the whole-batch code bit for bit.  Against
// groups by the half's own workgroups, us: refresh half of (2, 16, 1024, 72)
// 15.8 -> 18.9, full half of (2, 16, 2048, 72) 29.5 -> 31.5 (in one group 22.1
// and 35.9).
template <int MODE>
int key_groups(const AttnLaunch& a) {
    if (MODE != MODE_REFRESH && !one_query_block<MODE>(a, a.Bcall)) return 1;
    const long long nblocks = (long long)a.Bcall * a.H * ((a.L + bq<1>() - 1) / bq<1>());
    long long tiles = (a.L + BK - 1) / BK;
    if (MODE == MODE_REFRESH) return nblocks <= 256 && tiles >= 2 ? 2 : 1;
    if (MODE == MODE_WINDOW) {
        const long long band = (2LL * a.w + 2 * BK - 2) / BK + 1;   // of 64 queries, at most
        tiles = band < tiles ? band : tiles;
    }
    if (tiles < 8) return 1;
    return nblocks <= 256 ? 4 : (nblocks <= 512 ? 2 : 1);
}

// Whether a launch's outputs leave as whole lines, through LDS (time direct over
// rows, on two sets of buffers, 2160 launches of 33 to 4096 tokens; in MB of O):
//   - full and window attention with several destinations (a cache, both halves;
//     1.02 to 1.5), but not small windows of 64-query workgroups at d = 72 (two
//     destinations to 2.6 MB 0.98, above 1.01 to 1.15, four to 2 MB 0.98 to 1.00,
//     above 1.05 to 1.3; full attention there 1.00 and 1.01);
//   - with one destination, full attention at d = 64 in 64-query workgroups (1.02
//     to 1.09), and other launches of these that write more O than the caches
//     keep beside its inputs (reuse (64, 16, 405, 72), 60 MB, 1.03; (16, 16, 700,
//     64), 23 MB, 1.02; (8, 16, 1024, 72), 19 MB, 0.98 and 1.01; (8, 16, 256,
//     72), 4.7 MB, 0.97 and 0.98; (2, 16, 128, 72) 0.98).  Long walks of 128-query
//     workgroups gain nothing (reuse (2, 16, 8192, 72) 0.98);
//   - refreshes, whose R passes with them, but at d = 72 for small ones (one
//     or two destinations to 2 MB: 4 heads of 40 tokens 0.93, 128 of 100, 1.8 MB,
//     1.00, 256 of 100, 3.7 MB, 1.04 and 1.08; four to 1 MB 1.00, to 2 MB 1.02 to
//     1.09)
//     and, with split probabilities, one destination to 8 MB (192 heads of 512
//     0.97 and 0.98, 512 of 256, 19 MB, 0.99 and 1.03), two to 3 MB (0.96 to 0.99,
//     above 1.02 to 1.15).  At d = 64 rows win there as well (1.02 to 1.3).
// One kernel with both forms in it was slower than either (9.17 us at (8, 16,
// 256, 72), 9.05 and 9.11) and spilled in full attention at d = 72.
template <int D, int MODE, int QB>
bool store_as_rows(const AttnLaunch& a) {
    const size_t kib = (size_t)a.B * a.H * a.L * a.d * 2 >> 10;   // of O
    if constexpr (MODE == MODE_REFRESH_FINE) return D != 72 || kib > (a.ndst == 1 ? 8192 : a.ndst == 2 ? 3072 : 1024);
    if constexpr (MODE == MODE_REFRESH || MODE == MODE_REFRESH_SPLIT) return D != 72 || kib > (a.ndst == 4 ? 1024 : 2048);
    if (a.ndst > 1) return D != 72 || QB == 2 || MODE == MODE_FULL || MODE == MODE_ASC || kib > (a.ndst == 2 ? 2560 : 2048);
    if constexpr (MODE == MODE_FULL && D == 64 && QB == 1) return true;
    const long long keys = MODE == MODE_FULL || a.w >= a.L ? a.L : 2LL * a.w + 1;
    return QB == 1 && kib > 20 * 1024 && keys <= 400;
}

template <int D, int MODE, int QB>
hipError_t launch_attn(const AttnLaunch& a, hipStream_t stream) {
    using G = Geo<D>;
    Params p{};
    p.Q = (const uint16_t*)a.Q;
    p.K = (const uint16_t*)a.K;
    p.V = (const uint16_t*)a.V;
    p.Rin = (const float*)a.Rin;
    p.Rout = (float*)a.Rout;
    p.ndst = a.ndst;
    p.nout = a.nout;
    for (int i = 0; i < 4; ++i) p.dst[i] = (uint16_t*)(i < a.ndst ? a.dst[i] : nullptr);
    p.H = a.H;
    p.L = a.L;
    p.w = a.w;
    p.n_qt = (a.L + bq<QB>() - 1) / bq<QB>();
    const long long nb = (long long)p.n_qt * a.B * a.H;
    if (nb <= 0 || nb > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    p.nblocks = (int)nb;
    p.c = (float)(1.4426950408889634 / __builtin_sqrt((double)D));
    static_assert((size_t)2 * G::STAGE_ELEMS * sizeof(uint16_t) * waves_per_simd<D, QB, MODE>() <= 160 * 1024,
                  "one workgroup per wave slot of a SIMD must fit in LDS");
    if constexpr (QB == 1 && MODE != MODE_WINDOW_FINE && MODE != MODE_REFRESH_FINE) {
        constexpr int KM = MODE == MODE_REFRESH_SPLIT ? MODE_REFRESH : MODE;
        const int ks = key_groups<KM>(a);
        if constexpr (KM != MODE_REFRESH) {
            if (ks == 4) {
                hipLaunchKernelGGL((attn_keysplit_kernel<D, KM, 4>), dim3(p.nblocks), dim3(4 * NTHREADS), 0, stream, p);
                return hipGetLastError();
            }
        }
        if (ks == 2) {
            hipLaunchKernelGGL((attn_keysplit_kernel<D, KM, 2>), dim3(p.nblocks), dim3(2 * NTHREADS), 0, stream, p);
            return hipGetLastError();
        }
    }
    if constexpr (MODE == MODE_REFRESH && QB == 2) {
        // no registers left for rows at d = 72 (nine spills; 148 -> 152 us at (8,
        // 16, 1500, 72)), and at d = 64 they gained less than 1%
        hipLaunchKernelGGL((attn_kernel<D, MODE, QB, false>), dim3(p.nblocks), dim3(NTHREADS), 0, stream, p);
    } else if (store_as_rows<D, MODE, QB>(a)) {
        hipLaunchKernelGGL((attn_kernel<D, MODE, QB, true>), dim3(p.nblocks), dim3(NTHREADS), 0, stream, p);
    } else {
        hipLaunchKernelGGL((attn_kernel<D, MODE, QB, false>), dim3(p.nblocks), dim3(NTHREADS), 0, stream, p);
    }
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const AttnLaunch& a, hipStream_t stream) {
    const bool one = one_query_block<MODE>(a, a.B);
    switch (a.d) {
        case 64: return one ? launch_attn<64, MODE, 1>(a, stream) : launch_attn<64, MODE, 2>(a, stream);
        case 72: return one ? launch_attn<72, MODE, 1>(a, stream) : launch_attn<72, MODE, 2>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool head_dim_supported(int d) { return d == 64 || d == 72; }

hipError_t launch_full(const AttnLaunch& a, hipStream_t s) { return launch_mode<MODE_FULL>(a, s); }
hipError_t launch_asc(const AttnLaunch& a, hipStream_t s) { return launch_mode<MODE_ASC>(a, s); }
// Whether a refresh takes the one-pass two-accumulator form: where band-edge
// tiles, which the two-phase form visits twice, are a large part of the walk.
// Three things set its limit (times of two phases over one in brackets, B * H *
// ceil(L / 64) = n workgroups of 64 queries; 2766 launches of 513 to 1400 tokens
// were measured in both forms, of which the rule is never more than 5% slower
// than two phases, which took all of them beyond 512 tokens before, and 11%
// faster on average):
//   - rounds.  One pass holds 1024 workgroups at once at d = 64, 768 at d = 72
//     (three wavefronts per SIMD); two phases hold 1024, and beyond 1024 tokens
//     768 of twice the queries, which leaves half a round of n <= 768 idle.
//     d = 72: n = 576 of 1100 tokens (1.4 to 1.54), 769 to 1024 (1.03 to 1.10 with
//     w = L / 8, 0.92 to 0.99 from half the keys on), 1152 of 1024 (1.1 to 1.25),
//     1280 of 1280 (1.06 to 1.19);
//   - the band.  Nearly all keys in it leave two phases little more than full
//     attention's work: d = 72, n = 2880 of 900 tokens, w = 675 (1.04), w = 898
//     (0.98); beyond 1024 tokens from half the keys on, n = 2432 of 1216, w = 405
//     (1.08), w = 608 (1.00), w = 1214 (0.88);
//   - K/V copies per query, which two query blocks per wavefront halve: d = 72
//     beyond 1024 tokens, w = L / 8, n = 1281 to 2560 (1.01 to 1.30), to 5000 (1.01
//     to 1.2), to 10000 (0.96 to 1.04); d = 64 (1.06 to 1.3), (1.07 to 1.26) and
//     (1.04 to 1.14).
// As with the key groups, the whole call's batch decides.
bool one_pass_refresh(const AttnLaunch& a) {
    if (a.L <= 512) return true;
    if (a.L > 1280) return false;
    const long long n = (long long)a.Bcall * a.H * ((a.L + bq<1>() - 1) / bq<1>());
    if (n <= (a.d == 64 ? 1024 : 768)) return true;
    const bool half = 2LL * a.w >= a.L, most = 4LL * a.w > 3LL * a.L;   // of the keys to each side
    if (a.d == 64) return a.L <= 1024 || (a.L <= 1216 ? !most : !half);
    if (n <= 1024) return 8LL * a.w <= 3LL * a.L;
    if (n <= 1280) return true;
    if (a.L > 1024) return n <= 5000 && !half;
    return a.L <= 768 || !most;
}

// Bands of at most 31 keys take the two-phase form with split probabilities
// in its in-band phase (64-query workgroups), so that W, and with it R and
// every reuse that adds R, carries no unaveraged bf16 rounding of its weights.
hipError_t launch_refresh(const AttnLaunch& a, hipStream_t s) {
    if (a.w <= FINE_MAX_HALF_WIDTH && a.w < a.L - 1) {
        switch (a.d) {
            case 64: return launch_attn<64, MODE_REFRESH_FINE, 1>(a, s);
            case 72: return launch_attn<72, MODE_REFRESH_FINE, 1>(a, s);
            default: return hipErrorInvalidValue;
        }
    }
    if (!one_pass_refresh(a)) return launch_mode<MODE_REFRESH>(a, s);
    switch (a.d) {
        case 64: return launch_attn<64, MODE_REFRESH_SPLIT, 1>(a, s);
        case 72: return launch_attn<72, MODE_REFRESH_SPLIT, 1>(a, s);
        default: return hipErrorInvalidValue;
    }
}
// Narrow bands (at most 31 keys per query) apply each probability as a bf16
// value plus its bf16 rounding residual: with so few keys per row the bf16
// rounding of the weights does not average out, and alone it costs up to
// 2^-8 max|v - o| per output.  Such bands always take 64-query workgroups.
// A band covering every key keeps full attention's choice.
hipError_t launch_window(const AttnLaunch& a, hipStream_t s) {
    if (a.w <= FINE_MAX_HALF_WIDTH && a.w < a.L - 1) {
        switch (a.d) {
            case 64: return launch_attn<64, MODE_WINDOW_FINE, 1>(a, s);
            case 72: return launch_attn<72, MODE_WINDOW_FINE, 1>(a, s);
            default: return hipErrorInvalidValue;
        }
    }
    return launch_mode<MODE_WINDOW>(a, s);
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t stream) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 1023) / 1024;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(copy16_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const u32x4*)src, (u32x4*)dst, n16);
    return hipGetLastError();
}

}  // namespace dfa
