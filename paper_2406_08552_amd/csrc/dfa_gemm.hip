// Projections of the attention module for gfx950 (CDNA4): the fused QKV
// projection in front of the attention path and the output projection behind
// it (the module whose FLOPs Table 2 counts).
//
// Both are D = W Act^T with bf16 operands and fp32 accumulation:
//   W    [N][K]  weights, [out_features][in_features] (y = x W^T + b)
//   Act  token-major activations, K contiguous per token: X [M][K] for the
//        QKV projection, or the attention output O [B][H][L][d] read as the
//        [M][H * d] matrix of merged heads for the output projection
//   D    [N][M]  one output feature per row, one token per column
// The QKV projection's epilogue scatters chunks of eight features straight
// into Q, K or V in the [B][H][L][d] layout of the attention kernels (feature
// f = which * C + head * d + dim, and d is a multiple of 8, so a chunk never
// straddles a head); the output projection stores token-major Y [M][N] to
// every destination given (the unconditional half of an ASC step is one of
// them).
//
// Work decomposition.  Each wavefront owns MB x NB blocks of
// v_mfma_f32_32x32x16_bf16 (operand layouts: lane l, h = l / 32, A element
// e = A[l % 32][8h + e], B element e = B[8h + e][l % 32], output element
// i = D[8 (i/4) + 4h + i%4][l % 32]) and walks K in k-tiles of 64, one 128-byte
// line of every operand row: k-tiles of 32 made the caches move each line
// twice and cost 5-25%.  The k-tiles arrive by direct global -> LDS copies.
// Every shape sums over k in the same order, so all give identical results.
//   gemm_stream_kernel  large grids.  Persistent workgroups, two LDS stages,
//     one barrier per k-tile, operands read one MFMA group ahead.  The ring of
//     k-tiles runs on from one tile to the next: the next tile's first copies
//     are in flight while this one's output leaves, and its stores drain under
//     the next tile's MFMAs.
//   gemm_ring_kernel  grids of at most a workgroup per CU, where only depth
//     hides the copies' latency: four stages, one tile per workgroup.
//
// What bounds it, at 32768 tokens x 1152 features (PixArt-Sigma at 2048 px):
// in a steady stream of launches the chip's power limit (the shader clock
// falls with N(0, 1) data, where zeros, same instructions, keep it), then the
// output stores and the copies' latency at each k-tile's barrier; LDS bank
// conflicts take 1% of the cycles.  Measured there, against the
// kernels this replaced (whose partial vmcnt wait the barrier's own fence
// undid, and whose epilogue waited for each of its 32 bias loads in turn):
// QKV projection 337 -> 277 us, output projection 133 -> 108 us; at 2048
// tokens 26.2 -> 20.3 and 18.3 -> 13.0 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfa_internal.h"

namespace dfa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int GK = 64;                           // k per LDS stage: rows of eight 16-byte chunks, one cache line

// Workgroup tile: WF x WT wavefronts, each owning MB x NB blocks of 32 features
// x 32 tokens, fed through a ring of NST LDS stages.
template <int MB_, int NB_, int WF_, int WT_, int WGS_, int NST_ = 2>
struct Tile {
    static constexpr int MB = MB_, NB = NB_, WF = WF_, WT = WT_, NST = NST_;
    static constexpr int WGS = WGS_;                      // workgroups per CU
    static constexpr int NW = WF * WT, NT = 64 * NW;      // wavefronts, threads
    static constexpr int TF = 32 * MB * WF, TT = 32 * NB * WT;
    static constexpr int STAGE = (TF + TT) * GK;          // elements: feature rows, then token rows
    static constexpr int CPW = (TF + TT) / 8 / NW;        // 8-row copies per wavefront and k-tile,
    static constexpr int CPF = TF / 8 / NW;               // the first CPF of them feature rows
    static constexpr int SCRATCH = 32 * 32;               // scratch of a wavefront: one 32 x 32 block of output, or its biases
    static constexpr int STORES = 2 * MB * NB;            // stores of a wavefront's output, one destination
    static_assert(TF % (8 * NW) == 0 && TT % (8 * NW) == 0 && NW % 2 == 0, "copies per wavefront");
    static_assert(8 * MB <= 64 && 64 * MB <= SCRATCH, "biases of a wavefront");
    static_assert((size_t)(NST * STAGE + NW * SCRATCH) * 2 * WGS <= 160 * 1024, "LDS");
    static_assert(CPW * NST < 64, "vmcnt immediate");
};

// s_waitcnt immediate: at most vm vector memory operations outstanding, and
// (lds0) no LDS or scalar ones.
constexpr int waitcnt(int vm, bool lds0) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lds0 ? 0 : 0xF00); }

// Element offset of 16-byte chunk ch of row row of a stage: chunk ch sits at
// ch ^ ((row >> 1) & 7).  Two rows span the 64 banks, so 16 consecutive rows
// have their copies of one chunk on 16 distinct groups of four banks, and the
// operand reads (one chunk of 32 consecutive rows per half-wavefront) are free
// of conflicts; the copies fill whole rows.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int chunk_off(int row, int ch) { return row * GK + ((ch ^ swz(row)) << 3); }

enum { ACT_ROWS = 0, ACT_HEADS = 1 };   // activations: [M][K] rows, or O [B][H][L][d]
enum { OUT_QKV = 0, OUT_ROWS = 1 };     // epilogue: scatter to Q/K/V, or [M][N] rows

struct GemmParams {
    const uint16_t* W;
    const uint16_t* act;
    const float* bias;       // [N] or null
    uint16_t* dst[4];        // OUT_QKV: Q, K, V; OUT_ROWS: copies of Y
    int ndst;
    int M, N, K;             // tokens, output features, input features
    int L, H, d;             // token t = b * L + l; head geometry of Q/K/V/O
    int nft, ntt;            // feature and token tiles
    uint32_t lmul, lshift, dmul, dshift;   // division by L and by d (fast_div)
    int group;               // token tiles per group of the block order (1: all feature tiles of a token tile in turn)
    int nblocks;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}

// v_permlane32_swap exchanges the upper half of a with the lower half of b.
// The leading s_nop covers the VALU-write -> permlane-read hazard.
__device__ __forceinline__ void xchg32(uint32_t& a, uint32_t& b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

// n / v for 0 <= n < 2^30: with s = ceil(log2 v) and m = ceil(2^(30 + s) / v),
// m v - 2^(30 + s) < v <= 2^s, so n m >> (30 + s) is exact, and m <= 2^31.
__device__ __forceinline__ int fast_div(int n, uint32_t mul, uint32_t shift) { return (int)((uint64_t)n * mul >> shift); }

// The copies of one wavefront: copy i fills the eight rows from
// 8 (wave + i NW) of a stage, lane l the 16-byte slot l of them, with the
// chunk that the swizzle places there: every row is one whole 128-byte line
// of its operand.  Rows of one copy are all features or all tokens.
template <int ACT, class T>
struct Copier {
    uint32_t off[T::CPW];        // byte offset of the lane's chunk from its operand's uniform base
    const char* wbase;           // the uniform bases: W's first feature row of the tile, at the next k-tile,
    const char* abase;           // and (ACT_ROWS) the first token row
    const char* ptr[ACT == ACT_HEADS ? T::CPW - T::CPF : 1];   // ACT_HEADS token rows: the lane's address
    int j;                       // ACT_HEADS: dim of the lane's chunk within its head
    int wave, lrow, ch;

    __device__ __forceinline__ void init(int wave_, int lane) {
        wave = wave_;
        lrow = lane >> 3;
        // a lane's rows differ by multiples of 16 (NW is even), so they share the swizzle
        ch = (lane & 7) ^ swz(8 * wave + lrow);
    }
    // start of the tile at (n0, t0)
    __device__ __forceinline__ void start(const GemmParams& p, int n0, int t0) {
        asm volatile("" : "+v"(lrow), "+v"(ch));
        wbase = (const char*)(p.W + (size_t)n0 * p.K);
        abase = ACT == ACT_ROWS ? (const char*)(p.act + (size_t)t0 * p.K) : nullptr;
        j = 8 * ch;                                     // < d: d is at least 64
#pragma unroll
        for (int i = 0; i < T::CPW; ++i) {
            // rows beyond the last feature or token copy the last one (their outputs are not stored)
            if (i < T::CPF) {
                const int row = (wave + i * T::NW) * 8 + lrow;
                off[i] = (uint32_t)min(row, p.N - 1 - n0) * (uint32_t)(2 * p.K) + 16u * ch;
            } else {
                const int tr = min((wave + i * T::NW) * 8 + lrow - T::TF, p.M - 1 - t0);
                if constexpr (ACT == ACT_ROWS) {
                    off[i] = (uint32_t)tr * (uint32_t)(2 * p.K) + 16u * ch;
                } else {
                    const int t = t0 + tr, b = fast_div(t, p.lmul, p.lshift);
                    // token l = t - b L of head 0: row b H L + l
                    ptr[i - T::CPF] = (const char*)(p.act + ((size_t)t + (size_t)b * (p.H - 1) * p.L) * p.d + j);
                    off[i] = 0;
                }
            }
        }
    }

    // no further tile: every lane copies its chunk of the operands' first row
    __device__ __forceinline__ void park(const GemmParams& p) {
        wbase = (const char*)p.W;
        abase = (const char*)p.act;
#pragma unroll
        for (int i = 0; i < T::CPW; ++i) off[i] = 16u * ch;
        if constexpr (ACT == ACT_HEADS) {
            j = 8 * ch;
#pragma unroll
            for (int i = 0; i < T::CPW - T::CPF; ++i) ptr[i] = (const char*)p.act + 16 * ch;
        }
    }

    // issue the copies of the current k-tile into stage st and (advance) step to the next
    __device__ __forceinline__ void issue(const GemmParams& p, uint16_t* st, bool advance = true) {
        // opaque to the compiler, which would otherwise carry a 64-bit address
        // and an LDS address per copy in vector registers
        asm volatile("" : "+s"(wbase), "+s"(abase), "+s"(wave));
#pragma unroll
        for (int i = 0; i < T::CPW; ++i) asm volatile("" : "+v"(off[i]));
#pragma unroll
        for (int i = 0; i < T::CPW; ++i) {
            __attribute__((address_space(3))) void* to =
                (__attribute__((address_space(3))) void*)(st + (wave + i * T::NW) * 8 * GK);
            if (i < T::CPF)
                __builtin_amdgcn_global_load_lds((const void*)(wbase + off[i]), to, 16, 0, 0);
            else if constexpr (ACT == ACT_ROWS)
                __builtin_amdgcn_global_load_lds((const void*)(abase + off[i]), to, 16, 0, 0);
            else
                __builtin_amdgcn_global_load_lds((const void*)ptr[i - T::CPF], to, 16, 0, 0);
        }
        wbase += advance ? 2 * GK : 0;
        if constexpr (ACT == ACT_ROWS) {
            abase += advance ? 2 * GK : 0;
        } else {
            // the lane's chunk of the next k-tile, 64 features on, at most one head further (d >= 64)
            const bool w = j + GK >= p.d;
            const long long step = advance ? 2 * GK + (w ? 2LL * ((long long)p.L * p.d - p.d) : 0) : 0;
            j += advance ? GK - (w ? p.d : 0) : 0;
#pragma unroll
            for (int i = 0; i < T::CPW - T::CPF; ++i) ptr[i] += step;
        }
    }
};

template <int N_, bool AHEAD_ = true>
struct Left {
    static constexpr int N = N_;
    static constexpr bool AHEAD = AHEAD_;
};

template <class T>
struct Frag {
    bf16x8 a[T::MB], b[T::NB];
    // operands of the 16 k-values ks of a stage; ao and bo: element offsets of
    // the lane's chunks for ks = 0 (rows that differ by multiples of 32 share
    // the swizzle).  One offset from the stage per read: longer address chains
    // lose the compiler's knowledge of which stage is read.
    __device__ __forceinline__ void read(const uint16_t* st, int ks, int ao, int bo) {
#pragma unroll
        for (int mb = 0; mb < T::MB; ++mb)
            a[mb] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((ao ^ (16 * ks)) + 32 * mb * GK)));
#pragma unroll
        for (int nb = 0; nb < T::NB; ++nb)
            b[nb] = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + ((bo ^ (16 * ks)) + 32 * nb * GK)));
    }
};

// MFMAs [I0, I1) of the wavefront's MB x NB blocks.
template <class T, int I0, int I1>
__device__ __forceinline__ void mma(f32x16 (&acc)[T::MB][T::NB], const Frag<T>& f) {
#pragma unroll
    for (int i = I0; i < I1; ++i) {
        const int mb = i / T::NB, nb = i % T::NB;
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[mb], f.b[nb], acc[mb][nb], 0, 0, 0);
    }
}

// The accumulators start from the bias: output element i of a block is feature
// 8 (i / 4) + 4 h + i % 4 of its 32 (h = lane / 32), token lane % 32.  bv: four
// of the wavefront's biases per lane, handed round through its scratch.
template <class T>
__device__ __forceinline__ void init_acc(f32x16 (&acc)[T::MB][T::NB], uint16_t* scratch, f32x4 bv, int lane) {
    if (lane < 8 * T::MB) *(f32x4*)(scratch + 8 * lane) = bv;
    __builtin_amdgcn_wave_barrier();   // the wavefront's LDS accesses complete in order
#pragma unroll
    for (int mb = 0; mb < T::MB; ++mb)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            const f32x4 b = *(const f32x4*)(scratch + 2 * (32 * mb + 8 * jb + 4 * (lane >> 5)));
#pragma unroll
            for (int nb = 0; nb < T::NB; ++nb)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[mb][nb][4 * jb + i] = b[i];
            if (jb == 3) __builtin_amdgcn_sched_barrier(0);   // few biases in registers at a time
        }
}

// Output of one wavefront: its blocks of 32 features x 32 tokens, rounded to
// bf16, pass one by one through the wavefront's scratch as [token][feature]
// rows (chunk c of row t at c ^ ((t >> 2) & 3)), so that they leave as 16-byte
// chunks in row order.  A lane holds four consecutive features of a token and
// lane + 32 the next four: one exchange gives each lane a whole chunk.
template <int OUT, class T, bool WHOLE>
__device__ __forceinline__ void store_tile(const GemmParams& p, f32x16 (&acc)[T::MB][T::NB], uint16_t* scratch, int nw0,
                                           int tw0, int lane) {
    // opaque: nothing of the epilogue's addressing is to be kept in registers
    // through the next tile's k loop
    asm volatile("" : "+v"(lane));
    const int r32 = lane & 31, h = lane >> 5, srow = lane >> 2, sc = lane & 3;
    const int C = p.K;                                                    // OUT_QKV: N = 3 K
    const uint16_t* from = scratch + srow * 32 + ((sc ^ (srow >> 2)) << 3);   // and row srow + 16: same swizzle
    size_t trow[T::NB][2];
#pragma unroll
    for (int nb = 0; nb < T::NB; ++nb)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int t = tw0 + 32 * nb + 16 * i + srow;
            // OUT_QKV: (b H + head) L + l rows of d, with l = t - b L
            if constexpr (OUT == OUT_QKV)
                trow[nb][i] = ((size_t)t + (size_t)fast_div(min(t, p.M - 1), p.lmul, p.lshift) * (p.H - 1) * p.L) * p.d;
            else
                trow[nb][i] = (size_t)t * p.N;
        }
#pragma unroll
    for (int mb = 0; mb < T::MB; ++mb) {
        const int f = nw0 + 32 * mb + 8 * sc;
        uint16_t* out;
        if constexpr (OUT == OUT_QKV) {
            const int which = f >= 2 * C ? 2 : (f >= C ? 1 : 0), fr = f - which * C;
            const int head = fast_div(fr, p.dmul, p.dshift);
            out = (which == 2 ? p.dst[2] : (which == 1 ? p.dst[1] : p.dst[0])) + (size_t)head * (p.L - 1) * p.d + fr;
        } else {
            out = p.dst[0] + f;
        }
#pragma unroll
        for (int nb = 0; nb < T::NB; ++nb) {
            const f32x16& a = acc[mb][nb];
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) {
                uint32_t x0 = pack_bf16x2(a[8 * jp], a[8 * jp + 1]), x1 = pack_bf16x2(a[8 * jp + 2], a[8 * jp + 3]);
                uint32_t y0 = pack_bf16x2(a[8 * jp + 4], a[8 * jp + 5]), y1 = pack_bf16x2(a[8 * jp + 6], a[8 * jp + 7]);
                xchg32(x0, y0);
                xchg32(x1, y1);
                *(u32x4*)(scratch + r32 * 32 + (((2 * jp + h) ^ ((r32 >> 2) & 3)) << 3)) = u32x4{x0, x1, y0, y1};
            }
            __builtin_amdgcn_wave_barrier();   // the wavefront's LDS accesses complete in order
            u32x4 val[2] = {*(const u32x4*)from, *(const u32x4*)(from + 16 * 32)};
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int t = tw0 + 32 * nb + 16 * i + srow;
                if (!WHOLE && (t >= p.M || f >= p.N)) continue;
                *(u32x4*)(out + trow[nb][i]) = val[i];
                if constexpr (OUT == OUT_ROWS)
                    for (int di = 1; di < p.ndst; ++di) *(u32x4*)(p.dst[di] + f + trow[nb][i]) = val[i];
            }
        }
    }
}

// First feature and token of tile b: groups of p.group token tiles, each
// group's tiles feature tile by feature tile (a bijection; the last group may
// be short).
template <class T>
__device__ __forceinline__ void tile_origin(const GemmParams& p, int b, int& n0, int& t0) {
    const int grp = b / (p.group * p.nft), r = b - grp * (p.group * p.nft);
    const int gc = min(p.group, p.ntt - grp * p.group);
    n0 = r / gc * T::TF;
    t0 = (grp * p.group + r % gc) * T::TT;
}

template <int ACT, int OUT, class T>
__global__ void __launch_bounds__(T::NT) __attribute__((amdgpu_waves_per_eu(T::WGS * T::NW / 4, T::WGS * T::NW / 4)))
gemm_stream_kernel(GemmParams p) {
    constexpr int MB = T::MB, NB = T::NB;
    // one array per stage: the compiler then knows that the copies into one
    // stage do not touch the stage being read, and adds no wait of its own
    __shared__ __attribute__((aligned(16))) uint16_t s0[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t s1[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t scratch[T::NW * T::SCRATCH];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave % T::WF, wt = wave / T::WF;    // the wavefront's feature and token part
    const int r32 = lane & 31, h = lane >> 5;

    // Each XCD (workgroups are dealt to the eight of them in turn) takes a
    // contiguous range of tiles; its workgroups walk them side by side.
    const int x = blockIdx.x & 7, q = p.nblocks >> 3, rem = p.nblocks & 7;
    const int end = (x + 1) * q + min(x + 1, rem);
    const int stride = ((int)gridDim.x + 7 - x) >> 3;
    int blk = x * q + min(x, rem) + ((int)blockIdx.x >> 3);
    if (blk >= end) return;
    int n0, t0;
    tile_origin<T>(p, blk, n0, t0);

    Copier<ACT, T> cp;
    cp.init(wave, lane);
    const int nk = p.K / GK;                           // even
    // the biases of the wavefront's features, four to a lane
    f32x4 bv{0.f, 0.f, 0.f, 0.f};
    auto load_bias = [&](int n) {
        if (p.bias && lane < 8 * MB) bv = *(const f32x4*)(p.bias + min(n + 32 * MB * wf + 4 * lane, p.N - 4));
    };
    uint16_t* sw = scratch + wave * T::SCRATCH;
    cp.start(p, n0, t0);
    load_bias(n0);
    cp.issue(p, s0);
    cp.issue(p, s1);

    f32x16 acc[MB][NB];
    Frag<T> f0, f1;
    int ao = chunk_off(32 * MB * wf + r32, h), bo = chunk_off(T::TF + 32 * NB * wt + r32, h);
    auto fence = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // A k-tile from stage cur, whose first operands f0 holds; nxt holds the
    // k-tile behind it.  The k-tile's one barrier comes when this wavefront has
    // read the last operands of cur and its copies into nxt have landed (all
    // but the LEFT newest vector memory operations done): behind it, `then`
    // issues the copies that overwrite cur, and (AHEAD) the next k-tile's first
    // operands are read before the last MFMAs of this one.
    auto step = [&](auto left, const uint16_t* cur, const uint16_t* nxt, auto then) {
        // the next operands are read behind the first MFMAs of the current
        // ones: LDS reads and the copies share a counter that the compiler can
        // only wait out whole, so reads issued earlier would be waited for too
        constexpr int N = MB * NB, N0 = N > 2 ? 2 : 1;
        asm volatile("" : "+v"(ao), "+v"(bo));   // opaque: the reads' offsets are formed anew, not kept in registers
        mma<T, 0, N0>(acc, f0);
        __builtin_amdgcn_sched_barrier(0);
        f1.read(cur, 1, ao, bo);
        __builtin_amdgcn_sched_barrier(0);
        mma<T, N0, N>(acc, f0);
        mma<T, 0, N0>(acc, f1);
        __builtin_amdgcn_sched_barrier(0);
        f0.read(cur, 2, ao, bo);
        __builtin_amdgcn_sched_barrier(0);
        mma<T, N0, N>(acc, f1);
        mma<T, 0, N0>(acc, f0);
        __builtin_amdgcn_sched_barrier(0);
        f1.read(cur, 3, ao, bo);
        __builtin_amdgcn_sched_barrier(0);
        mma<T, N0, N>(acc, f0);
        fence();
        // not __syncthreads(): its fence would wait for every copy and store
        __builtin_amdgcn_s_waitcnt(waitcnt(decltype(left)::N, true));
        __builtin_amdgcn_s_barrier();
        fence();
        mma<T, 0, N0>(acc, f1);
        __builtin_amdgcn_sched_barrier(0);
        then();
        if constexpr (decltype(left)::AHEAD) f0.read(nxt, 0, ao, bo);
        __builtin_amdgcn_sched_barrier(0);
        mma<T, N0, N>(acc, f1);
        __builtin_amdgcn_sched_barrier(0);
    };
    // k-tiles 0 and 1 have landed
    fence();
    __builtin_amdgcn_s_waitcnt(waitcnt(0, true));
    __builtin_amdgcn_s_barrier();
    fence();
    f0.read(s0, 0, ao, bo);
    while (true) {
        init_acc<T>(acc, sw, bv, lane);
        auto more0 = [&] { cp.issue(p, s0); };
        auto more1 = [&] { cp.issue(p, s1); };
        if (nk > 2) {
            // the T::STORES newest operations in flight may be stores of the
            // previous tile, issued behind this tile's first two k-tiles of
            // copies (if it had fewer, everything has been waited for)
            step(Left<T::STORES>{}, s0, s1, more0);
            step(Left<0>{}, s1, s0, more1);
        }
        for (int kt = 4; kt < nk; kt += 2) {
            step(Left<0>{}, s0, s1, more0);
            step(Left<0>{}, s1, s0, more1);
        }
        const int nw0 = n0 + 32 * MB * wf, tw0 = t0 + 32 * NB * wt;
        const bool whole = n0 + T::TF <= p.N && t0 + T::TT <= p.M;
        // The tile's last two k-tiles, followed by the next tile's first two.
        // Behind the last tile the copies are issued all the same, of one
        // cached row: conditional ones make the compiler wait for all copies
        // at points where it cannot tell which are in flight.
        blk += stride;
        const bool more = blk < end;
        if (more) {
            tile_origin<T>(p, blk, n0, t0);
            cp.start(p, n0, t0);
        } else {
            cp.park(p);
        }
        step(Left<0>{}, s0, s1, [&] {
            load_bias(n0);
            cp.issue(p, s0);
        });
        step(Left<0, false>{}, s1, s0, [&] { cp.issue(p, s1); });
        fence();
        if (whole) {
            store_tile<OUT, T, true>(p, acc, sw, nw0, tw0, lane);   // at least T::STORES stores
        } else {
            store_tile<OUT, T, false>(p, acc, sw, nw0, tw0, lane);
            __builtin_amdgcn_s_waitcnt(waitcnt(0, true));
        }
        fence();
        if (!more) break;
        f0.read(s0, 0, ao, bo);
    }
    // no copy may land after this workgroup's LDS is given to another
    __builtin_amdgcn_s_waitcnt(waitcnt(0, true));
}

// One tile per workgroup, through a ring of four stages: for grids of about one
// workgroup per CU or fewer, where nothing else hides the copies' latency.
template <int ACT, int OUT, class T>
__global__ void __launch_bounds__(T::NT) __attribute__((amdgpu_waves_per_eu(T::WGS * T::NW / 4, T::WGS * T::NW / 4)))
gemm_ring_kernel(GemmParams p) {
    static_assert(T::NST == 4, "stages");
    __shared__ __attribute__((aligned(16))) uint16_t s0[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t s1[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t s2[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t s3[T::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t scratch[T::NW * T::SCRATCH];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave % T::WF, wt = wave / T::WF;
    const int r32 = lane & 31, h = lane >> 5;
    const int x = blockIdx.x & 7, q = p.nblocks >> 3, rem = p.nblocks & 7;
    int n0, t0;
    tile_origin<T>(p, x * q + min(x, rem) + ((int)blockIdx.x >> 3), n0, t0);

    Copier<ACT, T> cp;
    cp.init(wave, lane);
    const int nk = p.K / GK;                           // even
    f32x4 bv[T::MB][4];
#pragma unroll
    for (int mb = 0; mb < T::MB; ++mb)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) bv[mb][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p.bias) {
#pragma unroll
        for (int mb = 0; mb < T::MB; ++mb)
#pragma unroll
            for (int jb = 0; jb < 4; ++jb)
                bv[mb][jb] = *(const f32x4*)(p.bias + min(n0 + 32 * (T::MB * wf + mb) + 8 * jb + 4 * h, p.N - 4));
    }
    cp.start(p, n0, t0);
    // every k-tile issues the same number of copies: behind the last one its
    // own again, which nothing reads (nk is at least 2)
    cp.issue(p, s0);
    cp.issue(p, s1, nk > 2);
    cp.issue(p, s2, nk > 3);
    cp.issue(p, s3, nk > 4);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt(4 * T::CPW, false));   // the biases
    f32x16 acc[T::MB][T::NB];
#pragma unroll
    for (int mb = 0; mb < T::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < T::NB; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][nb][i] = bv[mb][i / 4][i % 4];
    Frag<T> f[4], g[4];
    int ao = chunk_off(32 * T::MB * wf + r32, h), bo = chunk_off(T::TF + 32 * T::NB * wt + r32, h);
    auto fence = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // k-tile kt, whose operands cf holds, from stage cur: at the barrier every
    // wavefront has read them, and k-tile kt + 1 has landed in nxt
    auto step = [&](int kt, Frag<T>(&cf)[4], Frag<T>(&nf)[4], uint16_t* cur, const uint16_t* nxt) {
        asm volatile("" : "+v"(ao), "+v"(bo));
        fence();
        __builtin_amdgcn_s_waitcnt(waitcnt(2 * T::CPW, true));
        __builtin_amdgcn_s_barrier();
        fence();
        cp.issue(p, cur, kt + 5 < nk);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) nf[ks].read(nxt, ks, ao, bo);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) mma<T, 0, T::MB * T::NB>(acc, cf[ks]);
        __builtin_amdgcn_sched_barrier(0);
    };
    fence();
    __builtin_amdgcn_s_waitcnt(waitcnt(3 * T::CPW, true));
    __builtin_amdgcn_s_barrier();
    fence();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f[ks].read(s0, ks, ao, bo);
    int kt = 0;
    for (; kt + 4 <= nk; kt += 4) {
        step(kt, f, g, s0, s1);
        step(kt + 1, g, f, s1, s2);
        step(kt + 2, f, g, s2, s3);
        step(kt + 3, g, f, s3, s0);
    }
    if (kt < nk) {
        step(kt, f, g, s0, s1);
        step(kt + 1, g, f, s1, s2);
    }
    uint16_t* sw = scratch + wave * T::SCRATCH;
    const int nw0 = n0 + 32 * T::MB * wf, tw0 = t0 + 32 * T::NB * wt;
    if (n0 + T::TF <= p.N && t0 + T::TT <= p.M) store_tile<OUT, T, true>(p, acc, sw, nw0, tw0, lane);
    else store_tile<OUT, T, false>(p, acc, sw, nw0, tw0, lane);
    // no copy may land after this workgroup's LDS is given to another
    __builtin_amdgcn_s_waitcnt(waitcnt(0, true));
}

void fast_divisor(int v, uint32_t& mul, uint32_t& shift) {
    int s = 0;
    while ((1LL << s) < v) ++s;
    shift = (uint32_t)(30 + s);
    mul = (uint32_t)(((1ULL << (30 + s)) + v - 1) / v);
}

template <int ACT, int OUT, class T>
hipError_t launch_shape(GemmParams& p, hipStream_t stream) {
    p.nft = (p.N + T::TF - 1) / T::TF;
    const long long ntt = ((long long)p.M + T::TT - 1) / T::TT, nb = ntt * p.nft;
    if (nb <= 0 || nb > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    p.ntt = (int)ntt;
    p.nblocks = (int)nb;
    fast_divisor(p.L, p.lmul, p.lshift);
    fast_divisor(p.d, p.dmul, p.dshift);
    if constexpr (T::NST > 2) {
        hipLaunchKernelGGL((gemm_ring_kernel<ACT, OUT, T>), dim3(p.nblocks), dim3(T::NT), 0, stream, p);
        return hipGetLastError();
    }
    const int grid = (int)(nb < 256 * T::WGS ? nb : 256 * T::WGS);
    hipLaunchKernelGGL((gemm_stream_kernel<ACT, OUT, T>), dim3(grid), dim3(T::NT), 0, stream, p);
    return hipGetLastError();
}

// Tile shapes, features x tokens, and the rule between them (all measured at
// 16 heads x 72 and other widths from 384 to 2304 features, times in us):
//   64 x 64, ring      while one such tile per CU covers the output (600 tokens
//                      x 1152 features 7.3 against 12.6 for the next shape;
//                      at 528 tiles 18.6 against 15.6)
//   128 x 128, ring    the same (2048 tokens x 1152: 13.0 against 16.4 for the
//                      next; at 288 tiles 25.6 against 18.6)
//   128 x 128, stream  two workgroups per CU, or
//   192 x 256, stream  one: by the rounds that each needs.  A round of the
//                      larger tile takes 1.25 of the smaller's (24 against 19
//                      at K = 1152) for 1.5 of its output; a last round of the
//                      smaller with one workgroup on a CU takes 0.65.
// Block order: a weight that fits one XCD's 4 MB L2 stays there while an XCD
// walks all feature tiles of one token tile after another.  A larger one (the
// QKV projection's 7.6 MB at C = 1152) would be fetched again for every token
// tile, so the tiles go in groups of 8 token tiles, feature tile by feature
// tile: an XCD's resident workgroups then share both operands' tiles.
using Tile64 = Tile<1, 1, 2, 2, 2, 4>;
using Tile128Ring = Tile<2, 1, 2, 4, 1, 4>;
using Tile128 = Tile<2, 2, 2, 2, 2>;
using Tile192 = Tile<3, 2, 2, 4, 1>;

template <class T>
long long tiles(const GemmParams& p) {
    return (long long)((p.N + T::TF - 1) / T::TF) * (((long long)p.M + T::TT - 1) / T::TT);
}

template <int ACT, int OUT>
hipError_t launch_gemm(GemmParams& p, hipStream_t stream) {
    p.group = (long long)p.N * p.K * 2 > (4LL << 20) ? 8 : 1;
    if (tiles<Tile64>(p) <= 256) return launch_shape<ACT, OUT, Tile64>(p, stream);
    const long long n128 = tiles<Tile128>(p), n192 = tiles<Tile192>(p);
    if (n128 <= 256) return launch_shape<ACT, OUT, Tile128Ring>(p, stream);
    const long long last = n128 % 512;
    const long long rounds128 = 100 * (n128 / 512) + (last == 0 ? 0 : (last <= 256 ? 65 : 100));
    const long long rounds192 = 125 * ((n192 + 255) / 256);
    if (rounds192 < rounds128) return launch_shape<ACT, OUT, Tile192>(p, stream);
    return launch_shape<ACT, OUT, Tile128>(p, stream);
}

}  // namespace

bool proj_shape_supported(int H, int d) { return H > 0 && (d == 64 || d == 72) && (H * d) % 128 == 0; }

hipError_t launch_qkv_proj(const ProjLaunch& a, hipStream_t stream) {
    GemmParams p{};
    p.W = (const uint16_t*)a.W;
    p.act = (const uint16_t*)a.act;
    p.bias = (const float*)a.bias;
    for (int i = 0; i < 3; ++i) p.dst[i] = (uint16_t*)a.dst[i];
    p.ndst = 3;
    p.L = a.L;
    p.H = a.H;
    p.d = a.d;
    p.M = a.B * a.L;
    p.K = a.H * a.d;
    p.N = 3 * p.K;
    return launch_gemm<ACT_ROWS, OUT_QKV>(p, stream);
}

hipError_t launch_out_proj(const ProjLaunch& a, hipStream_t stream) {
    GemmParams p{};
    p.W = (const uint16_t*)a.W;
    p.act = (const uint16_t*)a.act;
    p.bias = (const float*)a.bias;
    p.ndst = a.ndst;
    for (int i = 0; i < 4; ++i) p.dst[i] = (uint16_t*)(i < a.ndst ? a.dst[i] : nullptr);
    p.L = a.L;
    p.H = a.H;
    p.d = a.d;
    p.M = a.B * a.L;
    p.K = a.H * a.d;
    p.N = p.K;
    return launch_gemm<ACT_HEADS, OUT_ROWS>(p, stream);
}

}  // namespace dfa
