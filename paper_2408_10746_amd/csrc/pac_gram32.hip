// Gram-matrix formulation of the cached Parallel-Adapter step for an fp32 cache (the equations at the head of
// pac_gram.hip), in fp32: matrix instructions and everything kept between the launches.
//
// The layer-by-layer kernels read and write a d-wide side state and its gradient per layer, four dependent launches a layer,
// each a contraction too small to fill the chip (12 layers of 768 x 96, 4096 token rows: 53 launches, 1000 us).  Here no
// d-wide per-token array but the cache exists, and a step is six launches:
//   k_f_proj    U_l = b_l W_down^l of every layer, Q_kl = W_up^k W_down^l, chat, V, mean b_L, the row table
//   k_f_chain   forward: 16 token rows per workgroup walk all layers (h in LDS), the tile's share of the logits
//   k_f_chain   backward: logits, loss, dz; the same walk from the top for dpre
//   k_f_tok     E_l = b_l^T dpre_l, G_kl = h_k^T dpre_l, column sums      (+ k_f_sum where the tokens are split)
//   k_f_post    dW_down, dW_up, dW_cls and the vector gradients
//   k_adamw
//
// Errors: what is computed once and used for every token (Q, V) or summed over many of them (column sums, gates, the head)
// does not average out over the tokens as the per-layer kernels' errors do.  So no sum of those runs through one
// accumulator from end to end: matrix accumulators are emptied into a second one every 32 to 96 of K, and the few sums that
// every token or sample takes part in are kept in 64 bits.  Gradients against float64, geometric mean over 119 drawn
// configurations and 242 deep or narrow ones: 1.30e-7 and 1.47e-7, gates 1.29e-7 and 1.69e-7 (per-layer kernels 1.43e-7,
// 1.66e-7, 1.30e-7, 1.97e-7; with single accumulators 1.55e-7, 1.99e-7, 1.72e-7, 2.58e-7), at 2 us of a step of 400.
//
// All contractions are written on one pattern: an output tile's K range is dealt over the wavefronts of the workgroup, each
// loads both operands straight from memory into 16x16x4 fp32 matrix operands one unit of 16 in K ahead, and the partial
// tiles meet in LDS, added in wavefront order.  An fp32 matrix instruction takes 32 cycles for 2 KFLOP, so a wavefront with
// a 64 x 96 tile needs 2.5 KB of operands per 768 cycles: no operand has to be staged in LDS for its reuse, and there is no
// barrier in any K loop.  Operands contiguous along their K index are read as four K values a lane; operands contiguous
// along the other index as two or four neighbouring rows (columns) a lane, which become row 2 i + c (4 i + c) of the tile:
// nothing is transposed anywhere.  The projections are read from the parameter vector itself (4-byte aligned: the layer
// block's size is odd), so there are no copies of them either.
#include "pac_gemm.h"
#include "pac_internal.h"
#include <mutex>

namespace pac {

#define PAC_LAUNCH(prof, st, cls, ...)                         \
    do {                                                       \
        if (prof) (void)(prof)->mark((st), (cls), true);           \
        hipLaunchKernelGGL(__VA_ARGS__);                       \
        if (prof) (void)(prof)->mark((st), (cls), false);           \
    } while (0)

#define PAC_HIP_TRY(expr)                          \
    do {                                           \
        hipError_t e_ = (expr);                    \
        if (e_ != hipSuccess) return e_;           \
    } while (0)

static inline int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }
static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

typedef float f32x2 __attribute__((ext_vector_type(2)));
// the parameter vector's rows start anywhere: vector loads of 4-byte alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4u *>(p); }
__device__ __forceinline__ f32x2 load2(const float *p) { return *reinterpret_cast<const f32x2u *>(p); }
// from an address that is uniform over the wavefront and this lane's byte offset behind it: no address registers
__device__ __forceinline__ f32x4 load4(const float *p, uint32_t byte) { return *reinterpret_cast<const f32x4u *>(reinterpret_cast<const char *>(p) + byte); }
__device__ __forceinline__ f32x2 load2(const float *p, uint32_t byte) { return *reinterpret_cast<const f32x2u *>(reinterpret_cast<const char *>(p) + byte); }
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

__device__ __forceinline__ float gelu_f(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float u)
{
    const float Phi = 0.5f * (1.f + erff(u * 0.70710678118654752f));
    const float phi = 0.3989422804014327f * expf(-0.5f * u * u);
    return Phi + u * phi;
}
// Classes c0 .. c0 + 3 of one row of a [.][C] array: a row's classes lie together, so a load for each would touch the same
// lines again and again.  Past the last class its value once more.
__device__ __forceinline__ f32x4 load_classes(const float *row, int c0, int C)
{
    if (c0 + 4 <= C) return load4(row + c0);
    f32x4 v;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = row[min(c0 + c, C - 1)];
    return v;
}
// Sums of N values over the lanes, added as a tree of offsets 32, 16, .. 1: with every offset a lane keeps half of the values
// and hands the other half over, so N = 16 takes 17 exchanges, not 96.  Lane i ends with the sum of value i * N / 64.
template <int N, class T> __device__ __forceinline__ T lane_sums(T (&v)[N], int o = 32)
{
    if constexpr (N > 1) {
        const bool hi = threadIdx.x & o;
        T keep[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k)
            keep[k] = (hi ? v[k + N / 2] : v[k]) + __shfl_xor(hi ? v[k] : v[k + N / 2], o, 64);
        return lane_sums<N / 2>(keep, o / 2);
    } else {
        T s = v[0];
        for (; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        return s;
    }
}
__device__ __forceinline__ int pair_index(int k, int l) { return l * (l - 1) / 2 + k; } // k < l

constexpr int kT = kChainRows;   // 16
constexpr int kChunk = 256;      // columns of d per workgroup of the vector parts of the projection launch
constexpr int kZP = 32;          // pitch of Z: classes padded with zeros to one column block
constexpr int kTokRows = 64;     // rows of an output tile of the contractions over the tokens
constexpr int kMaxLayers = 64;

// Which sample a tile belongs to: tile0[s] tiles lie before sample s's (uniform over the workgroup)
__device__ __forceinline__ int sample_of(const int32_t *tile0, int B, int tile)
{
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tile0[mid] <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// contraction cores.  A lane is (i, g) = (lane % 16, lane / 16); a matrix instruction takes row i of A and column i of B at
// K index g from it, and leaves it rows 4 g + v of column i.
// ---------------------------------------------------------------------------

// Requests stay where they are written, a unit ahead of their use: left to itself the compiler moves each load down to its
// first use and waits there (the contractions over the tokens: 220 us, with the requests held 126).
__device__ __forceinline__ void hold_loads() { __builtin_amdgcn_sched_barrier(0); }
// LDS that only one wavefront uses: its lanes' reads and writes stay in order on both sides of this
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 32 NB columns of one K row: blocks of 64, four neighbouring columns a lane, and for odd NB one of 32 with two.  Piece q
// (of 2 NB) of a lane is column col(q, i); a lane's neighbours in memory are its neighbours in the wavefront, which the
// memory pipeline takes four at a time: with 16 rows side by side in the lanes instead it makes 64 accesses of 16 bytes.
template <int NB> struct Cols {
    f32x4 v[NB / 2 + 1];
    static __device__ __forceinline__ int col(int q, int i) { return q < NB / 2 * 4 ? 64 * (q / 4) + 4 * i + q % 4 : 64 * (NB / 2) + 2 * i + q % 4; }
    __device__ __forceinline__ float get(int q) const { return v[q / 4][q % 4]; }
    // row: uniform; row_off: bytes to this lane's own row
    __device__ __forceinline__ void load(const float *row, uint32_t row_off, int i)
    {
#pragma unroll
        for (int b = 0; b < NB / 2; ++b) v[b] = load4(row + 64 * b, row_off + 16 * i);
        if (NB & 1) {
            const f32x2 h = load2(row + 64 * (NB / 2), row_off + 8 * i);
            v[NB / 2][0] = h[0];
            v[NB / 2][1] = h[1];
        }
    }
    // the lane's pieces of one row of an array of 32 NB columns
    template <class F> static __device__ __forceinline__ void store(float *row, int i, const F &piece)
    {
#pragma unroll
        for (int b = 0; b < NB / 2; ++b)
            *reinterpret_cast<f32x4 *>(row + 64 * b + 4 * i) = f32x4{piece(4 * b), piece(4 * b + 1), piece(4 * b + 2), piece(4 * b + 3)};
        if (NB & 1) *reinterpret_cast<f32x2 *>(row + 64 * (NB / 2) + 2 * i) = f32x2{piece(2 * NB - 2), piece(2 * NB - 1)};
    }
};

// ROWS rows contiguous along K through a wavefront's own LDS, 32 of K a step: read as whole 128-byte pieces, eight lanes a
// row, and taken from LDS as operands (row 16 x + i, K = 16 h + 4 g).  The pitch spreads a fragment read over all banks.
constexpr int kStageK = 32, kStagePitch = kStageK + 4;
template <int ROWS> struct RowStage {
    const float *p[ROWS / 8]; // this lane's pieces at K = 0
    f32x4 v[ROWS / 8];
    template <class Row> __device__ __forceinline__ void init(const Row &row) // row(n): where row n starts
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int q = 0; q < ROWS / 8; ++q) p[q] = row(8 * q + (lane >> 3)) + 4 * (lane & 7);
    }
    __device__ __forceinline__ void fetch(int64_t k)
    {
#pragma unroll
        for (int q = 0; q < ROWS / 8; ++q) v[q] = load4(p[q] + k);
    }
    __device__ __forceinline__ void put(float *lds) const
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int q = 0; q < ROWS / 8; ++q)
            *reinterpret_cast<f32x4 *>(lds + (8 * q + (lane >> 3)) * kStagePitch + 4 * (lane & 7)) = v[q];
    }
    static __device__ __forceinline__ f32x4 frag(const float *lds, int x, int h, int i, int g)
    {
        return *reinterpret_cast<const f32x4 *>(lds + (16 * x + i) * kStagePitch + 16 * h + 4 * g);
    }
};

template <int RA, int NB> __device__ __forceinline__ void tt_zero(f32x4 (&acc)[RA][2 * NB])
{
#pragma unroll
    for (int c = 0; c < RA; ++c)
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q) acc[c][q] = zero4();
}
template <int RA, int NB> __device__ __forceinline__ void tt_move(f32x4 (&to)[RA][2 * NB], f32x4 (&from)[RA][2 * NB])
{
#pragma unroll
    for (int c = 0; c < RA; ++c)
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q) {
            to[c][q] += from[c][q];
            from[c][q] = zero4();
        }
}

// A: 16 RT rows contiguous along K, staged in LDS; B: rows contiguous along the columns, bp its row 0.  Steps of 32 in K:
// [s0, s1), the sums of each added to the total by themselves.
template <int RT, int NB>
__device__ __forceinline__ void nn_contract(f32x4 (&acc)[RT][2 * NB], RowStage<16 * RT> &A, float *lds, const float *bp, int ldb, int s0, int s1, int i, int g)
{
    struct Unit { Cols<NB> b[4]; };
    auto load = [&](Unit &t, int u) {
        const float *b = bp + (int64_t)16 * u * ldb;
#pragma unroll
        for (int e = 0; e < 4; ++e) t.b[e].load(b + (int64_t)e * ldb, 16 * g * ldb, i);
    };
    auto mma = [&](const Unit &t, int h) {
        f32x4 av[RT];
#pragma unroll
        for (int x = 0; x < RT; ++x) av[x] = RowStage<16 * RT>::frag(lds, x, h, i, g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int x = 0; x < RT; ++x)
#pragma unroll
                for (int q = 0; q < 2 * NB; ++q) acc[x][q] = mfma16(av[x][e], t.b[e].get(q), acc[x][q]);
    };
    if (s0 >= s1) return;
    f32x4 total[RT][2 * NB];
    tt_zero<RT, NB>(total);
    Unit s, t;
    A.fetch(s0 * kStageK);
    load(s, 2 * s0);
    A.put(lds);
    wave_sync();
    for (int st = s0; st < s1; ++st) {
        const int nx = min(st + 1, s1 - 1); // past the end: the last step again, never used
        A.fetch(nx * kStageK);
        load(t, 2 * st + 1);
        hold_loads();
        mma(s, 0);
        load(s, 2 * nx);
        hold_loads();
        mma(t, 1);
        wave_sync();
        A.put(lds);
        wave_sync();
        tt_move<RT, NB>(total, acc);
    }
    tt_move<RT, NB>(acc, total);
}

// Both operands contiguous along the other index, K rows apart: 16 RA rows (lane i: RA i + c), 32 NB columns.  Src:
//   Idx                    what has to be fetched before a unit's rows can be addressed (requested behind the unit before it)
//   prep(Idx &, u)         fetches it
//   a(Idx, u, e)           this lane's rows at K index 16 u + 4 e + g
//   b(u, e), b_off()       the other operand's row 16 u + 4 e at column 0 of the tile, and bytes from there to row + g
//   live(u, e)             whether that K index counts (else both operands are zero); only asked of the last unit
// FLUSH > 0 (a multiple of 3): the sums of so many units are added to the total by themselves.
template <int RA> struct RowVec;
template <> struct RowVec<2> { typedef f32x2 T; };
template <> struct RowVec<4> { typedef f32x4 T; };
template <int RA, int NB> struct TtUnit {
    typename RowVec<RA>::T a[4];
    Cols<NB> b[4];
};
template <int RA, int NB, int FLUSH = 0, class Src>
__device__ __forceinline__ void tt_contract(f32x4 (&acc)[RA][2 * NB], const Src &src, int u0, int u1, int i)
{
    static_assert(FLUSH % 3 == 0, "whole turns of the loop");
    f32x4 total[FLUSH ? RA : 1][2 * NB];
    if constexpr (FLUSH > 0) tt_zero<RA, NB>(total);
    auto finish = [&]() {
        if constexpr (FLUSH > 0) tt_move<RA, NB>(acc, total);
    };
    typedef typename Src::Idx Idx;
    auto prep = [&](Idx &ix, int u) { src.prep(ix, min(u, u1 - 1)); };
    auto load = [&](TtUnit<RA, NB> &t, const Idx &ix, int u) {
        u = min(u, u1 - 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            t.a[e] = src.a(ix, u, e);
            t.b[e].load(src.b(u, e), src.b_off(), i);
        }
    };
    auto mma = [&](const TtUnit<RA, NB> &t) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int x = 0; x < RA; ++x)
#pragma unroll
                for (int q = 0; q < 2 * NB; ++q) acc[x][q] = mfma16(t.a[e][x], t.b[e].get(q), acc[x][q]);
    };
    auto mask = [&](TtUnit<RA, NB> &t, int u) {
        if (!Src::kMask) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool on = src.live(u, e);
#pragma unroll
            for (int c = 0; c < RA; ++c) t.a[e][c] = on ? t.a[e][c] : 0.f;
#pragma unroll
            for (int q = 0; q < 2 * NB; ++q) t.b[e].v[q / 4][q % 4] = on ? t.b[e].get(q) : 0.f;
        }
    };
    if (u0 >= u1) return;
    // two units ahead: the rows of the cache come from HBM
    TtUnit<RA, NB> r0, r1, r2;
    Idx ix;
    prep(ix, u0);
    load(r0, ix, u0);
    prep(ix, u0 + 1);
    load(r1, ix, u0 + 1);
    prep(ix, u0 + 2);
    int u = u0;
    for (; u + 3 < u1; u += 3) {
        load(r2, ix, u + 2);
        prep(ix, u + 3);
        hold_loads();
        mma(r0);
        load(r0, ix, u + 3);
        prep(ix, u + 4);
        hold_loads();
        mma(r1);
        load(r1, ix, u + 4);
        prep(ix, u + 5);
        hold_loads();
        mma(r2);
        if constexpr (FLUSH > 0)
            if ((u - u0) % FLUSH == FLUSH - 3) tt_move<RA, NB>(total, acc);
    }
    if (u1 - u == 3) load(r2, ix, u + 2);
    hold_loads();
    if (u1 - u == 1) {
        mask(r0, u);
        mma(r0);
        finish();
        return;
    }
    mma(r0);
    if (u1 - u == 2) {
        mask(r1, u + 1);
        mma(r1);
        finish();
        return;
    }
    mma(r1);
    mask(r2, u + 2);
    mma(r2);
    finish();
}

// Both operands contiguous along K, both staged: 16 RT rows, 16 CT columns; steps of 32 in K, at(st): K offset of both
// operands' step; the A operand's units are scaled by scale(u)
template <int RT, int CT, class FA, class FB, class FS>
__device__ __forceinline__ void nt_contract(f32x4 (&acc)[RT][CT], RowStage<16 * RT> &A, RowStage<16 * CT> &B, float *lds, const FA &at_a,
                                            const FB &at_b, const FS &scale, int s0, int s1, int i, int g)
{
    if (s0 >= s1) return;
    float *lb = lds + 16 * RT * kStagePitch;
    A.fetch(at_a(s0));
    B.fetch(at_b(s0));
    A.put(lds);
    B.put(lb);
    wave_sync();
    for (int st = s0; st < s1; ++st) {
        const int nx = min(st + 1, s1 - 1);
        A.fetch(at_a(nx));
        B.fetch(at_b(nx));
        hold_loads();
        const float sc = scale(st);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 av[RT], bv[CT];
#pragma unroll
            for (int x = 0; x < RT; ++x) av[x] = RowStage<16 * RT>::frag(lds, x, h, i, g) * sc;
#pragma unroll
            for (int y = 0; y < CT; ++y) bv[y] = RowStage<16 * CT>::frag(lb, y, h, i, g);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int x = 0; x < RT; ++x)
#pragma unroll
                    for (int y = 0; y < CT; ++y) acc[x][y] = mfma16(av[x][e], bv[y][e], acc[x][y]);
        }
        wave_sync();
        A.put(lds);
        B.put(lb);
        wave_sync();
    }
}

// ---------------------------------------------------------------------------
// launch 1
// ---------------------------------------------------------------------------
struct FProjArgs {
    int blk_off; // first block of this launch (parts may be launched separately for timing)
    BatchMeta meta;
    int32_t tile0[kMaxBatch + 1]; // tiles of 16 RT rows before each sample's
    const float *cache, *params;
    int64_t PL;
    int L, d, C, nch;             // nch: 256-column chunks of d
    int nb_chat, nb_pb, nb_V, nb_tab, nb_Q, nb_U;
    int64_t *rowoff;
    int32_t *rowstride;
    float *cusum, *chatp;         // [L+1][d]; [L][nch][r] shares of (sum_{k<l} c_up^k) W_down^l
    float *V, *pb, *zpbp;         // [L r][C], [B][d], [B][nch][C]
    float *Qf, *Qb, *U;           // [pairs][r][r] in the forward and the backward chain's order, [L][M][r]
};

// U and Q tiles: 16 RT rows x r columns, K = d over the four wavefronts; after it the sums stand in LDS, [16 RT][r].  A tile
// reads all of W_down, so on 16 rows W_down's way through L1 takes twice as long (12 layers of 768 x 96, 4096 rows: the
// launch 133 us, on 32 rows 104, on 64, one workgroup a compute unit, 109; the matrix instructions take 53).
template <int RT, int NB> constexpr int proj_lds()
{
    constexpr int red = 2 * 16 * RT * 32 * NB * 4, stage = 4 * 16 * RT * kStagePitch * 4, small = (5 * kChunk + 4 * kMaxClasses + 4 * 32 * NB) * 4;
    return red > stage ? (red > small ? red : small) : (stage > small ? stage : small);
}
template <int RT, int NB> __device__ __forceinline__ void proj_tile(const FProjArgs &a, const float *arow /* row 0 */, int nrows,
                                                                    const float *Wd, float *lds)
{
    constexpr int r = 32 * NB, rows = 16 * RT;
    const int lane = threadIdx.x & 63, wave = wave_id(), i = lane & 15, g = lane >> 4, d = a.d;
    f32x4 acc[RT][2 * NB];
#pragma unroll
    for (int x = 0; x < RT; ++x)
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q) acc[x][q] = zero4();
    RowStage<rows> A;
    A.init([&](int n) { return arow + (int64_t)min(n, nrows - 1) * d; });
    const int steps = d / kStageK;
    nn_contract<RT, NB>(acc, A, lds + wave * rows * kStagePitch, Wd, r, steps * wave / 4, steps * (wave + 1) / 4, i, g);
    __syncthreads(); // every wavefront is done with its stage
    // wavefronts 2, 3 hand theirs to 0, 1 (in their lanes' order)
    f32x4 *hand = reinterpret_cast<f32x4 *>(lds) + (wave & 1) * RT * 2 * NB * 64 + lane;
    if (wave >= 2) {
#pragma unroll
        for (int x = 0; x < RT; ++x)
#pragma unroll
            for (int q = 0; q < 2 * NB; ++q) hand[(x * 2 * NB + q) * 64] = acc[x][q];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
        for (int x = 0; x < RT; ++x)
#pragma unroll
            for (int q = 0; q < 2 * NB; ++q) acc[x][q] += hand[(x * 2 * NB + q) * 64];
        wave_sync(); // its own piece of LDS again
#pragma unroll
        for (int x = 0; x < RT; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                Cols<NB>::store(lds + (wave * rows + 16 * x + 4 * g + v) * r, i, [&](int q) { return acc[x][q][v]; });
    }
    __syncthreads();
    float sum[(rows * r + 1023) / 1024][4];
#pragma unroll
    for (int q = 0; q < (rows * r + 1023) / 1024; ++q) {
        const int e = min((int)(threadIdx.x + 256 * q) * 4, rows * r - 4);
        *reinterpret_cast<f32x4 *>(sum[q]) = *reinterpret_cast<const f32x4 *>(lds + e) + *reinterpret_cast<const f32x4 *>(lds + rows * r + e);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < (rows * r + 1023) / 1024; ++q) {
        const int e = (threadIdx.x + 256 * q) * 4;
        if (e < rows * r) *reinterpret_cast<f32x4 *>(lds + e) = *reinterpret_cast<const f32x4 *>(sum[q]);
    }
    __syncthreads();
}

// Rows row0 .. + R - 1 of V (one layer's), by a wavefront, four classes at a time.  Bound by how often a wavefront touches the
// lines of W_cls, 64 rows of it at once: a load for each class and row of V took 80 us with 16 classes at 5 layers of 1248 x
// 256 (the step 358 us, 120 of it forward with three classes and 187 with 16), four classes a load and four rows 24 (287; 135).
// Sums of four products, then in 64 bits: V is used for every token, and in fp32 its error was the gates' and biases' largest
// (3 us more with every product in 64 bits at three classes, 40 at 16).
constexpr int kVRows = 4;
template <int R> __device__ __forceinline__ void v_rows(const FProjArgs &a, int row0, int r)
{
    const int lane = threadIdx.x & 63, L = a.L, d = a.d, C = a.C;
    if (row0 >= L * r) return;
    const float *Wc = a.params + (int64_t)L * a.PL;
    const float *wu = a.params + (int64_t)(row0 / r) * a.PL + (int64_t)d * r + r + (int64_t)(row0 % r) * d;
    for (int c0 = 0; c0 < C; c0 += 4) {
        double acc[R * 4];
#pragma unroll
        for (int x = 0; x < R * 4; ++x) acc[x] = 0.;
        for (int j0 = 0; j0 < d; j0 += 64 * 4) {
            float w[R][4];
            f32x4 wc[4];
#pragma unroll
            for (int x = 0; x < R; ++x)
#pragma unroll
                for (int u = 0; u < 4; ++u) w[x][u] = j0 + 64 * u + lane < d ? wu[(int64_t)x * d + j0 + 64 * u + lane] : 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) wc[u] = load_classes(Wc + (int64_t)min(j0 + 64 * u + lane, d - 1) * C, c0, C);
#pragma unroll
            for (int x = 0; x < R; ++x)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float part = w[x][0] * wc[0][c];
#pragma unroll
                    for (int u = 1; u < 4; ++u) part += w[x][u] * wc[u][c];
                    acc[4 * x + c] += (double)part;
                }
        }
        const float v = (float)lane_sums<R * 4>(acc);
        const int at = lane * (R * 4) / 64, c = c0 + at % 4;
        if (lane % (64 / (R * 4)) == 0 && c < C) a.V[(int64_t)(row0 + at / 4) * C + c] = v;
    }
}

template <int RT, int NB> __global__ __launch_bounds__(256) void k_f_proj(FProjArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int r = 32 * NB;
    const int t = threadIdx.x, lane = t & 63, wave = wave_id(), L = a.L, d = a.d, C = a.C;
    const int64_t dr = (int64_t)d * r;
    float *sh = reinterpret_cast<float *>(smem);
    int b = blockIdx.x + a.blk_off;
    if (b < a.nb_chat) {
        // cusum_l over a chunk of d, and its share of chat_l
        const int l = b / a.nch, ch = b % a.nch, j = ch * kChunk + t;
        float cu = 0.f;
        if (j < d) {
            for (int k0 = 0; k0 < l; k0 += 8) { // eight layers' loads issued together
                float c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = a.params[(int64_t)min(k0 + u, l - 1) * a.PL + 2 * dr + r + j];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (k0 + u < l) cu += c[u];
            }
            a.cusum[(int64_t)l * d + j] = cu;
        }
        if (l == L) return;
        sh[t] = cu;
        __syncthreads();
        float *part = sh + kChunk; // [4][r]
        const int nj = min(kChunk, d - ch * kChunk); // a multiple of 32
        const float *Wd = a.params + (int64_t)l * a.PL + (int64_t)ch * kChunk * r;
        for (int n = lane; n < r; n += 64) {
            float acc = 0.f;
            for (int q = wave; q < nj; q += 32) { // eight rows of this wavefront at a time
                float w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) w[u] = Wd[(int64_t)(q + 4 * u) * r + n];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += sh[q + 4 * u] * w[u];
            }
            part[wave * r + n] = acc;
        }
        __syncthreads();
        for (int n = t; n < r; n += 256)
            a.chatp[((int64_t)l * a.nch + ch) * r + n] = part[n] + part[r + n] + part[2 * r + n] + part[3 * r + n];
        return;
    }
    b -= a.nb_chat;
    if (b < a.nb_pb) {
        // mean of b_L over the sample's tokens, a chunk of d; its and cusum_L's share of the logits
        const int s = b / a.nch, ch = b % a.nch, len = a.meta.len[s];
        const float *src = a.cache + a.meta.off[s] + (int64_t)(L - 1) * len * d + min(ch * kChunk + 4 * lane, d - 4);
        f32x4 part[4] = {zero4(), zero4(), zero4(), zero4()};
#pragma unroll 2
        for (int q = wave; q < len; q += 16)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(src + (int64_t)min(q + 4 * e, len - 1) * d);
                part[e] += q + 4 * e < len ? v : zero4();
            }
        const f32x4 acc = (part[0] + part[1]) + (part[2] + part[3]);
        *reinterpret_cast<f32x4 *>(sh + wave * kChunk + 4 * lane) = acc;
        __syncthreads();
        const int j = ch * kChunk + t, jc = min(j, d - 1);
        const float mean = (sh[t] + sh[kChunk + t] + sh[2 * kChunk + t] + sh[3 * kChunk + t]) / (float)len;
        if (j < d) a.pb[(int64_t)s * d + j] = mean;
        float cu = 0.f;
        for (int k0 = 0; k0 < L; k0 += 8) {
            float c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = a.params[(int64_t)min(k0 + u, L - 1) * a.PL + 2 * dr + r + jc];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + u < L) cu += c[u];
        }
        const float y = j < d ? mean + cu : 0.f;
        const float *Wc = a.params + (int64_t)L * a.PL + (int64_t)jc * C;
        float *wred = sh + 4 * kChunk; // [4][kMaxClasses]
#pragma unroll
        for (int c = 0; c < kMaxClasses; ++c) {
            if (c >= C) continue;
            float v = y * Wc[c];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
            if (lane == 0) wred[wave * kMaxClasses + c] = v;
        }
        __syncthreads();
        if (t < C)
            a.zpbp[((int64_t)s * a.nch + ch) * C + t] = wred[t] + wred[kMaxClasses + t] + wred[2 * kMaxClasses + t] + wred[3 * kMaxClasses + t];
        return;
    }
    b -= a.nb_pb;
    if (b < a.nb_V) {
        // V[(k,i)][c] = sum_j W_up^k[i][j] W_cls[j][c]: a wavefront a row; above four classes kVRows of them share what they
        // read of W_cls
        if (C <= 4) v_rows<1>(a, b * 4 + wave, r);
        else v_rows<kVRows>(a, (b * 4 + wave) * kVRows, r);
        return;
    }
    b -= a.nb_V;
    if (b < a.nb_tab) {
        const int at = b * 256 + t, m = min(at, a.meta.M - 1);
        if (at >= max(a.meta.M, 16)) return; // (16 rows: see TokSrc)
        const int s = sample_of(a.meta.tok_start, a.meta.B, m);
        a.rowoff[at] = a.meta.off[s] + (int64_t)(m - a.meta.tok_start[s]) * d;
        a.rowstride[at] = a.meta.len[s] * d;
        return;
    }
    b -= a.nb_tab;
    if (b < a.nb_Q) {
        constexpr int per = r / (16 * RT);
        const int p = b / per, j0 = b % per * 16 * RT;
        int l = 1; // pair_index(k, l) = p
        while (l * (l + 1) / 2 <= p) ++l;
        const int k = p - l * (l - 1) / 2;
        proj_tile<RT, NB>(a, a.params + (int64_t)k * a.PL + dr + r + (int64_t)j0 * d, 16 * RT, a.params + (int64_t)l * a.PL, sh);
        // Both orders the chains read, a kilobyte a load: blocks of 16 x 16, lane (i, g) of a block with K = 4 g .. + 3 of
        // column i.  Forward K is j and the column n, backward the other way about.
        float *Qf = a.Qf + (int64_t)p * r * r, *Qb = a.Qb + (int64_t)p * r * r;
        for (int e = t; e < 4 * RT * r; e += 256) {
            const int n = e % r, jq = e / r; // j = j0 + 4 jq .. + 3
            f32x4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = sh[(4 * jq + c) * r + n];
            *reinterpret_cast<f32x4 *>(Qf + ((((j0 >> 4) + (jq >> 2)) * (r / 16) + (n >> 4)) * 64 + (jq & 3) * 16 + (n & 15)) * 4) = v;
            const int j = e / (r / 4), nq = e % (r / 4); // n = 4 nq .. + 3
            *reinterpret_cast<f32x4 *>(Qb + (((nq >> 2) * (r / 16) + ((j0 + j) >> 4)) * 64 + (nq & 3) * 16 + (j & 15)) * 4) =
                *reinterpret_cast<const f32x4 *>(sh + j * r + 4 * nq);
        }
        return;
    }
    b -= a.nb_Q;
    const int tiles = a.tile0[a.meta.B], l = b / tiles, tile = b % tiles;
    const int s = sample_of(a.tile0, a.meta.B, tile), t0 = (tile - a.tile0[s]) * 16 * RT, len = a.meta.len[s], nrows = min(16 * RT, len - t0);
    proj_tile<RT, NB>(a, a.cache + a.meta.off[s] + ((int64_t)l * len + t0) * d, nrows, a.params + (int64_t)l * a.PL, sh);
    float *U = a.U + ((int64_t)l * a.meta.M + a.meta.tok_start[s] + t0) * r;
    for (int e = 4 * t; e < nrows * r; e += 1024) *reinterpret_cast<f32x4 *>(U + e) = *reinterpret_cast<const f32x4 *>(sh + e);
}

// ---------------------------------------------------------------------------
// launches 2 and 3: the chains over the layers
// ---------------------------------------------------------------------------
struct FChainArgs {
    BatchMeta meta;
    int32_t tile0[kMaxBatch + 1]; // 16-row tiles before each sample's
    int L, d, C, nch;
    const float *params;
    int64_t PL;
    const float *U, *chatp, *Q; // [L][M][r], [L][nch][r], [pairs][r][r] in the direction's order
    float *Gp;                  // [L][M][r] GELU'(pre): written forward, read backward
    float *X;                   // H (forward) or DP (backward), [M][L r]
    float *part;                // column sums of X over each tile, [tiles][L r]
    const float *V, *zpbp;
    float *zpart;               // [tiles][C]
    const int32_t *labels;
    float *logits_out, *dz, *loss_part;
};

// Logits, loss term and dz of sample s, by a workgroup of at least C threads; zs, dzs: C floats of LDS each
__device__ __forceinline__ void f_head(const FChainArgs &a, int s, bool write, float *zs, float *dzs)
{
    const int t = threadIdx.x, C = a.C, B = a.meta.B;
    if (t < C) {
        float z = 0.f, zb = 0.f;
#pragma unroll 8
        for (int k = a.tile0[s]; k < a.tile0[s + 1]; ++k) z += a.zpart[(int64_t)k * C + t];
#pragma unroll 4
        for (int q = 0; q < a.nch; ++q) zb += a.zpbp[((int64_t)s * a.nch + q) * C + t];
        zs[t] = z / (float)a.meta.len[s] + zb + a.params[(int64_t)a.L * a.PL + (int64_t)a.d * C + t];
    }
    __syncthreads();
    if (t == 0) {
        float zmax = -INFINITY;
        for (int c = 0; c < C; ++c) zmax = fmaxf(zmax, zs[c]);
        float se = 0.f;
        for (int c = 0; c < C; ++c) se += expf(zs[c] - zmax);
        const float lse = zmax + logf(se);
        const int y = a.labels[s];
        for (int c = 0; c < C; ++c) {
            const float gz = (expf(zs[c] - lse) - (c == y ? 1.f : 0.f)) / (float)B;
            dzs[c] = gz;
            if (write) {
                if (a.logits_out) a.logits_out[s * C + c] = zs[c];
                a.dz[s * C + c] = gz;
            }
        }
        if (write) a.loss_part[s] = y >= 0 && y < C ? lse - zs[y] : NAN;
    }
    __syncthreads();
}
__global__ __launch_bounds__(64) void k_f_logits(FChainArgs a) // forward-only calls
{
    __shared__ float zs[kMaxClasses], dzs[kMaxClasses];
    f_head(a, blockIdx.x, true, zs, dzs);
}

// The recurrence is per token: a workgroup owns 16 rows and walks the layers, h (dpre) of the finished ones in LDS as the A
// operand, the r x r products read from L2 through a register FIFO that runs ahead across the layers' ends, a kilobyte a
// load.  (Loads with sixteen rows side by side in the lanes: 64 accesses of 16 bytes each, the backward chain 99 us against
// 77.)  A step's K range (all finished layers) is dealt in units of 16 over WK = 8 / WC wavefront groups of WC wavefronts
// with 32 NB columns each; the partial sums meet in LDS, where all threads finish the layer.  Columns dealt instead, six
// wavefronts of 16 at r = 96, would give two of four SIMDs twice the others' matrix instructions.
// 12 layers of r = 96, 256 workgroups, in cycles: 11 k until the first step, 1120 a unit and SIMD where its matrix
// instructions take 768 (operands arriving in registers hold them up: the bare loop takes 1000), 1.0 k (backward) or 2.7 k
// (forward: erf, exp) to finish a layer, 4 k for the rest: 77 and 91 us.  Measured and slower: four wavefronts (97, 111),
// half of the workgroup finishing while the other half starts on the next step's older layers (91, 103).
constexpr int kChainThreads = 512;
static size_t f_chain_lds(int L, int r, int WC)
{
    return 4 * ((size_t)L * kT * (r + 4) + (size_t)8 / WC * kT * r + (size_t)L * r + (size_t)(L + 3) / 4 * 4 + 2 * kMaxClasses + 8 * kMaxClasses);
}
template <bool FWD, int NB, int WC> __global__ __launch_bounds__(kChainThreads) void k_f_chain(FChainArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int r = 32 * NB * WC, RP = r + 4, KB = r / 16, WK = 8 / WC;
    constexpr int kDepth = NB == 1 ? 6 : NB == 2 ? 4 : NB == 3 ? 3 : 2; // units in flight, bounded by the register file
    const int L = a.L, Lr = L * r, M = a.meta.M;
    float *Hs = reinterpret_cast<float *>(smem);     // [L][16][RP]
    float *red = Hs + (size_t)L * kT * RP;           // [WK][16][r]
    float *vec = red + WK * kT * r;                  // [L][r]  (1 - lambda) chat + c_down (forward), dz V^T / len (backward)
    float *lamS = vec + (size_t)L * r;               // [L]
    float *zs = lamS + (L + 3) / 4 * 4, *dzs = zs + kMaxClasses, *zred = dzs + kMaxClasses; // [8][kMaxClasses]
    const int t = threadIdx.x, lane = t & 63, wave = wave_id(), i = lane & 15, g = lane >> 4;
    const int wc = wave % WC, wk = wave / WC;
    const int tile = blockIdx.x, s = sample_of(a.tile0, a.meta.B, tile);
    const int t0 = (tile - a.tile0[s]) * kT, len = a.meta.len[s], nrows = min(kT, len - t0), m0 = a.meta.tok_start[s] + t0;
    auto layer_at = [&](int step) { return FWD ? step : L - 1 - step; };

    // operand units: step `is` contracts units wk, wk + WK, .. of its is * KB, oldest layer first
    struct Slot { f32x4 v[2 * NB]; }; // four K values of each of the wavefront's 2 NB column blocks
    int is = 1, iq = wk;
    while (is < L && iq >= is * KB) ++is;
    int units = 0;
    for (int q = 1; q < L; ++q) units += max(0, q * KB - wk + WK - 1) / WK;
    auto issue = [&](Slot &f) {
        // once the sequence is exhausted its end is requested again and never used: every path issues the same loads
        const int st = is < L ? is : L - 1, q = is < L ? iq : (L - 1) * KB - 1;
        // forward the pairs (k, st) of a step are neighbours, and so are their rows of blocks
        const int k = L - 1 - q / KB;
        const int64_t blk = FWD ? (int64_t)st * (st - 1) / 2 * KB + q : (int64_t)pair_index(L - 1 - st, k) * KB + q % KB;
        const float *p = a.Q + (blk * KB + 2 * NB * wc) * 256 + 4 * lane;
#pragma unroll
        for (int y = 0; y < 2 * NB; ++y) f.v[y] = *reinterpret_cast<const f32x4 *>(p + 256 * y);
        if (is < L) {
            iq += WK;
            while (is < L && iq >= is * KB) { ++is; iq = wk; }
        }
    };
    Slot fifo[kDepth];
    if (units > 0) {
#pragma unroll
        for (int z = 0; z < kDepth; ++z) issue(fifo[z]);
    }
    {
        // U (GELU') of all layers, each where the layer's h (dpre) will stand: requested a step ahead instead, every step
        // waits for its own and so for the operands requested after them
        const float *src = (FWD ? a.U : a.Gp) + (int64_t)m0 * r;
        const int n = L * kT * (r / 4);
        for (int c0 = t; c0 < n; c0 += 8 * kChainThreads) {
            f32x4 v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int c = min(c0 + q * kChainThreads, n - 1), l = c / (kT * (r / 4)), row = c / (r / 4) % kT, cc = c % (r / 4);
                v[q] = *reinterpret_cast<const f32x4 *>(src + ((int64_t)l * M + min(row, nrows - 1)) * r + 4 * cc);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int c = c0 + q * kChainThreads, row = c / (r / 4); // row of the stacked layers' tiles
                if (c < n) *reinterpret_cast<f32x4 *>(Hs + (size_t)row * RP + 4 * (c % (r / 4))) = v[q];
            }
        }
    }
    for (int l = t; l < L; l += kChainThreads) lamS[l] = a.params[(int64_t)l * a.PL + a.PL - 1];
    if (!FWD) f_head(a, s, tile == a.tile0[s], zs, dzs);
    for (int c = t; c < Lr; c += kChainThreads) {
        if (FWD) {
            const int l = c / r, n = c % r;
            const float *pl = a.params + (int64_t)l * a.PL;
            float chat = 0.f;
#pragma unroll 4
            for (int q = 0; q < a.nch; ++q) chat += a.chatp[((int64_t)l * a.nch + q) * r + n];
            vec[c] = (1.f - pl[a.PL - 1]) * chat + pl[(int64_t)a.d * r + n];
        } else {
            double v = 0.;
            for (int q = 0; q < a.C; ++q) v += (double)dzs[q] * (double)a.V[(int64_t)c * a.C + q];
            vec[c] = (float)v / (float)len;
        }
    }
    f32x4 acc[2 * NB];
#pragma unroll
    for (int y = 0; y < 2 * NB; ++y) acc[y] = zero4();
    __syncthreads();

    constexpr int NT = kChainThreads, NE = kT * r / NT;
    auto finish = [&](int step) __attribute__((always_inline)) {
        const int l = layer_at(step);
        const float lam = lamS[l];
        float gp[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = t + NT * q, row = e / r, n = e % r;
            float sum = 0.f;
            if (step > 0) {
#pragma unroll
                for (int w = 0; w < WK; ++w) sum += red[w * kT * r + e];
            }
            float *h = Hs + ((size_t)l * kT + row) * RP + n;
            float out;
            if (FWD) {
                const float pre = lam * *h + (1.f - lam) * sum + vec[l * r + n];
                gp[q] = gelu_grad_f(pre);
                out = gelu_f(pre);
            } else {
                out = (vec[l * r + n] + sum) * *h;
            }
            *h = row < nrows ? out : 0.f;
        }
        if (FWD) {
            float *p = a.Gp + ((int64_t)l * M + m0) * r;
#pragma unroll
            for (int q = 0; q < NE; ++q)
                if ((t + NT * q) / r < nrows) p[t + NT * q] = gp[q];
        }
    };
    finish(0);
    __syncthreads();
    int cs = 1, cq = wk; // the unit to contract next
    auto settle_steps = [&]() __attribute__((always_inline)) { // steps whose units of this wavefront are all done
        while (cs < L && cq >= cs * KB) {
            float *mine = red + wk * kT * r;
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int y = 0; y < 2 * NB; ++y) mine[(4 * g + v) * r + 16 * (2 * NB * wc + y) + i] = acc[y][v];
#pragma unroll
            for (int y = 0; y < 2 * NB; ++y) acc[y] = zero4();
            __syncthreads();
            finish(cs++);
            __syncthreads();
            cq = wk;
        }
    };
    auto contract = [&](const Slot &f) {
        const int q = cq, k = layer_at(q / KB);
        f32x4 av = *reinterpret_cast<const f32x4 *>(Hs + ((size_t)k * kT + i) * RP + 16 * (q % KB) + 4 * g);
        if (!FWD) av *= 1.f - lamS[k];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int y = 0; y < 2 * NB; ++y) acc[y] = mfma16(av[e], f.v[y][e], acc[y]);
        cq += WK;
    };
    for (int p0 = 0; p0 < units; p0 += kDepth) {
#pragma unroll
        for (int z = 0; z < kDepth; ++z) {
            if (p0 + z < units) {
                settle_steps();
                contract(fifo[z]);
            }
            issue(fifo[z]);
        }
    }
    settle_steps();

    // every layer's tile is in LDS: to memory, with its column sums and (forward) the tile's share of the logits
    for (int c = t; c < L * kT * (r / 4); c += kChainThreads) {
        const int l = c / (kT * (r / 4)), row = c / (r / 4) % kT, cc = c % (r / 4);
        if (row < nrows)
            *reinterpret_cast<f32x4 *>(a.X + (int64_t)(m0 + row) * Lr + l * r + 4 * cc) =
                *reinterpret_cast<const f32x4 *>(Hs + ((size_t)l * kT + row) * RP + 4 * cc);
    }
    float zacc[kMaxClasses];
#pragma unroll
    for (int c = 0; c < kMaxClasses; ++c) zacc[c] = 0.f;
    for (int c0 = t; c0 < Lr; c0 += 4 * kChainThreads) {
        float sum[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = min(c0 + u * kChainThreads, Lr - 1), l = c / r, n = c % r;
            sum[u] = 0.f;
#pragma unroll
            for (int q = 0; q < kT; q += 4) {
                const float *h = Hs + ((size_t)l * kT + q) * RP + n;
                sum[u] += (h[0] + h[RP]) + (h[2 * RP] + h[3 * RP]);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + u * kChainThreads < Lr) a.part[(int64_t)tile * Lr + c0 + u * kChainThreads] = sum[u];
            else sum[u] = 0.f;
        if (FWD) {
#pragma unroll
            for (int q0 = 0; q0 < kMaxClasses; q0 += 4) // the loads of four classes under way together
                if (q0 < a.C) {
                    f32x4 v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        v[u] = load_classes(a.V + (int64_t)min(c0 + u * kChainThreads, Lr - 1) * a.C, q0, a.C);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int u = 0; u < 4; ++u) zacc[q0 + q] += sum[u] * v[u][q];
                }
        }
    }
    if (FWD) {
#pragma unroll
        for (int c0 = 0; c0 < kMaxClasses; c0 += 4)
            if (c0 < a.C) {
                float v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = zacc[c0 + c];
                const float sum = lane_sums<4>(v);
                if (lane % 16 == 0) zred[wave * kMaxClasses + c0 + lane / 16] = sum;
            }
        __syncthreads();
        if (t < a.C) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < 8; ++w) v += zred[w * kMaxClasses + t];
            a.zpart[(int64_t)tile * a.C + t] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// launch 4: contractions over the tokens
// ---------------------------------------------------------------------------
struct FTokArgs {
    int blk_off;
    BatchMeta meta;
    int32_t tile0[kMaxBatch + 1];
    const float *cache;
    const int64_t *rowoff;
    const int32_t *rowstride;
    int L, d, r, C, splits;
    int nb_tiles;           // tiles x splits
    const float *H, *DP;    // [M][L r]
    float *E, *G;           // [splits][L][d r], [splits][L r][L r]
    const float *HSpart, *cspart, *dz;
    float *Z, *cs, *dzsum;  // [L r][kZP], [L r], [C]
};

// Sums of the four wavefronts' 16 RA x 32 NB tiles, in wavefront order.  out: element 4 (thread + 256 q) of the tile and the
// three after it.
template <int RA, int NB> constexpr int tt_lds() { return 4 * 16 * RA * 32 * NB * 4; }
template <int RA, int NB> __device__ __forceinline__ void tt_meet(const f32x4 (&acc)[RA][2 * NB], float *red, f32x4 (&out)[RA * NB / 2])
{
    constexpr int cols = 32 * NB, rows = 16 * RA;
    const int lane = threadIdx.x & 63, wave = wave_id(), i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int c = 0; c < RA; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            Cols<NB>::store(red + (wave * rows + RA * (4 * g + v) + c) * cols, i, [&](int q) { return acc[c][q][v]; });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RA * NB / 2; ++q) { // 16 RA x 32 NB / 4 pieces over 256 threads
        const int e = 4 * (threadIdx.x + 256 * q);
        f32x4 s = *reinterpret_cast<const f32x4 *>(red + e);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4 *>(red + w * rows * cols + e);
        out[q] = s;
    }
}

// token rows of the cache (FROM_CACHE) or of H against those of DP.  The last unit ends with the range and repeats tokens of
// the one before it, which do not count again (fewer than 16 tokens in all: it starts at row 0, and the arrays have 16).
template <bool FROM_CACHE> struct TokSrc {
    static constexpr bool kMask = true;
    struct Idx { int64_t off[FROM_CACHE ? 4 : 1]; int32_t str[FROM_CACHE ? 4 : 1]; };
    const float *A, *B; // at column 0 of the tile
    const int64_t *rowoff;
    const int32_t *rowstride;
    int layer, Lr, m0, mend, g, at; // at: this lane's rows of A's tile
    __device__ __forceinline__ int base(int u) const { return max(0, min(m0 + 16 * u, mend - 16)); }
    __device__ __forceinline__ bool live(int u, int e) const
    {
        const int m = base(u) + 4 * e + g;
        return m >= m0 + 16 * u && m < mend;
    }
    __device__ __forceinline__ void prep(Idx &ix, int u) const
    {
        if (FROM_CACHE) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ix.off[e] = rowoff[base(u) + 4 * e + g];
                ix.str[e] = rowstride[base(u) + 4 * e + g];
            }
        }
    }
    __device__ __forceinline__ f32x4 a(const Idx &ix, int u, int e) const
    {
        if (FROM_CACHE) return load4(A + (ix.off[e] + (int64_t)layer * ix.str[e] + at));
        return load4(A + (int64_t)(base(u) + 4 * e) * Lr, 4u * (uint32_t)(g * Lr + at));
    }
    __device__ __forceinline__ const float *b(int u, int e) const { return B + (int64_t)(base(u) + 4 * e) * Lr; }
    __device__ __forceinline__ uint32_t b_off() const { return 4u * (uint32_t)(g * Lr); }
};

// 64 x 32 NB tiles, the tokens (of this split) over four wavefronts, one a SIMD.  A compute unit has 32 KB of lines under way
// at most, so it fetches about 16 bytes a clock where they come from behind L2 and 50 from L2, and a tile of 64 x 96 wants
// 13: a die takes neighbouring tiles of the list below, which share their columns of DP.  Eight wavefronts a workgroup drift
// apart until their rows fall out of L2 (193 us).  Bound by the matrix instructions, 12.2 GFLOP at 12 layers of 768 x 96
// and 4096 rows in 246 tiles, 83 us without a stall; 119 to 124 us, matrix units busy 67 % of it.
constexpr int kTokThreads = 256, kPostThreads = 256;
// Work items numbered so that a die (blocks go round the eight of them) takes neighbours
__device__ __forceinline__ int die_order(int b, int n)
{
    const int die = b & 7, at = b >> 3, full = n >> 3, more = n & 7; // the first `more` dies have one item more
    return die * full + min(die, more) + at;
}
template <int NB> __global__ __launch_bounds__(kTokThreads) void k_f_tok(FTokArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *red = reinterpret_cast<float *>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = wave_id(), i = lane & 15, g = lane >> 4;
    const int L = a.L, r = a.r, Lr = L * r, M = a.meta.M, C = a.C;
    int b = blockIdx.x + a.blk_off;
    if (b >= a.nb_tiles) {
        // column sums of dpre, Z_l = (sum over a sample's tokens of h_l, / len)^T dz: 64 columns, the samples over the
        // wavefronts.  (Dispatched last: in front of the tiles, one of which fills a compute unit, they delayed some of those.)
        b -= a.nb_tiles;
        const int col = b * 64 + lane, cc = min(col, Lr - 1);
        double cs = 0., z[kMaxClasses];
#pragma unroll
        for (int c = 0; c < kMaxClasses; ++c) z[c] = 0.;
        for (int s = wave; s < a.meta.B; s += 4) {
            float hp[4] = {0.f, 0.f, 0.f, 0.f}, cp[4] = {0.f, 0.f, 0.f, 0.f};
            const int q1 = a.tile0[s + 1];
#pragma unroll 2
            for (int q = a.tile0[s]; q < q1; q += 4)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t at = (int64_t)min(q + e, q1 - 1) * Lr + cc;
                    hp[e] += q + e < q1 ? a.HSpart[at] : 0.f;
                    cp[e] += q + e < q1 ? a.cspart[at] : 0.f;
                }
            const float hs = ((hp[0] + hp[1]) + (hp[2] + hp[3])) / (float)a.meta.len[s];
            cs += (double)((cp[0] + cp[1]) + (cp[2] + cp[3]));
#pragma unroll
            for (int c = 0; c < kMaxClasses; ++c)
                if (c < C) z[c] += (double)hs * (double)a.dz[s * C + c];
        }
        red[wave * 64 + lane] = cs;
        float *zr = red + kTokThreads; // [4][kMaxClasses][64]
#pragma unroll
        for (int c = 0; c < kMaxClasses; ++c) zr[(wave * kMaxClasses + c) * 64 + lane] = z[c];
        __syncthreads();
        if (t < 64 && col < Lr) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) v += red[w * 64 + t];
            a.cs[col] = v;
        }
        for (int e = t; e < 64 * kZP; e += kTokThreads) {
            const int q = e / kZP, c = e % kZP;
            float v = 0.f;
            if (c < kMaxClasses)
#pragma unroll
                for (int w = 0; w < 4; ++w) v += zr[(w * kMaxClasses + c) * 64 + q];
            if (b * 64 + q < Lr) a.Z[(int64_t)(b * 64 + q) * kZP + c] = v; // zero from class C on
        }
        if (b == 0 && t < C) {
            double v = 0.;
            for (int s = 0; s < a.meta.B; ++s) v += (double)a.dz[s * C + t];
            a.dzsum[t] = (float)v;
        }
        return;
    }
    // items: layer by layer, E's tiles and then those of G's columns (l, .); the splits fastest
    b = die_order(b, a.nb_tiles);
    const int nbc = r / (32 * NB), split = b % a.splits, tj = (a.d + kTokRows - 1) / kTokRows;
    b /= a.splits;
    int l = L - 1;
    for (;; --l) {
        const int per = nbc * (tj + (l * r + kTokRows - 1) / kTokRows);
        if (b < per || l == 0) break;
        b -= per;
    }
    const int mt = (M + 15) / 16, m0 = 16 * (mt * split / a.splits), mend = min(M, 16 * (mt * (split + 1) / a.splits));
    const int units = (mend - m0 + 15) / 16, u0 = units * wave / 4, u1 = units * (wave + 1) / 4;
    f32x4 acc[4][2 * NB];
    tt_zero<4, NB>(acc);
    f32x4 out[2 * NB];
    if (b < tj * nbc) {
        const int ct = b / tj, j0 = b % tj * kTokRows;
        TokSrc<true> src;
        src.A = a.cache; src.at = min(j0 + 4 * i, a.d - 4); src.B = a.DP + l * r + ct * 32 * NB;
        src.rowoff = a.rowoff; src.rowstride = a.rowstride; src.layer = l; src.Lr = Lr; src.m0 = m0; src.mend = mend; src.g = g;
        tt_contract<4, NB>(acc, src, u0, u1, i);
        tt_meet<4, NB>(acc, red, out);
        float *E = a.E + ((int64_t)split * L + l) * a.d * r + ct * 32 * NB;
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q) {
            const int e = 4 * (t + kTokThreads * q), row = j0 + e / (32 * NB);
            if (row < a.d) *reinterpret_cast<f32x4 *>(E + (int64_t)row * r + e % (32 * NB)) = out[q];
        }
        return;
    }
    // rows (k, .) of the layers before l against columns (l, .)
    b -= tj * nbc;
    const int ct = b % nbc, i0 = b / nbc * kTokRows;
    TokSrc<false> src;
    src.A = a.H + i0; src.at = 4 * i; src.B = a.DP + l * r + ct * 32 * NB; // (rows past the layers' end are the next layer's)
    src.rowoff = nullptr; src.rowstride = nullptr; src.layer = l; src.Lr = Lr; src.m0 = m0; src.mend = mend; src.g = g;
    tt_contract<4, NB>(acc, src, u0, u1, i);
    tt_meet<4, NB>(acc, red, out);
    float *G = a.G + (int64_t)split * Lr * Lr + l * r + ct * 32 * NB;
#pragma unroll
    for (int q = 0; q < 2 * NB; ++q) {
        const int e = 4 * (t + kTokThreads * q), row = i0 + e / (32 * NB);
        if (row < l * r) *reinterpret_cast<f32x4 *>(G + (int64_t)row * Lr + e % (32 * NB)) = out[q];
    }
}

// ordered sums of the token splits, in the first split's place; four elements a thread (both counts are multiples of 4)
__global__ __launch_bounds__(256) void k_f_sum(float *E, int64_t nE, float *G, int64_t nG, int splits, int Lr, int r)
{
    int64_t o = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    float *p = E;
    int64_t n = nE;
    if (o >= nE) {
        o -= nE;
        p = G;
        n = nG;
        if (o >= nG || o / Lr / r >= o % Lr / r) return; // only blocks of an earlier layer's rows exist
    }
    f32x4 v[8]; // splits <= 8
#pragma unroll
    for (int s = 0; s < 8; ++s)
        if (s < splits) v[s] = *reinterpret_cast<const f32x4 *>(p + s * n + o);
    f32x4 acc = v[0];
#pragma unroll
    for (int s = 1; s < 8; ++s)
        if (s < splits) acc += v[s];
    *reinterpret_cast<f32x4 *>(p + o) = acc;
}

// ---------------------------------------------------------------------------
// launch 5: the gradients
// ---------------------------------------------------------------------------
struct FPostArgs {
    int blk_off;
    int L, d, r, C, B;
    int nb_vec, nb_cls, nb_FW;
    const float *params;
    int64_t PL;
    const float *E, *G, *cusum, *cs, *Z, *dzsum, *dz, *pb;
    float *grads, *dlam_part;
    int slots; // per layer
};

// W_up rows (k, i) of the stacked layers (the parameter vector's) against rows of an array of pitch ldb
struct StackSrc {
    static constexpr bool kMask = false;
    struct Idx {};
    const float *A, *B; // W_up^0 at column 0 of its tile, the other operand at its
    int64_t PL;
    int KB, d, ldb, g, at;
    __device__ __forceinline__ bool live(int, int) const { return true; }
    __device__ __forceinline__ void prep(Idx &, int) const {}
    __device__ __forceinline__ f32x2 a(const Idx &, int u, int e) const
    {
        return load2(A + (int64_t)(u / KB) * PL + (int64_t)(16 * (u % KB) + 4 * e) * d, 4u * (uint32_t)(g * d + at));
    }
    __device__ __forceinline__ const float *b(int u, int e) const { return B + (int64_t)(16 * u + 4 * e) * ldb; }
    __device__ __forceinline__ uint32_t b_off() const { return 4u * (uint32_t)(g * ldb); }
};

template <int NB> constexpr int post_lds()
{
    constexpr int red = tt_lds<2, NB>(), stage = 4 * 64 * kStagePitch * 4;
    return red > stage ? red : stage;
}
// 32 x 32 NB tiles of F (rows of d) and 32 x 32 of W (columns of d), K dealt over the wavefronts; the longest contractions
// are dispatched first.  (64 rows and four wavefronts: the last layer's tiles alone take 21 us at 12 layers of 768 x 96.)
template <int NB> __global__ __launch_bounds__(kPostThreads) void k_f_post(FPostArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ float lamS[kMaxLayers], scratch[16];
    float *red = reinterpret_cast<float *>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = wave_id(), i = lane & 15, g = lane >> 4;
    const int L = a.L, d = a.d, r = a.r, C = a.C, Lr = L * r, KB = r / 16;
    const int64_t dr = (int64_t)d * r;
    const int nbc = r / (32 * NB), tj = d / 32;
    const float *Wc = a.params + (int64_t)L * a.PL;
    int b = blockIdx.x + a.blk_off;
    if (b < a.nb_cls) {
        // dW_cls[j][c] = sum_s (mean b_L + cusum_L)[j] dz[s][c] + sum_(k,i) W_up^k[i][j] Z_k[i][c]
        const int j0 = b * 32;
        f32x4 acc[2][2];
        tt_zero<2, 1>(acc);
        StackSrc src;
        src.A = a.params + dr + r + j0; src.at = 2 * i; src.B = a.Z; src.PL = a.PL; src.KB = KB; src.d = d; src.ldb = kZP; src.g = g;
        const int units = L * KB;
        tt_contract<2, 1, 3>(acc, src, units * wave / 4, units * (wave + 1) / 4, i);
        f32x4 out[1];
        tt_meet<2, 1>(acc, red, out);
        const int j = j0 + t / 8, c0 = t % 8 * 4;
        if (c0 < C) {
            const float cl = a.cusum[(int64_t)L * d + j];
            double sum[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[c] = (double)out[0][c];
#pragma unroll 8
            for (int s = 0; s < a.B; ++s) {
                const float p = a.pb[(int64_t)s * d + j] + cl;
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] += (double)p * (double)a.dz[s * C + min(c0 + c, C - 1)];
            }
            float *gc = a.grads + (int64_t)L * a.PL + (int64_t)j * C + c0;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) gc[c] = (float)sum[c];
        }
        return;
    }
    b -= a.nb_cls;
    const int nF = tj * nbc, nW = tj * (r / 32); // tiles of one layer
    const int rank = b / (nF + nW);              // F of the layers from the last down beside W of those from the first up
    int at = b % (nF + nW);
    if (rank < L && at < nF) {
        // dW_down^l = lambda E + (1 - lambda) F, F = sum_{k<l} W_up^kT G_kl + cusum_l^T cs_l; dlambda = <E - F, W_down>
        const int l = L - 1 - rank, slot = at, ct = slot / tj, j0 = slot % tj * 32;
        const float *pl = a.params + (int64_t)l * a.PL;
        f32x4 acc[2][2 * NB];
        tt_zero<2, NB>(acc);
        StackSrc src;
        src.A = a.params + dr + r + j0; src.at = 2 * i; src.B = a.G + l * r + ct * 32 * NB; src.PL = a.PL; src.KB = KB; src.d = d; src.ldb = Lr; src.g = g;
        // what the end reads, under way during the contraction
        const float lam = pl[a.PL - 1];
        constexpr int NP = NB;
        f32x4 Ev[NP], Wv[NP], csv[NP];
        float cu[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int e = 4 * (t + kPostThreads * q), row = j0 + e / (32 * NB), col = ct * 32 * NB + e % (32 * NB);
            Ev[q] = load4(a.E + (int64_t)l * dr + (int64_t)row * r + col);
            Wv[q] = load4(pl + (int64_t)row * r + col);
            csv[q] = load4(a.cs + l * r + col);
            cu[q] = a.cusum[(int64_t)l * d + row];
        }
        const int units = l * KB;
        tt_contract<2, NB, 6>(acc, src, units * wave / 4, units * (wave + 1) / 4, i);
        f32x4 out[NP];
        tt_meet<2, NB>(acc, red, out);
        double dlam = 0.;
        float *gw = a.grads + (int64_t)l * a.PL;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int e = 4 * (t + kPostThreads * q), row = j0 + e / (32 * NB), col = ct * 32 * NB + e % (32 * NB);
            f32x4 gv;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double F = (double)out[q][c] + (double)cu[q] * (double)csv[q][c];
                gv[c] = lam * Ev[q][c] + (1.f - lam) * (float)F;
                dlam += ((double)Ev[q][c] - F) * (double)Wv[q][c];
            }
            *reinterpret_cast<f32x4u *>(gw + (int64_t)row * r + col) = gv;
        }
        const float tot = block_sum((float)dlam, scratch);
        if (t == 0) a.dlam_part[(int64_t)l * a.slots + slot] = tot; // summed in slot order by the last launch
        return;
    }
    for (int l = t; l < L; l += kPostThreads) lamS[l] = a.params[(int64_t)l * a.PL + a.PL - 1];
    if (rank < L) {
        // dW_up^l = Z_l W_cls^T + sum_{k>l} (1 - lambda_k) G_lk W_down^kT: rows (l, .) of G along (k, n)
        __syncthreads();
        at -= nF;
        const int l = rank, i0 = at / tj * 32, j0 = at % tj * 32;
        f32x4 acc[2][2];
        tt_zero<2, 1>(acc);
        RowStage<32> A, B;
        A.init([&](int n) { return a.G + (int64_t)(l * r + i0 + n) * Lr + (l + 1) * r; });
        B.init([&](int n) { return a.params + (int64_t)(l + 1) * a.PL + (int64_t)(j0 + n) * r; });
        const int per = r / kStageK, steps = (L - 1 - l) * per; // a layer's steps
        nt_contract<2, 2>(acc, A, B, red + wave * 64 * kStagePitch, [&](int st) { return (int64_t)st * kStageK; },
                          [&](int st) { return (int64_t)(st / per) * a.PL + st % per * kStageK; },
                          [&](int st) { return 1.f - lamS[l + 1 + st / per]; }, steps * wave / 4, steps * (wave + 1) / 4, i, g);
        __syncthreads(); // every wavefront is done with its stage
#pragma unroll
        for (int x = 0; x < 2; ++x) // [wavefront][32 rows][32 columns]
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(wave * 32 + 16 * x + 4 * g + v) * 32 + 16 * y + i] = acc[x][y][v];
        __syncthreads();
        const int j = j0 + (t & 31);
        float *gw = a.grads + (int64_t)l * a.PL + dr + r;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) v[q] += red[(w * 32 + (t >> 5) + 8 * q) * 32 + (t & 31)];
        }
        const float *Z = a.Z + (int64_t)(l * r + i0 + (t >> 5)) * kZP;
#pragma unroll
        for (int c0 = 0; c0 < kMaxClasses; c0 += 4)
            if (c0 < C) {
                f32x4 z[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) z[q] = *reinterpret_cast<const f32x4 *>(Z + 8 * q * kZP + c0);
                const f32x4 wc = load_classes(Wc + (int64_t)j * C, c0, C);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c0 + c < C)
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] += z[q][c] * wc[c];
            }
#pragma unroll
        for (int q = 0; q < 4; ++q) gw[(int64_t)(i0 + (t >> 5) + 8 * q) * d + j] = v[q];
        return;
    }
    b -= L * (nF + nW);
    if (b == a.nb_vec - 1) { // dc_down^l = cs_l; dc_cls = sum_s dz_s
        for (int c = t; c < Lr; c += kPostThreads) a.grads[(int64_t)(c / r) * a.PL + dr + c % r] = a.cs[c];
        if (t < C) a.grads[(int64_t)L * a.PL + (int64_t)d * C + t] = a.dzsum[t];
        return;
    }
    // dc_up^k[j] = (sum_s dz_s) W_cls^T [j] + sum_{k'>k} (1 - lambda_k') W_down^k'[j] . cs_k': four lanes a row of r
    const int jp = kPostThreads / 4 / L, jj = (t >> 2) / L, k = (t >> 2) % L, q4 = t & 3, j = b * jp + jj;
    const bool act = jj < jp && j < d;
    const float *w = a.params + (int64_t)k * a.PL + (int64_t)(act ? j : 0) * r, *cs = a.cs + k * r;
    float dot = 0.f;
#pragma unroll 4
    for (int n = 4 * q4; n < r; n += 16) {
        const f32x4 x = load4(w + n), y = *reinterpret_cast<const f32x4 *>(cs + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) dot += x[e] * y[e];
    }
    dot += __shfl_xor(dot, 1, 64);
    dot += __shfl_xor(dot, 2, 64);
    float base = 0.f;
    for (int c = 0; c < C; ++c) base += a.dzsum[c] * Wc[(int64_t)(act ? j : 0) * C + c];
    __syncthreads();
    if (act && q4 == 0) red[jj * L + k] = (1.f - lamS[k]) * dot;
    __syncthreads();
    if (!act || q4 != 0) return;
    for (int k2 = k + 1; k2 < L; ++k2) base += red[jj * L + k2];
    a.grads[(int64_t)k * a.PL + 2 * dr + r + j] = base;
}

// the two sums whose terms come from many workgroups, where no optimizer launch follows to do them
__global__ __launch_bounds__(64) void k_f_finish(const float *loss_part, int B, float *loss_out, const float *dlam_part, int slots,
                                                 int L, int64_t PL, float *grads)
{
    const int t = threadIdx.x;
    if (t == 0) {
        float tot = 0.f;
        for (int s = 0; s < B; ++s) tot += loss_part[s];
        *loss_out = tot / (float)B;
    }
    if (grads)
        for (int l = t; l < L; l += 64) {
            double acc = 0.;
#pragma unroll 8
            for (int s = 0; s < slots; ++s) acc += (double)dlam_part[(int64_t)l * slots + s];
            grads[(int64_t)l * PL + PL - 1] = (float)acc;
        }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Columns of a step's units: all of them in one wavefront where the chains' LDS allows it, else (and above r = 96, where its
// registers do not) in two, with half as many partial sums.  0: no room either way
static int chain_wc(int L, int r)
{
    if (r <= 96 && f_chain_lds(L, r, 1) <= 160 * 1024) return 1;
    return r % 64 == 0 && f_chain_lds(L, r, 2) <= 160 * 1024 ? 2 : 0;
}
static int tok_blocks(int r) { return r % 96 == 0 ? 3 : r % 64 == 0 ? 2 : 1; } // r = 32, 64, 96, 128, 192, 256

// Adapters at most half as wide as the hidden state, all layers' 16 rows of h in a compute unit's LDS
bool f32_gram_fits(const Dims &D)
{
    if (D.cache_dtype == 0 || (D.flags & 1)) return false; // PAC_FLAG_PER_LAYER
    if (D.r != 32 && D.r != 64 && D.r != 96 && D.r != 128 && D.r != 192 && D.r != 256) return false;
    return D.L >= 2 && D.L <= kMaxLayers && 2 * D.r <= D.d && chain_wc(D.L, D.r) != 0;
}

// Times in us of both formulations, fitted to 1133 configurations on both sides of the line (2 to 60 layers, d = 64 to 8192,
// every width, 1 to 16384 rows, 1 to 16 classes), within 8 % of those near it in the mean.  What the Gram formulation does
// between layers (L^2 r^2 a row, one row tile after another in a compute unit, and L^2 r^2 d however few the rows are) stands
// against the per-layer kernels' launches, their d-wide state and the weights of one layer at a time.  It is 1.9 x as fast on
// the geometric mean, and loses with wide adapters on few rows or with d = 2 r on many: forward only, 5 layers of 512 x 256,
// 240 rows, 110 us against 96, 31 of 128 x 64, 8192 rows, 502 / 425; steps of 8 layers of 384 x 192, one row, 271 / 242.  What
// the rule picks took up to 1.06 x the other's time in a step and 1.09 x forward only, but for 45 layers of 64 x 32, 16384
// rows (593 / 532).
bool f32_gram_pays(const Dims &D, int B, int M, int ntiles, bool grads)
{
    const double L = D.L, d = D.d, r = D.r, LM = L * M, rounds = cdiv(ntiles, 256), pairs = L * (L - 1) / 2;
    const double chain = pairs * r * r * rounds / 1e6, weights = pairs * r * r * d / 1e9, proj = L * ntiles * 16 * d * r / 1e9;
    double gram, per_layer;
    if (grads) {
        gram = 34.9 + 1.42 * L * rounds + 175 * chain + 24.9 * weights + 30.3 * proj + 0.0046 * d + 52e-6 * L * d * r + 19.3e-6 * LM * r +
               3.6e-9 * M * (L * d * r + pairs * r * r);
        per_layer = 24.8 + L * (13 + 0.0133 * d + 0.0502 * r + 12.7e-6 * d * r) + LM * (1.1e-3 + 5.95e-6 * d + 86e-9 * d * r) +
                    183e-6 * d * B * D.C;
    } else {
        gram = 19.2 + 0.44 * L * rounds + 96 * chain + 17.3 * weights + 24.2 * proj + 0.0128 * d;
        per_layer = 16 + L * (5.34 + 0.00693 * d + 0.0262 * r) + LM * (98e-6 + 2.75e-6 * d + 31.3e-9 * d * r);
    }
    return gram < per_layer;
}

// Token splits: the tiles' rounds over the 256 compute units against what a launch for the sums costs
static int tok_splits(int L, int d, int r, int64_t M)
{
    const int nb = tok_blocks(r), nbc = cdiv(r / 32, nb);
    int tiles = L * nbc * cdiv(d, kTokRows);
    for (int l = 1; l < L; ++l) tiles += nbc * cdiv(l * r, kTokRows);
    const double us = (double)M * kTokRows * 32 * nb * 2 / 0.55e6; // one tile on one compute unit
    int best = 1;
    double least = 1e30;
    for (int s = 1; s <= 8 && M >= (int64_t)128 * s; ++s) {
        const double bytes = 4.0 * (s + 1) * ((double)L * d * r + 0.5 * L * r * L * r);
        const double cost = cdiv((int64_t)tiles * s, 256) * (us / s + 2.0) + (s > 1 ? 4.0 + bytes / 3e6 : 0.0);
        if (cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}

void plan_f32_gram_workspace(const Dims &D, WsLayout &W, int64_t &o)
{
    auto take = [&](int64_t bytes) { int64_t at = o; o = align256(o + bytes); return at; };
    const int64_t Lr = (int64_t)D.L * D.r;
    W.max_tiles = D.B_max * cdiv(D.n_max, kT);
    W.pairs = D.L * (D.L - 1) / 2;
    const int nch = cdiv(D.d, kChunk);
    W.f_splits = tok_splits(D.L, D.d, D.r, D.Mmax);
    const int64_t rows = D.Mmax > 16 ? D.Mmax : 16; // the contractions over the tokens read 16 rows at a time
    W.rowoff = take(rows * 8);
    W.rowstride = take(rows * 4);
    W.dz = take((int64_t)D.B_max * D.C * 4);
    W.pooled = take((int64_t)D.B_max * D.d * 4);
    W.g_zpart = take((int64_t)W.max_tiles * D.C * 4);
    W.g_zpb = take((int64_t)D.B_max * nch * D.C * 4);
    W.g_loss_part = take((int64_t)D.B_max * 4);
    W.g_cusum = take((int64_t)(D.L + 1) * D.d * 4);
    W.g_chat = take(Lr * nch * 4);
    W.g_V = take(Lr * D.C * 4);
    W.g_QpN = take((int64_t)W.pairs * D.r * D.r * 4);
    W.g_QpT = take((int64_t)W.pairs * D.r * D.r * 4);
    W.pre_all = take(D.Mmax * Lr * 4); // U
    W.g_Gp = take(D.Mmax * Lr * 4);
    W.h_all = take(rows * Lr * 4);
    W.g_DP = take(rows * Lr * 4);
    W.g_HSpart = take((int64_t)W.max_tiles * Lr * 4);
    W.g_cspart = take((int64_t)W.max_tiles * Lr * 4);
    W.g_Z = take(Lr * kZP * 4);
    W.g_cs = take(Lr * 4);
    W.g_dzsum = take(kMaxClasses * 4);
    W.g_dlam_slots = D.d / 32 * cdiv(D.r / 32, tok_blocks(D.r));
    W.g_dlam_part = take((int64_t)D.L * W.g_dlam_slots * 4);
    W.grads = take(D.P * 4);
    W.g_Epart = take((int64_t)W.f_splits * D.L * D.d * D.r * 4);
    W.g_GGpart = take((int64_t)W.f_splits * Lr * Lr * 4);
}

// 32-row projection tiles where they still fill the chip twice over and ragged samples do not leave many of them empty
static int proj_row_tiles(int L, int r, int t16, int t32) { return r <= 128 && (int64_t)L * t32 >= 512 && 20 * t32 <= 11 * t16 ? 2 : 1; }

void f32_gram_plan(const Dims &D, const WsLayout &F, const int32_t *lens, int B, int M, int32_t out[4])
{
    int t16 = 0, t32 = 0;
    for (int s = 0; s < B; ++s) {
        const int len = lens ? lens[s] : D.n_max;
        t16 += cdiv(len, 16);
        t32 += cdiv(len, 32);
    }
    const int splits = tok_splits(D.L, D.d, D.r, M);
    out[0] = 1;
    out[1] = 16 * proj_row_tiles(D.L, D.r, t16, t32);
    out[2] = splits < F.f_splits ? splits : F.f_splits;
    out[3] = chain_wc(D.L, D.r);
}

template <auto Kern> static hipError_t allow_lds_once(int lds)
{
    static std::once_flag once;
    static hipError_t result = hipSuccess;
    std::call_once(once, [&] {
        result = hipFuncSetAttribute(reinterpret_cast<const void *>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    return result;
}

// A launch of several parts: in one go, or (for per-part timing) one launch per part with its own profile class
template <class Args, class Kern>
static void launch_parts(Profiler *prof, hipStream_t st, bool split, Kern kern, Args a, int nparts, const int *counts,
                         const int *classes, int whole_class, unsigned threads, size_t lds)
{
    int total = 0;
    for (int p = 0; p < nparts; ++p) total += counts[p];
    a.blk_off = 0;
    if (!split) {
        PAC_LAUNCH(prof, st, whole_class, kern, dim3(total), dim3(threads), lds, st, a);
        return;
    }
    for (int p = 0; p < nparts; ++p) {
        if (counts[p] > 0) PAC_LAUNCH(prof, st, classes[p], kern, dim3(counts[p]), dim3(threads), lds, st, a);
        a.blk_off += counts[p];
    }
}

static int tiles_of(const BatchMeta &meta, int rows, int32_t (&tile0)[kMaxBatch + 1])
{
    int n = 0;
    for (int s = 0; s < meta.B; ++s) {
        tile0[s] = n;
        n += cdiv(meta.len[s], rows);
    }
    tile0[meta.B] = n;
    return n;
}

template <int NB, int WC> static hipError_t run_f32_gram(const Dims &D, const WsLayout &W, const BatchMeta &meta, const StepIO &io)
{
    constexpr int r = 32 * NB * WC, NBT = r % 96 == 0 ? 3 : r % 64 == 0 ? 2 : 1;
    hipStream_t st = io.stream;
    Profiler *prof = io.prof;
    char *ws = io.ws;
    const int L = D.L, d = D.d, C = D.C, M = meta.M, B = meta.B, Lr = L * r, nch = cdiv(d, kChunk);
    const bool split = (D.flags & 2) != 0; // PAC_FLAG_SPLIT_LAUNCH
    auto at = [&](int64_t off) { return (float *)(ws + off); };
    int64_t *rowoff = (int64_t *)(ws + W.rowoff);
    int32_t *rowstride = (int32_t *)(ws + W.rowstride);
    {
        FProjArgs a;
        a.meta = meta;
        a.cache = (const float *)io.cache; a.params = io.params; a.PL = D.PL; a.L = L; a.d = d; a.C = C; a.nch = nch;
        a.rowoff = rowoff; a.rowstride = rowstride; a.cusum = at(W.g_cusum); a.chatp = at(W.g_chat); a.V = at(W.g_V);
        a.pb = at(W.pooled); a.zpbp = at(W.g_zpb); a.Qf = at(W.g_QpT); a.Qb = at(W.g_QpN); a.U = at(W.pre_all);
        const int t16 = tiles_of(meta, 16, a.tile0), t32 = tiles_of(meta, 32, a.tile0);
        const int rt = proj_row_tiles(L, r, t16, t32);
        const int tiles = tiles_of(meta, 16 * rt, a.tile0);
        a.nb_chat = (L + 1) * nch; a.nb_pb = B * nch; a.nb_V = cdiv(Lr, C > 4 ? 4 * kVRows : 4); a.nb_tab = cdiv(M, 256);
        a.nb_Q = W.pairs * (r / (rt > 1 ? 32 : 16)); a.nb_U = L * tiles;
        const int counts[6] = {a.nb_chat, a.nb_pb, a.nb_V, a.nb_tab, a.nb_Q, a.nb_U};
        const int classes[6] = {KC_G_PREP_CHAT, KC_G_PROJ_PB, KC_G_PREP_V, KC_G_PREP_SETUP, KC_G_PROJ_Q, KC_G_PROJ_U};
        auto go = [&](auto kern, int lds) { launch_parts(prof, st, split, kern, a, 6, counts, classes, KC_G_PROJ, 256, lds); };
        if constexpr (r <= 128) {
            PAC_HIP_TRY((allow_lds_once<&k_f_proj<2, NB * WC>>(proj_lds<2, NB * WC>())));
            if (rt == 2) go(&k_f_proj<2, NB * WC>, proj_lds<2, NB * WC>());
        }
        PAC_HIP_TRY((allow_lds_once<&k_f_proj<1, NB * WC>>(proj_lds<1, NB * WC>())));
        if (rt == 1) go(&k_f_proj<1, NB * WC>, proj_lds<1, NB * WC>());
    }
    PAC_HIP_TRY(hipGetLastError());
    FChainArgs ca;
    ca.meta = meta;
    const int tiles = tiles_of(meta, kT, ca.tile0);
    ca.L = L; ca.d = d; ca.C = C; ca.nch = nch; ca.params = io.params; ca.PL = D.PL; ca.U = at(W.pre_all); ca.chatp = at(W.g_chat);
    ca.Q = at(W.g_QpT); ca.Gp = at(W.g_Gp); ca.V = at(W.g_V); ca.zpbp = at(W.g_zpb); ca.zpart = at(W.g_zpart);
    ca.labels = io.labels; ca.logits_out = io.logits_out; ca.dz = at(W.dz); ca.loss_part = at(W.g_loss_part);
    const size_t lds = f_chain_lds(L, r, WC);
    PAC_HIP_TRY((allow_lds_once<&k_f_chain<true, NB, WC>>(160 * 1024)));
    PAC_HIP_TRY((allow_lds_once<&k_f_chain<false, NB, WC>>(160 * 1024)));
    ca.X = at(W.h_all); ca.part = at(W.g_HSpart);
    PAC_LAUNCH(prof, st, KC_G_CHAIN_FWD, (k_f_chain<true, NB, WC>), dim3(tiles), dim3(kChainThreads), lds, st, ca);
    PAC_HIP_TRY(hipGetLastError());
    if (!io.grads) {
        PAC_LAUNCH(prof, st, KC_G_HEAD, k_f_logits, dim3(B), dim3(64), 0, st, ca);
        PAC_LAUNCH(prof, st, KC_G_FINISH, k_f_finish, dim3(1), dim3(64), 0, st, ca.loss_part, B, io.loss_out, (const float *)nullptr, 0, L, D.PL, (float *)nullptr);
        return hipGetLastError();
    }
    ca.Q = at(W.g_QpN); ca.X = at(W.g_DP); ca.part = at(W.g_cspart);
    PAC_LAUNCH(prof, st, KC_G_CHAIN_BWD, (k_f_chain<false, NB, WC>), dim3(tiles), dim3(kChainThreads), lds, st, ca);
    PAC_HIP_TRY(hipGetLastError());
    const int nbc = r / 32 / NBT;
    int splits = tok_splits(L, d, r, M);
    if (splits > W.f_splits) splits = W.f_splits;
    {
        FTokArgs a;
        a.meta = meta;
        tiles_of(meta, kT, a.tile0);
        a.cache = (const float *)io.cache; a.rowoff = rowoff; a.rowstride = rowstride; a.L = L; a.d = d; a.r = r; a.C = C; a.splits = splits;
        a.H = at(W.h_all); a.DP = at(W.g_DP); a.E = at(W.g_Epart); a.G = at(W.g_GGpart);
        a.HSpart = at(W.g_HSpart); a.cspart = at(W.g_cspart); a.dz = at(W.dz); a.Z = at(W.g_Z); a.cs = at(W.g_cs); a.dzsum = at(W.g_dzsum);
        a.nb_tiles = L * nbc * cdiv(d, kTokRows) * splits;
        for (int l = 1; l < L; ++l) a.nb_tiles += nbc * cdiv(l * r, kTokRows) * splits;
        const int counts[2] = {a.nb_tiles, cdiv(Lr, 64)};
        const int classes[2] = {KC_G_TOKRED_E, KC_G_TOKRED_VEC};
        constexpr int red = tt_lds<4, NBT>(), small = kTokThreads * (1 + kMaxClasses) * 4, lds_tok = red > small ? red : small;
        PAC_HIP_TRY((allow_lds_once<&k_f_tok<NBT>>(lds_tok)));
        launch_parts(prof, st, split, &k_f_tok<NBT>, a, 2, counts, classes, KC_G_TOKRED, kTokThreads, lds_tok);
    }
    if (splits > 1) {
        const int64_t nE = (int64_t)L * d * r, nG = (int64_t)Lr * Lr;
        PAC_LAUNCH(prof, st, KC_G_GGSUM, k_f_sum, dim3(cdiv((nE + nG) / 4, 256)), dim3(256), 0, st, at(W.g_Epart), nE, at(W.g_GGpart), nG, splits, Lr, r);
    }
    PAC_HIP_TRY(hipGetLastError());
    FPostArgs pa;
    pa.L = L; pa.d = d; pa.r = r; pa.C = C; pa.B = B; pa.params = io.params; pa.PL = D.PL;
    pa.E = at(W.g_Epart); pa.G = at(W.g_GGpart); pa.cusum = at(W.g_cusum); pa.cs = at(W.g_cs); pa.Z = at(W.g_Z); pa.dzsum = at(W.g_dzsum);
    pa.dz = at(W.dz); pa.pb = at(W.pooled); pa.grads = io.grads; pa.dlam_part = at(W.g_dlam_part);
    pa.slots = d / 32 * nbc;
    pa.nb_cls = d / 32; pa.nb_FW = L * (pa.slots + d / 32 * (r / 32)); pa.nb_vec = cdiv(d, kPostThreads / 4 / L) + 1;
    {
        const int counts[3] = {pa.nb_cls, pa.nb_FW, pa.nb_vec};
        const int classes[3] = {KC_G_POST_VEC, KC_G_POST_F, KC_G_POST_VEC};
        PAC_HIP_TRY((allow_lds_once<&k_f_post<NBT>>(post_lds<NBT>())));
        launch_parts(prof, st, split, &k_f_post<NBT>, pa, 3, counts, classes, KC_G_POST, kPostThreads, post_lds<NBT>());
    }
    if (io.defer) { // the optimizer launch that follows does the last two sums
        io.defer->used = true;
        io.defer->loss_part = ca.loss_part; io.defer->B = B; io.defer->loss_out = io.loss_out;
        io.defer->dlam_part = pa.dlam_part; io.defer->slots = pa.slots; io.defer->wide = true; io.defer->grads = io.grads;
    } else {
        PAC_LAUNCH(prof, st, KC_G_FINISH, k_f_finish, dim3(1), dim3(64), 0, st, ca.loss_part, B, io.loss_out, (const float *)pa.dlam_part, pa.slots, L, D.PL, io.grads);
    }
    return hipGetLastError();
}

hipError_t launch_f32_gram_loss_grad(const Dims &D, const WsLayout &W, const BatchMeta &meta, const StepIO &io)
{
    switch (D.r) {
    case 32: return run_f32_gram<1, 1>(D, W, meta, io);
    case 64: return chain_wc(D.L, D.r) == 1 ? run_f32_gram<2, 1>(D, W, meta, io) : run_f32_gram<1, 2>(D, W, meta, io);
    case 96: return run_f32_gram<3, 1>(D, W, meta, io);
    case 128: return run_f32_gram<2, 2>(D, W, meta, io);
    case 192: return run_f32_gram<3, 2>(D, W, meta, io);
    case 256: return run_f32_gram<4, 2>(D, W, meta, io);
    }
    return hipErrorInvalidValue;
}

} // namespace pac
