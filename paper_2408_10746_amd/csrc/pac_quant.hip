// Block-wise absmax quantisation (Eq. "quan"), its inverse (Eq. "dequan") and the mixed-precision linear layer on
// the stored form, optionally with the cache fill fused into its epilogue (declared in include/pac_quant.h).
#include "../../include/pac_quant.h"
#include "pac_gemm.h"
#include "pac_internal.h"
#include <cmath>

namespace pac {

static inline bool q_aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// ---------------------------------------------------------------------------
// quantise, any block size: one wavefront per block; lanes take pairs of neighbouring values (one byte of 4-bit codes)
// ---------------------------------------------------------------------------
template <int BITS>
__global__ __launch_bounds__(256) void k_quant(const float *__restrict__ x, int64_t n, int block, int64_t nblocks,
                                               int8_t *__restrict__ codes, float *__restrict__ consts)
{
    constexpr float qmax = BITS == 8 ? 127.f : 7.f;
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (int64_t)gridDim.x * 4;
    for (int64_t b = wave; b < nblocks; b += nwaves) {
        const int64_t b0 = b * block;
        const int len = (int)(n - b0 < block ? n - b0 : block);
        float amax = 0.f;
        for (int e = lane; e < len; e += 64) amax = fmaxf(amax, fabsf(x[b0 + e]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        const float c = amax == 0.f ? 1.f : qmax / amax; // correctly rounded 32-bit division
        if (lane == 0) consts[b] = c;
        for (int e = 2 * lane; e < len; e += 128) {
            // 32-bit products, rounded on their own (no contraction with anything), then to the nearest integer, ties to even
            const int q0 = (int)rintf(__fmul_rn(c, x[b0 + e]));
            const int q1 = e + 1 < len ? (int)rintf(__fmul_rn(c, x[b0 + e + 1])) : 0;
            if (BITS == 8) {
                codes[b0 + e] = (int8_t)q0;
                if (e + 1 < len) codes[b0 + e + 1] = (int8_t)q1;
            } else {
                // block is even, so b0 + e is even: this pair is one byte, the even index in the low nibble
                reinterpret_cast<uint8_t *>(codes)[(b0 + e) >> 1] = (uint8_t)((q0 & 0xf) | ((q1 & 0xf) << 4));
            }
        }
    }
}

// The same for blocks of 4 .. 256 values that tile the tensor exactly (block = 4 x a power of two, n a multiple of
// block, 16-byte aligned input): a lane takes four neighbouring values with one 16-byte load, the block's lanes find
// the absmax with lane exchanges, and the four codes leave as one 4-byte (2-byte) store.  One group of four per
// thread, no strided walk.  Same arithmetic, same bits.
template <int BITS>
__global__ __launch_bounds__(256) void k_quant4(const f32x4 *__restrict__ x, int64_t ngroups, int lanes_per_block,
                                                int8_t *__restrict__ codes, float *__restrict__ consts)
{
    constexpr float qmax = BITS == 8 ? 127.f : 7.f;
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = q < ngroups; // (whole blocks never straddle the end: ngroups is a multiple of lanes_per_block)
    const f32x4 v = x[live ? q : ngroups - 1];
    float amax = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
    for (int o = 1; o < lanes_per_block; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
    const float c = amax == 0.f ? 1.f : qmax / amax; // correctly rounded 32-bit division
    if (!live) return;
    if ((q & (lanes_per_block - 1)) == 0) consts[q / lanes_per_block] = c;
    int qv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) qv[e] = (int)rintf(__fmul_rn(c, v[e]));
    if (BITS == 8)
        reinterpret_cast<uint32_t *>(codes)[q] = (uint32_t)(qv[0] & 0xff) | ((uint32_t)(qv[1] & 0xff) << 8) |
                                                 ((uint32_t)(qv[2] & 0xff) << 16) | ((uint32_t)(qv[3] & 0xff) << 24);
    else
        reinterpret_cast<uint16_t *>(codes)[q] = (uint16_t)((qv[0] & 0xf) | ((qv[1] & 0xf) << 4) | ((qv[2] & 0xf) << 8) |
                                                            ((qv[3] & 0xf) << 12));
}

__device__ __forceinline__ int nibble_value(uint32_t byte, int hi)
{
    const int nib = hi ? (int)(byte >> 4) & 0xf : (int)byte & 0xf;
    return nib >= 8 ? nib - 16 : nib;
}

template <int BITS>
__global__ __launch_bounds__(256) void k_dequant(const int8_t *__restrict__ codes, const float *__restrict__ consts,
                                                 int64_t n, int block, float *__restrict__ out)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        const int q = BITS == 8 ? (int)codes[i] : nibble_value(reinterpret_cast<const uint8_t *>(codes)[i >> 1], (int)(i & 1));
        out[i] = __fdiv_rn((float)q, consts[i / block]);
    }
}

// ---------------------------------------------------------------------------
// linear layer on the stored form.  64 WT x 64 WT output tile per workgroup, four wavefronts of WT x WT accumulators of
// 32 x 32 each; K in steps of BK staged through two LDS buffers (x as it is, the codes converted to bf16, which holds
// every code exactly).  A quantisation block's partial sum is kept apart (its first matrix instruction starts from
// zero) and enters the total multiplied by 1 / c of that block and column: in the 32 x 32 accumulator layout all 16
// values of a lane belong to one output column.
// What bounds it: the vector units, which convert the codes and do one multiply-add per output value and block, and the
// barrier of each step.  Hence the launch bound of two workgroups per compute unit: it holds the kernel to 256
// registers, all of them vector registers, where the compiler otherwise kept one set of sums in accumulation registers
// and moved each value out (and back) at every block end.  4096 x 4096 x 4096, 8 bits: blocks of 64 265 -> 209 us,
// of 256 201 -> 170 us, of 32 317 -> 277 us (BK = 32), the constant of the next block requested a block early.
// ---------------------------------------------------------------------------
// bytes per LDS row of a K step: 20 (36) words, so that the 16-byte reads of 16 neighbouring rows meet every bank once
template <int BK> constexpr int kDqPitch = BK * 2 + 16;

struct DqArgs {
    const bf16_t *x;
    int M, K, N, block;
    const int8_t *codes;
    const float *consts;
    float *y;          // dense output, or null
    // fused cache fill (y == null): row m of x is token m % n_max of sample m / n_max
    void *cache;
    int cache_f32, n_max, layer;
    BatchMeta meta;
};

__device__ __forceinline__ uint16_t dq_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu) != 0u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The sums of 32 WTM x 32 WTN outputs a wavefront, from row mw of the tile and column nw on.  Into the cache, each of the tile's
// TM rows is looked up once and kept in LDS, which no wavefront reads any more: looked up at every value instead, a division
// and two dependent loads each, a tile of 128 x 64 took 4 us longer than one of 64 x 64 (1032 x 96, K = 512, blocks of 32: 18.5
// us against 14.5, now 14.3 and 11.7; 500 drawn calls 0.69 to 0.86 of their time by form).
template <int WTM, int WTN, int TM, int THREADS>
__device__ __forceinline__ void dq_store(const DqArgs &a, const f32x16 (&tot)[WTM][WTN], char *lds, int m0, int mw, int nw)
{
    const int i = threadIdx.x & 31, g = (threadIdx.x >> 5) & 1;
    if (a.y) {
#pragma unroll
        for (int y = 0; y < WTN; ++y) {
            const int n = nw + y * 32 + i;
            if (n >= a.N) continue;
#pragma unroll
            for (int x = 0; x < WTM; ++x)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + mw + x * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
                    if (m < a.M) a.y[(int64_t)m * a.N + n] = tot[x][y][v];
                }
        }
        return;
    }
    int64_t *row = reinterpret_cast<int64_t *>(lds); // [TM], -1: not stored
    for (int e = threadIdx.x; e < TM; e += THREADS) {
        int64_t o = -1;
        if (m0 + e < a.M) {
            const int smp = (m0 + e) / a.n_max, tok = m0 + e - smp * a.n_max, len = a.meta.len[smp];
            if (tok < len) o = a.meta.off[smp] + ((int64_t)a.layer * len + tok) * a.N;
        }
        row[e] = o;
    }
    __syncthreads();
    auto put = [&](auto store) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < WTM; ++x)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t o = row[mw + x * 32 + 8 * (v >> 2) + 4 * g + (v & 3)];
                if (o < 0) continue;
#pragma unroll
                for (int y = 0; y < WTN; ++y)
                    if (nw + y * 32 + i < a.N) store(o + nw + y * 32 + i, tot[x][y][v]);
            }
    };
    if (a.cache_f32) put([&](int64_t o, float f) { reinterpret_cast<float *>(a.cache)[o] = f; });
    else put([&](int64_t o, float f) { reinterpret_cast<uint16_t *>(a.cache)[o] = dq_bf16_rne(f); });
}

template <int BITS, int BK, int WT> __global__ __launch_bounds__(256, 2) void k_dq_linear(DqArgs a)
{
    constexpr int TILE = 64 * WT, PITCH = kDqPitch<BK>, PIECES = TILE * BK / 8 / 256, CPR = BK / 8;
    __shared__ __attribute__((aligned(16))) char As[2][TILE * PITCH];
    __shared__ __attribute__((aligned(16))) char Bs[2][TILE * PITCH];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int i = lane & 31, g = lane >> 5;
    const int m0 = blockIdx.y * TILE, n0 = blockIdx.x * TILE;
    const int K = a.K, nsteps = K / BK, bpr = K / a.block, steps_per_block = a.block / BK;
    // this thread's share of a K step: 16 bytes of PIECES x rows, 8 codes of PIECES W rows (256 / CPR rows apart)
    const int lrow = t / CPR, lch = t % CPR;
    const bf16_t *xp[PIECES];
    const int8_t *wp[PIECES];
#pragma unroll
    for (int h = 0; h < PIECES; ++h) {
        const int xm = min(m0 + lrow + 256 / CPR * h, a.M - 1), wr = min(n0 + lrow + 256 / CPR * h, a.N - 1);
        xp[h] = a.x + (int64_t)xm * K + lch * 8;
        wp[h] = a.codes + (BITS == 8 ? (int64_t)wr * K + lch * 8 : ((int64_t)wr * K + lch * 8) / 2);
    }
    auto load = [&](int s, u32x4 (&av)[PIECES], uint64_t (&bv)[PIECES]) {
#pragma unroll
        for (int h = 0; h < PIECES; ++h) {
            av[h] = *reinterpret_cast<const u32x4 *>(xp[h] + s * BK);
            if (BITS == 8) bv[h] = *reinterpret_cast<const uint64_t *>(wp[h] + s * BK);
            else bv[h] = *reinterpret_cast<const uint32_t *>(wp[h] + s * (BK / 2));
        }
    };
    auto store = [&](int buf, const u32x4 (&av)[PIECES], const uint64_t (&bv)[PIECES]) {
#pragma unroll
        for (int h = 0; h < PIECES; ++h) {
            *reinterpret_cast<u32x4 *>(As[buf] + (lrow + 256 / CPR * h) * PITCH + lch * 16) = av[h];
            // a code is an integer of at most 8 bits: its fp32 image has zero low mantissa bits, so the upper half of
            // that image IS its bf16 value (no rounding happens); two codes per 32-bit word
            u32x4 w;
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                int q0, q1;
                if (BITS == 8) {
                    const uint32_t word = (uint32_t)(bv[h] >> (32 * (e2 >> 1)));
                    q0 = (int)(word << (24 - 16 * (e2 & 1))) >> 24;
                    q1 = (int)(word << (16 - 16 * (e2 & 1))) >> 24;
                } else {
                    const uint32_t word = (uint32_t)bv[h];
                    q0 = (int)(word << (28 - 8 * e2)) >> 28;
                    q1 = (int)(word << (24 - 8 * e2)) >> 28;
                }
                w[e2] = (__float_as_uint((float)q0) >> 16) | (__float_as_uint((float)q1) & 0xffff0000u);
            }
            *reinterpret_cast<u32x4 *>(Bs[buf] + (lrow + 256 / CPR * h) * PITCH + lch * 16) = w;
        }
    };
    f32x16 tot[WT][WT], part[WT][WT];
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int y = 0; y < WT; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) tot[x][y][v] = part[x][y][v] = 0.f;
    const float *crow[WT];
    float cnext[WT]; // the coming block's constant, on its way since the block before began
#pragma unroll
    for (int y = 0; y < WT; ++y) {
        crow[y] = a.consts + (int64_t)min(n0 + wn * (32 * WT) + y * 32 + i, a.N - 1) * bpr;
        cnext[y] = crow[y][0];
    }
    auto compute = [&](int buf, bool first) {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 fa[WT], fb[WT];
#pragma unroll
            for (int x = 0; x < WT; ++x)
                fa[x] = *reinterpret_cast<const bf16x8 *>(As[buf] + (wm * (32 * WT) + x * 32 + i) * PITCH + ks * 32 + g * 16);
#pragma unroll
            for (int y = 0; y < WT; ++y)
                fb[y] = *reinterpret_cast<const bf16x8 *>(Bs[buf] + (wn * (32 * WT) + y * 32 + i) * PITCH + ks * 32 + g * 16);
#pragma unroll
            for (int x = 0; x < WT; ++x)
#pragma unroll
                for (int y = 0; y < WT; ++y) {
                    f32x16 c0 = part[x][y];
                    if (ks == 0 && first) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) c0[v] = 0.f; // a new block's partial sum starts from zero
                    }
                    part[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x], fb[y], c0, 0, 0, 0);
                }
        }
    };
    u32x4 av[PIECES];
    uint64_t bv[PIECES];
    load(0, av, bv);
    store(0, av, bv);
    __syncthreads();
    int in_block = 0, blk = 0;
    float cnow[WT];
    for (int s = 0; s < nsteps; ++s) {
        const int buf = s & 1;
        if (in_block == 0) {
#pragma unroll
            for (int y = 0; y < WT; ++y) {
                cnow[y] = cnext[y];
                cnext[y] = crow[y][min(blk + 1, bpr - 1)];
            }
        }
        if (s + 1 < nsteps) load(s + 1, av, bv);
        if (in_block == 0) compute(buf, true);
        else compute(buf, false);
        if (++in_block == steps_per_block) {
            in_block = 0;
            ++blk;
#pragma unroll
            for (int y = 0; y < WT; ++y) {
                const float inv = __fdiv_rn(1.f, cnow[y]);
#pragma unroll
                for (int x = 0; x < WT; ++x)
#pragma unroll
                    for (int v = 0; v < 16; ++v) tot[x][y][v] += part[x][y][v] * inv;
            }
        }
        if (s + 1 < nsteps) store(buf ^ 1, av, bv);
        __syncthreads();
    }
    dq_store<WT, WT, TILE, 256>(a, tot, &As[0][0], m0, wm * (32 * WT), n0 + wn * (32 * WT));
}

// ---------------------------------------------------------------------------
// The same product (bit for bit) for blocks of 32 and 64: a block's products of one 32 x 32 piece are two or four matrix
// instructions, so a partial sum lives from one piece to the next and only the running sums take registers throughout.
// While a piece's matrix instructions run, the vector units scale the piece before it and turn this thread's next codes
// into the next step's tile: in k_dq_linear a step is matrix instructions, then scaling, then conversions, one behind the
// other (1670 cycles a wavefront and step of 64 x 64, 512 of them matrix instructions).  A step of 256 x 128 reads 40 KB from L2
// or behind it (128 x 128 tiles 48 KB for as much) and 128 KB of fragments from LDS.  No unit is near its limit: matrix units
// busy 38 % of the time, LDS 33 %, L2 hits 84 %; a wavefront waits 32 % of its time for memory or a barrier and 28 % to issue,
// with one workgroup a compute unit.  4096 x 4096 x 4096 with operands from memory, against k_dq_linear on 128 x 128 tiles:
// blocks of 64, 209 -> 182 us, of 32, 291 -> 221; 128 x 128 tiles 201 and 234, eight wavefronts of 128 x 256 200 and 235, four
// wavefronts of 256 x 128 with a wider piece each 212.  The order of tiles below: 216 -> 201.
// ---------------------------------------------------------------------------
template <int BITS, int BLK, int WTM, int WTN, int WM, int OCC> __global__ __launch_bounds__(128 * WM, OCC) void k_dq_short(DqArgs a)
{
    constexpr int BK = 64, WN = 2, TM = 32 * WM * WTM, TN = 32 * WN * WTN, PITCH = kDqPitch<BK>;
    constexpr int RP = 8 * WM * WN, PA = TM / RP, PB = TN / RP, KS = BLK / 16, NBLK = BK / BLK; // rows a pass, passes
    constexpr int NT = WTM * WTN * NBLK; // blocks of 32 x 32 x BLK a step
    __shared__ __attribute__((aligned(16))) char lds[2 * (TM + TN) * PITCH];
    auto As = [&](int s) { return lds + (s & 1) * TM * PITCH; };
    auto Bs = [&](int s) { return lds + 2 * TM * PITCH + (s & 1) * TN * PITCH; };
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int i = lane & 31, g = lane >> 5;
    // A die (blocks go round the eight of them) takes a run of tiles eight high: what its workgroups read at a time, 8 + 8
    // tiles of rows for 64 of the output, stays in its L2
    int m0, n0;
    {
        const int nt = (a.N + TN - 1) / TN, mt = (a.M + TM - 1) / TM, all = nt * mt, die = blockIdx.x & 7;
        const int v = die * (all >> 3) + min(die, all & 7) + (blockIdx.x >> 3), mg = v / (8 * nt) * 8, high = min(8, mt - mg);
        m0 = (mg + v % (8 * nt) % high) * TM;
        n0 = v % (8 * nt) / high * TN;
    }
    const int K = a.K, nsteps = (K + BK - 1) / BK, bpr = K / BLK;
    const int lrow = t >> 3, lch = t & 7;
    const bf16_t *xp[PA];
    const int8_t *wp[PB];
#pragma unroll
    for (int h = 0; h < PA; ++h) xp[h] = a.x + (int64_t)min(m0 + lrow + RP * h, a.M - 1) * K + lch * 8;
#pragma unroll
    for (int h = 0; h < PB; ++h) {
        const int wr = min(n0 + lrow + RP * h, a.N - 1);
        wp[h] = a.codes + (BITS == 8 ? (int64_t)wr * K + lch * 8 : ((int64_t)wr * K + lch * 8) / 2);
    }
    u32x4 av[PA];
    uint64_t bv[PB];
    // blocks of 32: a last step of one block reads its pieces twice, and the second half counts as zero
    auto kof = [&](int s) { s = min(s, nsteps - 1); return BLK == 32 && s * BK + lch * 8 >= K ? s * BK - 32 : s * BK; };
    auto load_a = [&](int h, int k) { av[h] = *reinterpret_cast<const u32x4 *>(xp[h] + k); };
    auto load_b = [&](int h, int k) {
        if (BITS == 8) bv[h] = *reinterpret_cast<const uint64_t *>(wp[h] + k);
        else bv[h] = *reinterpret_cast<const uint32_t *>(wp[h] + k / 2);
    };
    auto store_a = [&](int h, int s) {
        const bool dead = BLK == 32 && s * BK + lch * 8 >= K;
        *reinterpret_cast<u32x4 *>(As(s) + (lrow + RP * h) * PITCH + lch * 16) = dead ? u32x4{0, 0, 0, 0} : av[h];
    };
    auto store_b = [&](int h, int s) {
        u32x4 w;
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            int q0, q1;
            if (BITS == 8) {
                const uint32_t word = (uint32_t)(bv[h] >> (32 * (e2 >> 1)));
                q0 = (int)(word << (24 - 16 * (e2 & 1))) >> 24;
                q1 = (int)(word << (16 - 16 * (e2 & 1))) >> 24;
            } else {
                const uint32_t word = (uint32_t)bv[h];
                q0 = (int)(word << (28 - 8 * e2)) >> 28;
                q1 = (int)(word << (24 - 8 * e2)) >> 28;
            }
            // bytes 2, 3 of both images
            w[e2] = __builtin_amdgcn_perm(__float_as_uint((float)q1), __float_as_uint((float)q0), 0x07060302u);
        }
        *reinterpret_cast<u32x4 *>(Bs(s) + (lrow + RP * h) * PITCH + lch * 16) = w;
    };
    f32x16 tot[WTM][WTN];
#pragma unroll
    for (int x = 0; x < WTM; ++x)
#pragma unroll
        for (int y = 0; y < WTN; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) tot[x][y][v] = 0.f;
    const float *crow[WTN];
    float cnext[WTN][NBLK];
    auto consts = [&](int s) {
#pragma unroll
        for (int y = 0; y < WTN; ++y)
#pragma unroll
            for (int q = 0; q < NBLK; ++q) cnext[y][q] = crow[y][min(s * NBLK + q, bpr - 1)];
    };
#pragma unroll
    for (int y = 0; y < WTN; ++y) crow[y] = a.consts + (int64_t)min(n0 + wn * (32 * WTN) + y * 32 + i, a.N - 1) * bpr;
#pragma unroll
    for (int h = 0; h < PA; ++h) load_a(h, kof(0));
#pragma unroll
    for (int h = 0; h < PB; ++h) load_b(h, kof(0));
    consts(0);
#pragma unroll
    for (int h = 0; h < PA; ++h) { store_a(h, 0); load_a(h, kof(1)); }
#pragma unroll
    for (int h = 0; h < PB; ++h) { store_b(h, 0); load_b(h, kof(1)); }
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 part[2];
    part[1] = zero;
    float pinv = 0.f; // of the block whose sums wait in part[(NT - 1) & 1]
    __syncthreads();
    for (int s = 0; s < nsteps; ++s) {
        float inv[WTN][NBLK];
#pragma unroll
        for (int y = 0; y < WTN; ++y)
#pragma unroll
            for (int q = 0; q < NBLK; ++q) inv[y][q] = s * NBLK + q < bpr ? __fdiv_rn(1.f, cnext[y][q]) : 0.f;
        consts(s + 1);
        const char *A = As(s) + (wm * (32 * WTM) + i) * PITCH + g * 16, *B = Bs(s) + (wn * (32 * WTN) + i) * PITCH + g * 16;
        const int k2 = kof(s + 2);
        bf16x8 fa[WTM][KS], fb[2][KS];
        auto read_a = [&](int q) {
#pragma unroll
            for (int x = 0; x < WTM; ++x)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) fa[x][ks] = *reinterpret_cast<const bf16x8 *>(A + x * 32 * PITCH + (q * KS + ks) * 32);
        };
        auto read_b = [&](int n) { // the n-th column block of the step
            const int q = n / WTN, y = n % WTN;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) fb[n & 1][ks] = *reinterpret_cast<const bf16x8 *>(B + y * 32 * PITCH + (q * KS + ks) * 32);
        };
        read_a(0);
        read_b(0);
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int n = b / WTM, x = b % WTM, y = n % WTN, q = n / WTN;
            if (x == 0 && y == 0 && q > 0) read_a(q);
            if (x == 0 && n + 1 < WTN * NBLK) read_b(n + 1);
            part[b & 1] = zero;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) part[b & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[x][ks], fb[n & 1][ks], part[b & 1], 0, 0, 0);
            // the block before it, and this block's share of the next step's tiles
            const int bp = (b + NT - 1) % NT, np = bp / WTM, xp_ = bp % WTM, yp = np % WTN, qp = np / WTN;
            const float pi = b == 0 ? pinv : inv[yp][qp];
#pragma unroll
            for (int v = 0; v < 16; ++v) tot[xp_][yp][v] += part[(b + 1) & 1][v] * pi;
            if (b == NT - 1) pinv = inv[y][q];
#pragma unroll
            for (int h = PA * b / NT; h < PA * (b + 1) / NT; ++h) { store_a(h, s + 1); load_a(h, k2); }
#pragma unroll
            for (int h = PB * b / NT; h < PB * (b + 1) / NT; ++h) { store_b(h, s + 1); load_b(h, k2); }
#pragma unroll
            for (int j = 0; j < KS; ++j) { // one matrix instruction, eight vector instructions
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
            }
            __builtin_amdgcn_sched_barrier(0); // no piece's sums wait longer than to the next one
        }
        static_assert(NT % 2 == 0, "the last block's sums wait in part[1]");
        __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) tot[WTM - 1][WTN - 1][v] += part[1][v] * pinv;
    dq_store<WTM, WTN, TM, 128 * WM>(a, tot, lds, m0, wm * (32 * WTM), n0 + wn * (32 * WTN));
}

static pac_status check_quant_args(const void *a, const void *b, const void *c, int64_t n, int32_t block, int32_t bits)
{
    if (!a || !b || !c) return PAC_ERR_NULL;
    if (bits != 8 && bits != 4) return PAC_ERR_SHAPE;
    if (n < 0 || block < 1 || (bits == 4 && (block & 1))) return PAC_ERR_RANGE;
    return PAC_OK;
}

// Which kernel and tiles.  Blocks of 32 and 64, all forms measured at 6200 drawn shapes with operands from memory and 3200 with
// operands in the last-level cache (16 to 4096 rows, 64 to 4096 columns, K = 256 to 4096, both bit widths, dense and into the
// activation cache).  Two questions, each answered by the logarithm of the two forms' times' ratio as it follows from K, the
// number of tiles, the bit width and where the output goes:
//  - up to three quarters as many 128 x 128 tiles (blocks of 32: as many) as compute units, and up to 64 rows: k_dq_short on 128 x
//    64 tiles, three a compute unit, or k_dq_linear's 64 x 64, of which there are more.  Long K hides the first step's wait; the
//    mean of both kinds' fits, as it is waited for longer with operands from memory: blocks of 32, 135 x 1229, K = 576, 4 bits,
//    10.9 us against 10.8 from memory and 10.8 / 9.5 from the cache, 22 x 3067, K = 928, 15.6 / 18.6 from memory; blocks of 64,
//    128 x 4096 out, K = 4096, 45 / 49 from memory.  Into the activation cache each thread has twice the rows to store behind
//    its last step: 527 x 96, K = 1536, 23.7 / 21.5.
//  - above that many: k_dq_short on wider tiles, or 64 x 64 where K is short: 2546 x 1558, K = 352, blocks of 32, 16.6 / 14.1.
//    128 x 128 tiles run two workgroups a compute unit; 256 x 128 tiles, one workgroup of eight wavefronts, take their place
//    where rounds of them end sooner: a round of 256 against 1.09 for 512 of the smaller, 0.65 where those are one a compute
//    unit.  512 tiles of 256 rows 176 / 190 us (4096 x 4096 x 4096), 172 of them 79.7 / 94.9, 192 76.7 / 84.4, but 128 69.8 /
//    56.9, 288 193 / 167, 384 154 / 146; not for K below 448, where their one first step is waited for by all: 2441 x 2794, K =
//    352, 22.5 / 18.8.
// What this picks is 0.9 % off the fastest form in the mean from memory and 1.0 % from the cache (the sums of both: a rule for
// one kind loses twice that at the other).
// k_dq_linear otherwise, on 64 x 64 tiles up to as many 128 x 128 ones as compute units: longer blocks, K = 4096, 256 tiles
// 72.5 against 74.5 us, 64 tiles 49 / 72, 320 tiles 110.6 / 89.8; odd multiples of 32 keep K steps of 32, where a wide tile
// has less to hide its barriers behind (up to 320); up to 64 rows leave half of a wide tile and more empty.
enum DqForm { DQ_STEP_64, DQ_STEP_128, DQ_SHORT_64, DQ_SHORT_128, DQ_SHORT_256 };
static DqForm dq_short_tiles(int64_t tiles128, int M, int K, int N)
{
    if (K < 448) return DQ_SHORT_128;
    const int64_t tiles256 = (int64_t)((M + 255) / 256) * ((N + 127) / 128), rest = tiles128 % 512;
    const int64_t rounds128 = 109 * (tiles128 / 512) + (rest > 256 ? 109 : rest > 0 ? 65 : 0); // hundredths
    return 100 * ((tiles256 + 255) / 256) <= rounds128 ? DQ_SHORT_256 : DQ_SHORT_128;
}

static DqForm dq_form(int M, int K, int N, int block, int bits, bool to_cache)
{
    const int64_t tiles128 = (int64_t)((N + 127) / 128) * ((M + 127) / 128), tiles64 = (int64_t)((N + 63) / 64) * ((M + 127) / 128);
    const bool b64 = block == 64, many = M > 64 && tiles128 > (b64 ? 192 : block == 32 || block % 64 == 0 ? 256 : 320);
    if (block != 32 && block != 64) return many ? DQ_STEP_128 : DQ_STEP_64;
    const double lk = std::log(K / 1024.0), four = bits == 4, cache = to_cache, few_rows = M <= 64;
    if (many) {
        const double lt = std::log((double)tiles128 / 256.0);
        const double ratio = b64 ? -0.254 - 0.126 * lk - 0.224 * lt + 0.040 * four + 0.126 * cache
                                 : -0.237 - 0.217 * lk - 0.279 * lt + 0.041 * four + 0.090 * cache;
        return ratio < -0.02 ? dq_short_tiles(tiles128, M, K, N) : DQ_STEP_64;
    }
    const double ln = std::log((double)tiles64);
    const double ratio = b64 ? (bits == 8 ? 0.129 - 0.096 * lk - 0.026 * ln + 0.072 * cache : 0.163 - 0.088 * lk - 0.027 * ln + 0.079 * cache)
                             : (bits == 8 ? 0.036 - 0.167 * lk - 0.040 * ln + 0.019 * few_rows + 0.110 * cache
                                          : 0.071 - 0.152 * lk - 0.038 * ln + 0.038 * few_rows + 0.101 * cache);
    return ratio < 0 ? DQ_SHORT_64 : DQ_STEP_64;
}

template <int WTN, int WM, int OCC> static void dq_launch_short(const DqArgs &a, int bits, hipStream_t st)
{
    constexpr int TM = 64 * WM, TN = 64 * WTN;
    const dim3 grid((unsigned)((a.N + TN - 1) / TN) * (unsigned)((a.M + TM - 1) / TM));
    if (a.block == 64) {
        if (bits == 8) hipLaunchKernelGGL((k_dq_short<8, 64, 2, WTN, WM, OCC>), grid, dim3(128 * WM), 0, st, a);
        else hipLaunchKernelGGL((k_dq_short<4, 64, 2, WTN, WM, OCC>), grid, dim3(128 * WM), 0, st, a);
    } else {
        if (bits == 8) hipLaunchKernelGGL((k_dq_short<8, 32, 2, WTN, WM, OCC>), grid, dim3(128 * WM), 0, st, a);
        else hipLaunchKernelGGL((k_dq_short<4, 32, 2, WTN, WM, OCC>), grid, dim3(128 * WM), 0, st, a);
    }
}

template <int BITS, int BK, int WT> static void dq_launch_as(const DqArgs &a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.N + 64 * WT - 1) / (64 * WT)), (unsigned)((a.M + 64 * WT - 1) / (64 * WT)));
    hipLaunchKernelGGL((k_dq_linear<BITS, BK, WT>), grid, dim3(256), 0, st, a);
}

template <int WT> static void dq_launch(const DqArgs &a, int bits, hipStream_t st)
{
    // a K step never spans two blocks; blocks that are an odd multiple of 32 keep steps of 32
    if (a.block % 64 == 0) {
        if (bits == 8) dq_launch_as<8, 64, WT>(a, st);
        else dq_launch_as<4, 64, WT>(a, st);
    } else {
        if (bits == 8) dq_launch_as<8, 32, WT>(a, st);
        else dq_launch_as<4, 32, WT>(a, st);
    }
}

hipError_t launch_dq_linear(const void *x, int M, int K, const int8_t *codes, const float *consts, int N, int block,
                            int bits, float *y, void *cache, int cache_f32, int n_max, int layer, const BatchMeta *meta,
                            hipStream_t st)
{
    DqArgs a{};
    a.x = static_cast<const bf16_t *>(x); a.M = M; a.K = K; a.N = N; a.block = block; a.codes = codes; a.consts = consts;
    a.y = y; a.cache = cache; a.cache_f32 = cache_f32; a.n_max = n_max; a.layer = layer;
    if (meta) a.meta = *meta;
    const DqForm form = dq_form(M, K, N, block, bits, y == nullptr);
    if (form == DQ_SHORT_256) dq_launch_short<2, 4, 1>(a, bits, st);
    else if (form == DQ_SHORT_128) dq_launch_short<2, 2, 2>(a, bits, st);
    else if (form == DQ_SHORT_64) dq_launch_short<1, 2, 3>(a, bits, st);
    else if (form == DQ_STEP_128) dq_launch<2>(a, bits, st);
    else dq_launch<1>(a, bits, st);
    return hipGetLastError();
}

static int check_dq_linear_shape(int32_t M, int32_t K, int32_t N, int32_t block, int32_t bits)
{
    if (bits != 8 && bits != 4) return PAC_ERR_SHAPE;
    if (M < 1 || N < 1 || K < 32 || K % 32) return PAC_ERR_SHAPE;
    if (block < 32 || block % 32 || K % block) return PAC_ERR_RANGE;
    return PAC_OK;
}

int check_dq_linear_args(const void *x, int32_t M, int32_t K, const int8_t *codes, const float *consts, int32_t N,
                                int32_t block, int32_t bits)
{
    if (!x || !codes || !consts) return PAC_ERR_NULL;
    const int s = check_dq_linear_shape(M, K, N, block, bits);
    if (s != PAC_OK) return s;
    if (!q_aligned(x, 16) || !q_aligned(codes, 8) || !q_aligned(consts, 4)) return PAC_ERR_ALIGN;
    return PAC_OK;
}

} // namespace pac

using namespace pac;

extern "C" {

pac_status pac_quant_blockwise(const float *x, int64_t n, int32_t block, int32_t bits, int8_t *codes, float *consts,
                               void *hip_stream)
{
    pac_status s = check_quant_args(x, codes, consts, n, block, bits);
    if (s != PAC_OK) return s;
    if (!q_aligned(x, 4) || !q_aligned(consts, 4)) return PAC_ERR_ALIGN;
    if (n == 0) return PAC_OK;
    (void)hipGetLastError();
    const int64_t nblocks = (n + block - 1) / block;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int lpb = block / 4;
    if (block % 4 == 0 && lpb <= 64 && (lpb & (lpb - 1)) == 0 && n % block == 0 && q_aligned(x, 16) &&
        q_aligned(codes, bits == 8 ? 4 : 2) && n / 4 <= ((int64_t)1 << 30) * 256) {
        const int64_t ngroups = n / 4;
        const unsigned g4 = (unsigned)((ngroups + 255) / 256);
        if (bits == 8)
            hipLaunchKernelGGL(k_quant4<8>, dim3(g4), dim3(256), 0, st, reinterpret_cast<const f32x4 *>(x), ngroups, lpb, codes, consts);
        else
            hipLaunchKernelGGL(k_quant4<4>, dim3(g4), dim3(256), 0, st, reinterpret_cast<const f32x4 *>(x), ngroups, lpb, codes, consts);
        return hipGetLastError() == hipSuccess ? PAC_OK : PAC_ERR_DEVICE;
    }
    int64_t grid = (nblocks + 3) / 4;
    if (grid > 256 * 16) grid = 256 * 16;
    if (bits == 8) hipLaunchKernelGGL(k_quant<8>, dim3((unsigned)grid), dim3(256), 0, st, x, n, block, nblocks, codes, consts);
    else hipLaunchKernelGGL(k_quant<4>, dim3((unsigned)grid), dim3(256), 0, st, x, n, block, nblocks, codes, consts);
    return hipGetLastError() == hipSuccess ? PAC_OK : PAC_ERR_DEVICE;
}

pac_status pac_dequant_blockwise(const int8_t *codes, const float *consts, int64_t n, int32_t block, int32_t bits,
                                 float *out, void *hip_stream)
{
    pac_status s = check_quant_args(codes, consts, out, n, block, bits);
    if (s != PAC_OK) return s;
    if (!q_aligned(out, 4) || !q_aligned(consts, 4)) return PAC_ERR_ALIGN;
    if (n == 0) return PAC_OK;
    (void)hipGetLastError();
    int64_t grid = (n + 255) / 256;
    if (grid > 256 * 32) grid = 256 * 32;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (bits == 8) hipLaunchKernelGGL(k_dequant<8>, dim3((unsigned)grid), dim3(256), 0, st, codes, consts, n, block, out);
    else hipLaunchKernelGGL(k_dequant<4>, dim3((unsigned)grid), dim3(256), 0, st, codes, consts, n, block, out);
    return hipGetLastError() == hipSuccess ? PAC_OK : PAC_ERR_DEVICE;
}

pac_status pac_dequant_linear(const void *x, int32_t M, int32_t K, const int8_t *codes, const float *consts, int32_t N,
                              int32_t block, int32_t bits, float *y, void *hip_stream)
{
    pac_status s = (pac_status)check_dq_linear_args(x, M, K, codes, consts, N, block, bits);
    if (s != PAC_OK) return s;
    if (!y) return PAC_ERR_NULL;
    if (!q_aligned(y, 4)) return PAC_ERR_ALIGN;
    (void)hipGetLastError();
    return launch_dq_linear(x, M, K, codes, consts, N, block, bits, y, nullptr, 0, 0, 0, nullptr,
                            static_cast<hipStream_t>(hip_stream)) == hipSuccess ? PAC_OK : PAC_ERR_DEVICE;
}

pac_status pac_dequant_linear_tiles(int32_t M, int32_t K, int32_t N, int32_t block, int32_t bits, int32_t to_cache, int32_t out[3])
{
    if (!out) return PAC_ERR_NULL;
    const int s = check_dq_linear_shape(M, K, N, block, bits);
    if (s != PAC_OK) return (pac_status)s;
    const DqForm form = dq_form(M, K, N, block, bits, to_cache != 0);
    out[0] = form == DQ_SHORT_64 || form == DQ_SHORT_128 || form == DQ_SHORT_256;
    out[1] = form == DQ_STEP_64 ? 64 : form == DQ_SHORT_256 ? 256 : 128;
    out[2] = form == DQ_STEP_64 || form == DQ_SHORT_64 ? 64 : 128;
    return PAC_OK;
}

} // extern "C"
