// Small and odd-sized shard products: fp32 of any size, bf16 operands whose rows are not whole 16-byte vectors.
//
// What bounds these products is latency, not arithmetic: 32 x 512 x 256 is 8 MFLOP, and a shard of it fills a handful of
// workgroups that each walk K alone.  So K is cut over the waves of a workgroup: every wave multiplies its own K chunks of
// a 32 x 32 (or 64 x 64) output block with MFMAs on fragments that it loads straight from global memory into registers,
// up to four chunks ahead (nothing is shared between the waves before the end, so there is no barrier in the K loop), and
// the waves' partial blocks are added once through LDS.  The same LDS block turns the accumulators into rows, so that any
// row pitch is stored coalesced.  bf16 operands use v_mfma_f32_32x32x16_bf16, fp32 ones v_mfma_f32_32x32x2_f32 (products
// and sums in fp32, K in a fixed order: chunks of one wave in increasing order, then waves in increasing order).
//
// (bf16 A B, the forward layout, short K and most of fp32 run on the ordered kernel of gemm_small.hip instead.)
// Measured on MI355X (before: the plain kernel of 64 x 64 tiles, K walked by one workgroup):
//   bf16 A B^T / A^T B 256 x 2047 x 2047 202 -> 18-24 us, 4 x (101 x 225 x 1500) 140 -> 8-13 us, 4095 x 4093 x 4091 2720 ->
//   550-600 us; fp32 256 x 2047 x 2047 204 -> 41-44 us, 4 x (32 x 128 x 256) 25.5 -> 8 us, 4095 x 4093 x 4091 2730 -> 1210-1520 us.
// What is left of the small ones is the launch, one trip to memory each for the pointers, the operands and the results.
//
// A chunk is one 128-byte line of an operand row: 64 bf16 or 32 fp32 values of K.  Lane l holds row l % 32 of a block and,
// with h = l / 32, the K values 16 s + 8 h .. + 7 of MFMA step s (bf16) or 8 i + 4 h + e of steps i, e (fp32).
//   K-contiguous bf16: whole rows of a chunk are loaded as 4-byte words, 32 lanes to a row, and turned into fragments
//     through a wave-private LDS tile.  (A lane that loads 16 bytes of its own row, as the fragment wants them, touches 64
//     lines per load, most of them at odd 16-byte positions: 256 x 2047 x 2047 took 105 us that way, NT layout.)
//   K-contiguous fp32: 16-byte loads of the lane's own row, which need no alignment beyond the element's (the target runs
//     with unaligned global access on; the type below says so to the compiler).
//   Row-contiguous operand: one load per K value, coalesced along the rows.  bf16 with 64-row blocks: lane l loads the pair
//   of rows 2 l, 2 l + 1 as one 4-byte word, which feeds both 32-row fragments (which rows a fragment holds is free as long
//   as the write-out agrees), so both fragments come out of eight loads and eight byte permutes.
// Rows past the end are clamped (they feed results that are never stored).  What K leaves over after whole chunks is the
// last whole chunk's worth of K once more with the values already taken zeroed in both operands; K below one chunk is
// loaded value by value from clamped addresses, zeroed past the end.
#pragma once
#include <cstdint>
#include <type_traits>
#include "tt_device.h"
#include "gemm_core.h"

namespace tt {
namespace small {

using core::bf16x8;
using core::f32x16;

struct __attribute__((packed, aligned(4))) Quad32 { float f[4]; };      // 16 bytes at any 4-byte boundary
struct __attribute__((packed, aligned(2))) Pair16 { uint32_t w; };      // 4 bytes at any 2-byte boundary
struct __attribute__((packed, aligned(4))) Pair32 { uint32_t w[2]; };   // 8 bytes at any 4-byte boundary

template <int NS> struct ParamsT { // tables of NS shards
    const void *A[NS];
    const void *B[NS];
    void *C[NS];
    int32_t M, N, K;
    int64_t lda, ldb;     // elements between rows of the stored matrices
    int32_t ldc;
    int32_t tiles_m, tiles_n; // workgroup tiles
    int32_t per_xcd, total;   // per_xcd = 0: workgroups in launch order
    int32_t ksplit, kchunk;   // K cut between workgroups (partial results), as in the other engines
    int32_t wm, wn, wk;       // waves of a workgroup along M, N and K
    int32_t relu, out_bf16;
};
using ParamsS = ParamsT<64>;

// T blocks of 32 per side of a wave's output; most waves a workgroup has
template <int T> constexpr int waves_of() { return T == 1 ? 8 : 4; }
template <bool BF> constexpr int chunk_k() { return BF ? 64 : 32; }

// One operand of a wave's block: T * 32 rows, K contiguous (KC) or rows contiguous.
// OFF: type of a lane's byte offset from the wave-uniform block origin (32 bits unless the row pitch is huge).
template <bool BF, bool KC, int T, class OFF> struct Operand {
    static constexpr int ES = BF ? 2 : 4;
    static constexpr bool PAIR = BF && !KC && T == 2; // rows 2 l and 2 l + 1 of the block share a lane
    static constexpr bool STAGED = BF && KC;          // through the wave's LDS tile: T * 32 rows of 128 bytes
    static constexpr int kLdsBytes = STAGED ? T * 32 * 128 : 0;
    const char *base;   // row `row0`, k = 0
    int64_t kstep;      // bytes from k to k + 1
    OFF off[PAIR ? 1 : T];
    OFF word_off, last_off; // staged: this lane's word of rows 2 i + h; of the last row alone
    int last_pair;          // ... the pair that row is in, if it stands alone there or pairs past it are asked for
    int64_t pair_step;      // ... bytes from one pair of rows to the next
    int shift;          // PAIR: 16 where the pair was moved back by one row at the end of an odd operand

    __device__ __forceinline__ static int row_in_block(int t, int l32) { return PAIR ? 2 * l32 + t : 32 * t + l32; }

    __device__ __forceinline__ void init(const void *mat, int64_t ld, int row0, int rows, int lane)
    {
        const int l32 = lane & 31, h = lane >> 5;
        // (a pair needs two rows to load from: a block of one row starts one row early; rows >= 2 on that path)
        const int first = PAIR && row0 == rows - 1 ? row0 - 1 : row0;
        const int last = rows - 1 - first; // >= 0, pairs: >= 1
        kstep = KC ? ES : ld * ES;
        base = reinterpret_cast<const char *>(mat) + (KC ? (int64_t)first * ld : (int64_t)first) * ES;
        shift = 0;
        if constexpr (PAIR) {
            // the first row of the pair; where it is the last row there is, the pair before it is loaded and shifted
            int r = row0 - first + 2 * l32;
            if (r >= last) { shift = r > last ? 0 : 16; r = last - 1; }
            off[0] = (OFF)r * (OFF)ES + (OFF)(8 * h) * (OFF)kstep;
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                int r = 32 * t + l32;
                r = r < last ? r : last;
                off[t] = KC ? (OFF)r * (OFF)(ld * ES) + (OFF)((BF ? 8 : 4) * h * ES)
                            : (OFF)r * (OFF)ES + (OFF)((BF ? 8 : 4) * h) * (OFF)kstep;
            }
            if constexpr (STAGED) {
                pair_step = 2 * ld * ES;
                last_pair = last / 2;
                word_off = (OFF)h * (OFF)(ld * ES) + (OFF)(4 * l32);
                last_off = last & 1 ? word_off : (OFF)(4 * l32);
            }
        }
    }
    __device__ __forceinline__ const char *at(int t, int64_t k) const { return base + k * kstep + off[t]; }

    // registers of one chunk
    struct Raw {
        uint32_t w[BF ? (KC ? T * 16 : (PAIR ? 32 : T * 32)) : T * 16];
    };

    // whole chunk starting at k0
    __device__ __forceinline__ void load(Raw &r, int k0) const
    {
        if constexpr (STAGED) {
#pragma unroll
            for (int i = 0; i < T * 16; ++i) { // (scalar: which pair of rows; pairs past the last repeat it)
                const bool inside = i < last_pair;
                const char *p = base + (int64_t)k0 * ES + (inside ? i : last_pair) * pair_step;
                r.w[i] = reinterpret_cast<const Pair16 *>(p + (inside ? word_off : last_off))->w;
            }
        } else if constexpr (BF && PAIR) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) r.w[s * 8 + e] = reinterpret_cast<const Pair16 *>(at(0, k0 + 16 * s + e))->w;
        } else if constexpr (BF) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e) r.w[(t * 4 + s) * 8 + e] = *reinterpret_cast<const uint16_t *>(at(t, k0 + 16 * s + e));
        } else if constexpr (KC) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Quad32 c = *reinterpret_cast<const Quad32 *>(at(t, k0 + 8 * i));
#pragma unroll
                    for (int e = 0; e < 4; ++e) r.w[(t * 4 + i) * 4 + e] = __float_as_uint(c.f[e]);
                }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) r.w[(t * 4 + i) * 4 + e] = *reinterpret_cast<const uint32_t *>(at(t, k0 + 8 * i + e));
        }
    }

    // one K value of one block row, zero from kend on (by AND: a select over a load would be turned into a branch, and a
    // wait for every load).  The lane's own K offset is inside off[]; it is taken out of the clamped position, so the
    // address never passes the last K value.
    __device__ __forceinline__ uint32_t load_one(int t, int k, int kend, int h) const
    {
        const int kl = (BF ? 8 : 4) * h, kk = k + kl < kend ? k : kend - 1 - kl; // kk + kl is the K value read
        const char *p = at(PAIR ? 0 : t, kk);
        uint32_t v;
        if constexpr (PAIR) v = reinterpret_cast<const Pair16 *>(p)->w;
        else v = BF ? *reinterpret_cast<const uint16_t *>(p) : *reinterpret_cast<const uint32_t *>(p);
        return v & (k + kl < kend ? 0xffffffffu : 0u);
    }
    // the chunk at k0, of which only the K values before kend exist
    __device__ __forceinline__ void load_tail(Raw &r, int k0, int kend, int lane) const
    {
        const int h = lane >> 5;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int t = 0; t < (PAIR ? 1 : T); ++t) {
                if constexpr (BF && KC) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t lo = load_one(t, k0 + 16 * s + 2 * q, kend, h), hi = load_one(t, k0 + 16 * s + 2 * q + 1, kend, h);
                        r.w[(t * 4 + s) * 4 + q] = lo | (hi << 16);
                    }
                } else if constexpr (BF) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) r.w[(t * 4 + s) * 8 + e] = load_one(t, k0 + 16 * s + e, kend, h);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) r.w[(t * 4 + s) * 4 + e] = load_one(t, k0 + 8 * s + e, kend, h);
                }
            }
        }
    }

    // staged operands: the loaded rows into the wave's LDS tile (16-byte chunk q of row r at q ^ (r / 2 % 8)) ...
    __device__ __forceinline__ void stage(Raw &r, char *lds, int lane) const
    {
        if constexpr (STAGED) {
            const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
            for (int i = 0; i < T * 16; ++i)
                *reinterpret_cast<uint32_t *>(lds + (2 * i + h) * 128 + (((l32 >> 2) ^ (i & 7)) << 4) + (l32 & 3) * 4) = r.w[i];
        }
    }
    // ... and, after all of them, back as the lane's fragments
    __device__ __forceinline__ void unstage(Raw &r, const char *lds, int lane) const
    {
        if constexpr (STAGED) {
            const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int row = 32 * t + l32;
                    const core::u32x4 v = *reinterpret_cast<const core::u32x4 *>(lds + row * 128 + (((2 * s + h) ^ ((row >> 1) & 7)) << 4));
#pragma unroll
                    for (int q = 0; q < 4; ++q) r.w[(t * 4 + s) * 4 + q] = v[q];
                }
        }
    }

    // bf16 fragment of block t, MFMA step s (MASK: the chunk's K values below `skip` read as zero)
    template <bool MASK> __device__ __forceinline__ bf16x8 frag(const Raw &r, int t, int s, int skip, int lane) const
    {
        union { uint32_t w[4]; bf16x8 v; } u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (KC) u.w[q] = r.w[(t * 4 + s) * 4 + q];
            else if constexpr (PAIR) {
                const uint32_t a = r.w[s * 8 + 2 * q] >> shift, b = r.w[s * 8 + 2 * q + 1] >> shift;
                u.w[q] = t == 0 ? (a & 0xffffu) | (b << 16) : (a >> 16) | (b & 0xffff0000u);
            } else u.w[q] = r.w[(t * 4 + s) * 8 + 2 * q] | (r.w[(t * 4 + s) * 8 + 2 * q + 1] << 16);
            if constexpr (MASK) {
                const int k = 16 * s + 8 * (lane >> 5) + 2 * q;
                u.w[q] &= k >= skip ? 0xffffffffu : k + 1 >= skip ? 0xffff0000u : 0u;
            }
        }
        return u.v;
    }
    template <bool MASK> __device__ __forceinline__ float value(const Raw &r, int t, int i, int e, int skip, int lane) const
    {
        const float v = __uint_as_float(r.w[(t * 4 + i) * 4 + e]);
        return !MASK || 8 * i + 4 * (lane >> 5) + e >= skip ? v : 0.0f;
    }
};

// bytes of LDS per wave: its output block as fp32 rows, or its staged operands before that
template <bool BF, bool A_KC, bool B_KC, int T> constexpr int lds_per_wave()
{
    return T * T * 4096 > (BF && A_KC ? T * 4096 : 0) + (BF && B_KC ? T * 4096 : 0) ? T * T * 4096
                                                                                    : (BF && A_KC ? T * 4096 : 0) + (BF && B_KC ? T * 4096 : 0);
}

// one wave's output block: adds the WK partial blocks of the workgroup's waves and stores this wave's share of the rows
// (LW: floats from one wave's block to the next)
template <int WK, int S, int LW> __device__ __forceinline__ void store_share(const ParamsS &p, const float *blk, void *C, int my_k, int m0, int n0, int lane)
{
    constexpr int N = S * S / WK / 64, U = N < 4 ? N : 4;
    for (int i0 = 0; i0 < N; i0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int in = my_k * (S * S / WK) + (i0 + u) * 64 + lane;
            float v = blk[in];
#pragma unroll
            for (int q = 1; q < WK; ++q) v += blk[q * LW + in];
            if (p.relu) v = v > 0.0f ? v : 0.0f;
            const int row = m0 + in / S, col = n0 + in % S;
            if (row < p.M && col < p.N) {
                const size_t o = (size_t)row * p.ldc + col;
                if (p.out_bf16) reinterpret_cast<uint16_t *>(C)[o] = (uint16_t)core::f32_to_bf16_bits(v);
                else reinterpret_cast<float *>(C)[o] = v;
            }
        }
    }
}

template <bool BF, bool A_KC, bool B_KC, int T, class OFF>
__device__ __forceinline__ void run_small(const ParamsS &p, char *lds)
{
    constexpr int KU = chunk_k<BF>(), S = T * 32, LW = lds_per_wave<BF, A_KC, B_KC, T>();
    const int logical = p.per_xcd > 0 ? core::logical_block(p.per_xcd, p.total) : (int)blockIdx.x;
    if (logical < 0) return; // uniform over the workgroup
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = logical / tiles, t = logical - vshard * tiles;
    const int wk = p.wk, wn = p.wn;
    const int m_wg = (t % p.tiles_m) * (p.wm * S), n_wg = (t / p.tiles_m) * (wn * S);
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int kend = p.kchunk < p.K - kbeg ? kbeg + p.kchunk : p.K;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int my_k = wave % wk, blk = wave / wk;
    const int m0 = m_wg + blk / wn * S, n0 = n_wg + blk % wn * S;

    f32x16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    using OA = Operand<BF, A_KC, T, OFF>;
    using OB = Operand<BF, B_KC, T, OFF>;
    using RA = typename OA::Raw;
    using RB = typename OB::Raw;
    OA a;
    OB b;
    // four chunks on their way per wave; two where a chunk takes more than 32 registers, or where both operands are staged
    // (the staging's own registers do not fit beside four)
    constexpr int PD = (sizeof(RA) + sizeof(RB)) / 4 > 32 || (OA::STAGED && OB::STAGED) ? 2 : 4;
    char *const lds_a = lds + wave * LW, *const lds_b = lds_a + OA::kLdsBytes;

    const auto multiply = [&](const RA &xa, const RB &xb, int skip, auto mask) {
        constexpr bool MASK = decltype(mask)::value;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (MASK && (BF ? 16 : 8) * (s + 1) <= skip) continue; // (wave-uniform) nothing left of this step
            if constexpr (BF) {
                bf16x8 fa[T], fb[T];
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    fa[i] = a.template frag<MASK>(xa, i, s, skip, lane);
                    fb[i] = b.template frag<MASK>(xb, i, s, skip, lane);
                }
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.template value<MASK>(xa, i, s, e, skip, lane),
                                                                            b.template value<MASK>(xb, j, s, e, skip, lane), acc[i][j], 0, 0, 0);
            }
        }
    };
    // rows as loaded -> fragments (wave-private LDS: operations of a wave execute in order, only the compiler needs a fence)
    const auto restage = [&](RA &xa, RB &xb) {
        if constexpr (OA::STAGED || OB::STAGED) {
            a.stage(xa, lds_a, lane);
            b.stage(xb, lds_b, lane);
            __builtin_amdgcn_wave_barrier();
            a.unstage(xa, lds_a, lane);
            b.unstage(xb, lds_b, lane);
            __builtin_amdgcn_wave_barrier();
        }
    };

    if (m0 < p.M && n0 < p.N && kend > kbeg) { // (wave-uniform)
        a.init(p.A[shard], p.lda, m0, p.M, lane);
        b.init(p.B[shard], p.ldb, n0, p.N, lane);
        if (kend - kbeg >= KU) {
            // chunks my_k, my_k + wk, ... of this wave; the last of all may start early (see the top) and then skips what
            // the one before it has taken
            const int chunks = (int)(((int64_t)kend - kbeg + KU - 1) / KU);
            if (my_k < chunks) {
                RA ra[PD];
                RB rb[PD];
                // loads past this wave's last chunk fetch the last chunk of all again (never used), so no load sits under a branch
                const auto at = [&](int c) { const int64_t k = kbeg + (int64_t)c * KU; return (int)(k < kend - KU ? k : kend - KU); };
#pragma unroll
                for (int d = 0; d < PD; ++d) {
                    a.load(ra[d], at(my_k + d * wk));
                    b.load(rb[d], at(my_k + d * wk));
                }
                for (int c = my_k; c < chunks; c += PD * wk) {
#pragma unroll
                    for (int d = 0; d < PD; ++d) { // (unrolled: the register ring is indexed by constants)
                        const int cd = c + d * wk;
                        if (cd >= chunks) break;
                        restage(ra[d], rb[d]);
                        const int skip = (int)(kbeg + (int64_t)cd * KU - at(cd)); // 0 for whole chunks
                        if (skip == 0) multiply(ra[d], rb[d], 0, std::false_type());
                        else multiply(ra[d], rb[d], skip, std::true_type());
                        a.load(ra[d], at(cd + PD * wk));
                        b.load(rb[d], at(cd + PD * wk));
                    }
                }
            }
        } else if (my_k == 0) {
            RA ra;
            RB rb;
            a.load_tail(ra, kbeg, kend, lane);
            b.load_tail(rb, kbeg, kend, lane);
            multiply(ra, rb, 0, std::false_type());
        }
    }

    // every wave leaves its block in LDS as rows; then each adds and stores its share of its block's rows
    float *mine = reinterpret_cast<float *>(lds + wave * LW);
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                mine[OA::row_in_block(i, m) * S + OB::row_in_block(j, lane & 31)] = acc[i][j][e];
            }
    __syncthreads();
    const float *const first = reinterpret_cast<const float *>(lds + blk * wk * LW);
    void *const C = p.C[vshard];
    if (wk == 1) store_share<1, S, LW / 4>(p, first, C, my_k, m0, n0, lane);
    else if (wk == 2) store_share<2, S, LW / 4>(p, first, C, my_k, m0, n0, lane);
    else if (wk == 4) store_share<4, S, LW / 4>(p, first, C, my_k, m0, n0, lane);
    else if constexpr (T == 1) store_share<8, S, LW / 4>(p, first, C, my_k, m0, n0, lane);
}

} // namespace small
} // namespace tt
