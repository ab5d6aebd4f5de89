// The multiplication of the direct-to-LDS engines on v_mfma_f32_16x16x32_bf16: fragment reads, one k-step, write-out.
//
// Why this instruction: a large product on this chip is held back by power before it is by issue slots.  Multiplication
// alone, operands already in registers, 256 CUs, random normal values: 2060-2095 TFLOP/s with 16 x 16 x 32 blocks, 1820 with
// 32 x 32 x 16 (all zeros: 2470 either way).  A 16 x 16 x 32 block passes through half as many accumulators per flop.
//
// Why written out: a k-step (32 of K) of a wave multiplies fragments that are in registers while those of the next k-step are
// on their way from LDS, and loads into LDS go out once these reads are under way; fences of the compiler's scheduler keep
// that order.  2048 x 8192 x 8192, one 256 x 256 tile per CU, two LDS stages of 64, TFLOP/s: reads spread over the whole k-step
// 1243, over its first three quarters 1441, over its first half 1470, that with the loads in the second half 1494 (without
// any loads 1740; the four-stage ring of 32 1353; four waves of 128 x 128 instead of eight of 128 x 64 1391).
//
// Layout of a block: the instruction's operands are exchanged, so that a lane ends up with row lane % 16 and four
// consecutive columns 4 (lane / 16) .. + 3 of every 16 x 16 block of C, which it can store as one vector.
#pragma once
#include <cstdint>
#include "tt_device.h"
#include "gemm_core.h"

namespace tt {
namespace mma {

using core::bf16x8;
using core::f32x4;
using core::u32x2;
using core::u32x4;

// operands of s_waitcnt: at most n vector-memory operations outstanding (_lds: and no LDS operation)
constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
constexpr int waitcnt_vm_lds(int n) { return waitcnt_vm(n) & ~(15 << 8); }

// Row-contiguous operands, tile[k][ROWS / 8 chunks of 8 rows]: chunk position p of k-row k holds row-chunk p ^ rc_swizzle(k).  A
// transpose read of 16 x 32 takes eight pieces of 32 bytes at a time, of k-rows k0 .. k0 + 3 and k0 + 8 .. k0 + 11.  Tiles of 64 rows
// (k-rows of 128 bytes, two to a turn of the banks) have all eight in different banks by bits 1 and 3 of k; by bits 0 and 1,
// as wider tiles, two each share theirs (filter gradient of 24 x 35 x 41 pixels, 384 to 64 channels, 8 shards 55.6 -> 54.5 us with the
// order of the reads in gemm_core2.h; 0.9 M cycles of conflicts -> 0.6 M in one of 32 x 14 x 14, 64 to 64, 8 shards).
template <int ROWS> __device__ __forceinline__ int rc_swizzle(int k) { return ROWS == 64 ? (k & 2) | ((k >> 1) & 4) : (k & 3) << 1; }

// Fragments (16 rows x 32 k, 8 values of K per lane) of an operand tile of ROWS rows and 64 k in LDS; layouts as in gemm_core2.h.
// T: 16-row blocks of a wave, from row w0 on (a multiple of 16 T, of 64 where T is 4 or more).
// BK = 32: one k-step; rows of 64 bytes, chunk position p of row r holds k-chunk p ^ (-(r >> 2) & 3).
template <int ROWS, bool KC, int T, int BK = 64> struct Reader {
    static constexpr bool kc = KC;
    static constexpr int NOFF = KC ? BK / 32 : T < 4 ? T : 4;
    uint32_t off[NOFF]; // the lane's part of the address; the rest are constants
    __device__ __forceinline__ void init(int w0, int lane)
    {
        const int r = lane & 15, q = lane >> 4;
        if constexpr (KC) {
            off[0] = (uint32_t)((w0 + r) * (2 * BK) + ((q ^ (BK == 64 ? (r >> 1) & 7 : -(r >> 2) & 3)) << 4));
            if constexpr (BK == 64) off[1] = off[0] ^ 64u; // k-step 1: chunks 4 to 7
        } else {
            const int k = q * 8 + (r >> 2), c = (w0 >> 3) + ((r & 3) >> 1);
#pragma unroll
            for (int i = 0; i < NOFF; ++i)
                off[i] = (uint32_t)(k * (ROWS * 2) + (((c + 2 * i) ^ rc_swizzle<ROWS>(k)) << 4) + (r & 1) * 8);
        }
    }
    __device__ __forceinline__ bf16x8 read(const char *tile, int ks, int i) const
    {
        if constexpr (KC) {
            return *reinterpret_cast<const bf16x8 *>(tile + off[ks] + i * (32 * BK));
        } else {
            union { dev::s16x4 h[2]; bf16x8 v; } u;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                u.h[h] = dev::lds_read_tr16_b64(tile + off[i & 3] + (i >> 2) * 128 + (ks * 32 + h * 4) * (ROWS * 2));
            return u.v;
        }
    }
};

template <int TM, int TN> struct Frags {
    bf16x8 a[TM], b[TN];
};

template <class RA, class RB, int TM, int TN>
__device__ __forceinline__ void read_frags(Frags<TM, TN> &f, const RA &ra, const RB &rb, const char *At, const char *Bt, int ks)
{
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = rb.read(Bt, ks, j);
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = ra.read(At, ks, i);
}

// acc += cur.a cur.b, and meanwhile nxt = the fragments of k-step ks of the tiles At, Bt, and NLOAD calls issue(0 ..).  The
// step is cut into slots of two MFMAs.  Reads: the first half of the slots (three quarters where fragments take two transpose
// reads each).  Loads into LDS: the second half, or, SPREAD, all slots (a little better where both operands take transpose
// reads).
template <int NLOAD, bool SPREAD, class RA, class RB, int TM, int TN, class Issue>
__device__ __forceinline__ void k_step(f32x4 (&acc)[TM][TN], const Frags<TM, TN> &cur, Frags<TM, TN> &nxt, const RA &ra, const RB &rb,
                                       const char *At, const char *Bt, int ks, Issue &&issue)
{
    constexpr int MM = TM * TN, SL = MM / 2, RD = TM + TN;
    static_assert(MM % 2 == 0 && SL >= 2, "slots");
    constexpr int RS = RA::kc && RB::kc ? SL / 2 : SL * 3 / 4;
    constexpr int L0 = SPREAD ? 0 : SL / 2, LS = SL - L0;
    int mm = 0, rd = 0, ld = 0;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int rto = s >= RS ? RD : (s + 1) * RD / RS, lto = s < L0 ? 0 : (s - L0 + 1) * NLOAD / LS;
#pragma unroll
        for (; rd < rto; ++rd) {
            if (rd < TN) nxt.b[rd] = rb.read(Bt, ks, rd);
            else nxt.a[rd - TN] = ra.read(At, ks, rd - TN);
        }
#pragma unroll
        for (; ld < lto; ++ld) issue(ld);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (; mm < 2 * (s + 1); ++mm) { // rows of blocks back and forth: one operand of each MFMA is the one before's
            const int i = mm / TN, j = i & 1 ? TN - 1 - mm % TN : mm % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.b[j], cur.a[i], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int TM, int TN> __device__ __forceinline__ void multiply(f32x4 (&acc)[TM][TN], const Frags<TM, TN> &f)
{
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jj = 0; jj < TN; ++jj) {
            const int j = i & 1 ? TN - 1 - jj : jj;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
        }
}

template <int TM, int TN> __device__ __forceinline__ void clear(f32x4 (&acc)[TM][TN])
{
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
}

// ---- write-out of a wave's 16 TM x 16 TN block through a wave-private strip of LDS: 16 rows of up to 64 bf16 (fp32: 32) columns
// at a time are turned round and leave as 16-byte vectors of whole row segments (VEC), or, where C's rows do not take
// those, element by element with the lanes of a wave side by side.
constexpr int kStripBytes = 16 * (64 + 8) * 2; // per wave
template <bool OUT_BF16, bool VEC, bool NTS, int TM, int TN>
__device__ __forceinline__ void store_block_as(const f32x4 (&acc)[TM][TN], char *strip, void *Cv, int ldc, int row0, int col0, int M, int N,
                                            bool relu, int lane)
{
    constexpr int E = OUT_BF16 ? 2 : 4, JW = OUT_BF16 ? (TN < 4 ? TN : 4) : (TN < 2 ? TN : 2); // blocks side by side
    constexpr int W = JW * 16, PITCH = W * E + 16, EPV = 16 / E, VPR = W / EPV, NV = 16 * VPR / 64;
    static_assert(16 * PITCH <= kStripBytes && TN % JW == 0 && NV >= 1, "strip");
    const int r = lane & 15, q = lane >> 4;
    char *mine = strip + r * PITCH + q * 4 * E;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jb = 0; jb < TN; jb += JW) {
#pragma unroll
            for (int j = 0; j < JW; ++j) {
                f32x4 v = acc[i][jb + j];
                if (relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
                }
                if constexpr (OUT_BF16) {
                    const u32x2 o = {core::pack_bf16x2(v[0], v[1]), core::pack_bf16x2(v[2], v[3])};
                    *reinterpret_cast<u32x2 *>(mine + j * 32) = o;
                } else {
                    *reinterpret_cast<f32x4 *>(mine + j * 64) = v;
                }
            }
            // wave-private data and LDS operations of a wave execute in order: only the compiler needs a fence
            __builtin_amdgcn_wave_barrier();
            if constexpr (VEC) {
#pragma unroll
                for (int n = 0; n < NV; ++n) {
                    const int idx = lane + 64 * n, lrow = idx / VPR, vc = idx % VPR;
                    const int row = row0 + i * 16 + lrow, col = col0 + jb * 16 + vc * EPV;
                    const u32x4 o = *reinterpret_cast<const u32x4 *>(strip + lrow * PITCH + vc * 16);
                    if (row < M && col < N) // N is a multiple of the vector's length here: a vector is all in or all out
                        dev::store16<NTS>(reinterpret_cast<char *>(Cv) + ((size_t)row * ldc + col) * E, o);
                }
            } else {
                constexpr int RPI = 64 / W; // rows per store
                const int lcol = lane % W, col = col0 + jb * 16 + lcol;
#pragma unroll
                for (int n = 0; n < 16 / RPI; ++n) {
                    const int lrow = n * RPI + lane / W, row = row0 + i * 16 + lrow;
                    if (row < M && col < N) {
                        const char *s = strip + lrow * PITCH + lcol * E;
                        if constexpr (OUT_BF16) reinterpret_cast<uint16_t *>(Cv)[(size_t)row * ldc + col] = *reinterpret_cast<const uint16_t *>(s);
                        else __builtin_nontemporal_store(*reinterpret_cast<const float *>(s), reinterpret_cast<float *>(Cv) + (size_t)row * ldc + col);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
}

// nts: non-temporal stores (non_temporal_results in tt_internal.h says when)
template <bool OUT_BF16, bool VEC, int TM, int TN>
__device__ __forceinline__ void store_block(const f32x4 (&acc)[TM][TN], char *strip, void *Cv, int ldc, int row0, int col0, int M, int N,
                                            bool relu, int lane, bool nts)
{
    if (!VEC || nts) store_block_as<OUT_BF16, VEC, true>(acc, strip, Cv, ldc, row0, col0, M, N, relu, lane);
    else store_block_as<OUT_BF16, VEC, false>(acc, strip, Cv, ldc, row0, col0, M, N, relu, lane);
}

} // namespace mma
} // namespace tt
