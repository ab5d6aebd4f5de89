// Second bf16 MFMA tile engine: operand tiles go from global memory straight into LDS (global_load_lds_dwordx4, no
// register hop and no LDS store instructions), eight waves per workgroup (two per SIMD), BM x 256 tiles, two LDS stages of 64 k.
// K steps, fragments and write-out are those of gemm_mma.h; how operand elements are addressed is a policy ("loader"): dense
// matrices here, gathered image windows and runs of pixels in conv.hip.  K need not be a multiple of 64.
//
// LDS layouts (no padding is possible: a wave-wide direct load writes 64 x 16 contiguous bytes, lane by lane; instead
// each lane chooses WHICH global chunk it fetches, which gives an XOR swizzle for free):
//   K-contiguous operand  tile[row][8 chunks of 8 k]   chunk position p of row r holds k-chunk p ^ ((r >> 1) & 7);
//                         fragments are plain 16-byte reads.
//   row-contiguous operand tile[k][ROWS / 8 chunks of 8 rows]  chunk position p of k-row k holds row-chunk p ^ ((k & 3) << 1)
//                         (64 rows: see rc_swizzle in gemm_mma.h);
//                         fragments are two ds_read_b64_tr_b16 (LDS transpose reads): within 16 lanes, lane i receives
//                         element i % 4 of the 4-element rows addressed by lanes 4e + i / 4, e = 0..3, so addressing
//                         row (k0 + j / 4, rows 4 (j % 4) ..) from lane j hands lane i the values (k0 + e, row i).
// Out-of-range chunks (K tails, image padding) are fetched from a 16-byte block of zeros instead of being masked.
#pragma once
#include <cstdint>
#include "tt_device.h"
#include "gemm_core.h"
#include "gemm_mma.h"

namespace tt {
namespace core2 {

using core::BK;

constexpr int kThreads2 = 512;
constexpr int BM2 = 256, BN2 = 256;
constexpr size_t kSmemBytes = 2 * (size_t)(BM2 + BN2) * BK * 2; // 128 KB

__device__ __attribute__((aligned(16))) const uint32_t g_zero_chunk[4] = {0, 0, 0, 0};

__device__ __forceinline__ uint64_t uniform64(const char *p)
{
    // wave-uniform by construction; say so, or an "s" operand may be handed a vector register pair (readfirstlane
    // returns a signed int: go through uint32_t so the low half is not sign-extended)
    const uint64_t b64 = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b64);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b64 >> 32));
    return ((uint64_t)hi << 32) | (uint64_t)lo;
}

// a lane's chunk at base + off, or zeros for lanes that have none (some_missing: whether there are such lanes, wave-uniform)
__device__ __forceinline__ void chunk_or_zero(uint32_t off, uint64_t base, bool have, bool some_missing, uint32_t lds_wave_addr)
{
    if (!some_missing) dev::lds_dma16(off, base, lds_wave_addr);
    else dev::lds_dma16(have ? (const void *)(reinterpret_cast<const char *>(base) + off) : (const void *)g_zero_chunk, lds_wave_addr);
}

// ---- loaders of one operand's ROWS x 64 tiles, by the NT threads of a workgroup.  Thread t fetches chunks t + NT i,
// ---- i < loads2<ROWS, NT>(), to 16 (t + NT i).
//   begin<ROWS>(row0)      : K tile 0 of the rows from row0 on is the current one
//   next<ROWS>()           : the K tile after it
//   issue<ROWS>(i, lds)    : chunk i of the current tile; lds: address of the tile's stage in LDS
// Where ROWS is no multiple of 64, the last chunks belong to the first waves alone.
template <int ROWS, int NT = kThreads2> constexpr int loads2() { return (ROWS * 8 + NT - 1) / NT; }
__device__ __forceinline__ uint32_t wave2() { return (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
template <int ROWS, int NT = kThreads2> __device__ __forceinline__ bool mine2(int i)
{
    return (i + 1) * NT <= ROWS * 8 || (int)wave2() * 64 + i * NT < ROWS * 8;
}
template <int NT = kThreads2> __device__ __forceinline__ uint32_t chunk_lds2(uint32_t lds, int i) { return lds + (wave2() * 64u + (uint32_t)i * NT) * 16u; }

// KC: rows of the operand have K contiguous
template <int NT> struct DenseKCT {
    static constexpr bool KC = true;
    const char *base;
    int ld, rows, K;
    uint32_t voff[8]; // this lane's chunks, bytes from the K tile's start
    int k;            // of this lane's chunks, from the start of the product
    __device__ __forceinline__ int kc() const { return ((threadIdx.x & 7) ^ ((threadIdx.x >> 4) & 7)) * 8; }
    template <int ROWS> __device__ __forceinline__ void begin(int row0)
    {
#pragma unroll
        for (int i = 0; i < loads2<ROWS, NT>(); ++i) {
            int r = row0 + (int)(threadIdx.x >> 3) + NT / 8 * i;
            r = r < rows ? r : rows - 1; // rows past the end only feed C rows that are never stored
            voff[i] = ((uint32_t)r * (uint32_t)ld + (uint32_t)kc()) * 2u;
        }
        k = 0;
    }
    template <int ROWS> __device__ __forceinline__ void next() { k += BK; }
    template <int ROWS> __device__ __forceinline__ void issue(int i, uint32_t lds) const
    {
        if (!mine2<ROWS, NT>(i)) return;
        const char *b = base + (size_t)k * 2;
        if (k + BK <= K) dev::lds_dma16(voff[i], uniform64(b), chunk_lds2<NT>(lds, i));
        else dev::lds_dma16(k + kc() < K ? (const void *)(b + voff[i]) : (const void *)g_zero_chunk, chunk_lds2<NT>(lds, i));
    }
};
// RC: rows contiguous, K strides
template <int NT> struct DenseRCT {
    static constexpr bool KC = false;
    const char *base;
    int ld, rows, K;
    uint32_t voff; // this lane's first chunk, bytes from the K tile's start
    int k;
    template <int ROWS> __device__ __forceinline__ void begin(int row0)
    {
        constexpr int CPR = ROWS / 8;
        const int kr = threadIdx.x / CPR, pc = threadIdx.x % CPR;
        int r = row0 + ((pc ^ mma::rc_swizzle<ROWS>(kr)) << 3);
        r = r < rows ? r : rows - 8;
        voff = ((uint32_t)kr * (uint32_t)ld + (uint32_t)r) * 2u;
        k = 0;
    }
    template <int ROWS> __device__ __forceinline__ void next() { k += BK; }
    template <int ROWS> __device__ __forceinline__ void issue(int i, uint32_t lds) const
    {
        constexpr int CPR = ROWS / 8, KR = NT / CPR;
        const char *b = base + (size_t)(k + i * KR) * (size_t)ld * 2;
        if (k + BK <= K) dev::lds_dma16(voff, uniform64(b), chunk_lds2<NT>(lds, i));
        else dev::lds_dma16(k + i * KR + (int)(threadIdx.x / CPR) < K ? (const void *)(b + voff) : (const void *)g_zero_chunk, chunk_lds2<NT>(lds, i));
    }
};

using DenseKC2 = DenseKCT<kThreads2>;
using DenseRC2 = DenseRCT<kThreads2>;

// LDS of a product on BM x 256 tiles: two stages, later the strips of the write-out
template <int BM> constexpr size_t smem_bytes2() { return 2 * (size_t)(BM + BN2) * BK * 2; }
static_assert(smem_bytes2<BM2>() == kSmemBytes && 8 * mma::kStripBytes <= smem_bytes2<64>(), "stages and strips");

// C tile (m0, n0) of C = A B on WM x WN waves and NS stages of LDS; smem: NS (BM + BN) 128 bytes, 16-byte aligned.
template <bool OUT_BF16, bool VEC_STORE, int BM, int BN, int WM, int WN, int NS, class LA, class LB>
__device__ __forceinline__ void tile_product(LA &la, LB &lb, void *Cv, int ldc, int M, int N, int K, int m0, int n0, bool relu, char *smem,
                                             bool nts = true)
{
    constexpr int NT = WM * WN * 64, TM = BM / WM / 16, TN = BN / WN / 16;
    static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0 && (LA::KC || 512 % BM == 0), "tile sides");
    static_assert(WM * WN * mma::kStripBytes <= NS * (BM + BN) * BK * 2, "strips");
    constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2, NA = loads2<BM, NT>(), NL = NA + loads2<BN, NT>();
    constexpr bool UNEVEN = BM * 8 % NT != 0; // a wave may have a chunk less than NL in a tile
    static_assert(!UNEVEN || NS == 2, "counted waits");
    constexpr bool SPREAD = (!LA::KC && !LB::KC) || NS > 2;
    constexpr bool PLAIN_STEP = BM == 64 && NT == 512;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave / WN) * (TM * 16), wn0 = (wave % WN) * (TN * 16);
    const uint32_t lds0 = dev::lds_addr(smem);
    const int nk = (K + BK - 1) / BK;
    auto issue = [&](int i, uint32_t stage) {
        if (i < NA) la.template issue<BM>(i, stage);
        else lb.template issue<BN>(i - NA, stage + A_BYTES);
    };
    auto next = [&](bool more) { // past the end of K the last tile is fetched again, so that the wait counts stay the same
        if (more) {
            la.template next<BM>();
            lb.template next<BN>();
        }
    };
    mma::Reader<BM, LA::KC, TM> ra;
    mma::Reader<BN, LB::KC, TN> rb;
    ra.init(wm0, lane);
    rb.init(wn0, lane);
    mma::Frags<TM, TN> f0, f1;
    core::f32x4 acc[TM][TN];
    mma::clear(acc);
    la.template begin<BM>(m0);
    lb.template begin<BN>(n0);
    if constexpr (PLAIN_STEP) {
        // four waves per SIMD cover each other's reads: a tile's fragments when it has landed, the next tile on its way meanwhile.
        // (What a tile waits for is its predecessor's loads, so what stands in front of these is kept short.)
#pragma unroll
        for (int i = 0; i < NL; ++i) issue(i, lds0);
        for (int kt = 0; kt < nk; ++kt) {
            next(kt + 1 < nk);                              // (its divisions while the tile is still on its way)
            __builtin_amdgcn_s_waitcnt(mma::waitcnt_vm(0)); // this wave's chunks of the tile have landed
            __syncthreads();                                // everyone's have; everyone is done reading the other stage
            if (kt + 1 < nk) {
#pragma unroll
                for (int i = 0; i < NL; ++i) issue(i, lds0 + (uint32_t)((kt & 1) ^ 1) * STAGE);
            }
            const char *At = smem + (kt & 1) * STAGE;
            __builtin_amdgcn_sched_barrier(0);
            mma::read_frags(f0, ra, rb, At, At + A_BYTES, 0);
            mma::k_step<0, false>(acc, f0, f1, ra, rb, At, At + A_BYTES, 1, [](int) {});
            mma::multiply(acc, f1);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            if (st > 0) next(st < nk);
#pragma unroll
            for (int i = 0; i < NL; ++i) issue(i, lds0 + (uint32_t)st * STAGE);
        }

        __builtin_amdgcn_s_waitcnt(mma::waitcnt_vm((NS - 1) * NL - UNEVEN)); // this wave's chunks of the first tiles have landed
        __syncthreads();                                                     // everyone's have
        mma::read_frags(f0, ra, rb, smem, smem + A_BYTES, 0);

        int cs = 0;
        for (int kt = 0; kt < nk; ++kt) {
            const char *At = smem + cs * STAGE;
            mma::k_step<0, SPREAD>(acc, f0, f1, ra, rb, At, At + A_BYTES, 1, [](int) {});
            // this wave has read the tile and its chunks of the next one have landed; then everyone's
            __builtin_amdgcn_s_waitcnt(mma::waitcnt_vm_lds((NS - 2) * NL));
            __syncthreads();
            next(kt + NS < nk);
            const uint32_t lds_free = lds0 + (uint32_t)cs * STAGE;
            cs = cs + 1 == NS ? 0 : cs + 1;
            const char *nA = smem + cs * STAGE;
            mma::k_step<NL, SPREAD>(acc, f1, f0, ra, rb, nA, nA + A_BYTES, 0, [&](int i) { issue(i, lds_free); });
        }
    }
    // the re-fetches have landed and all fragment reads are done before the stages are reused
    __builtin_amdgcn_s_waitcnt(mma::waitcnt_vm_lds(0));
    __syncthreads();
    mma::store_block<OUT_BF16, VEC_STORE>(acc, smem + wave * mma::kStripBytes, Cv, ldc, m0 + wm0, n0 + wn0, M, N, relu, lane, nts);
}

// ... on BM x 256 tiles; 512 threads; smem: smem_bytes2<BM>(), 16-byte aligned.
// BM < 256: products with few rows, whose 256-row tile would take in and multiply rows that do not exist, and products whose
// tiles come out at better numbers (conv.hip).
template <bool OUT_BF16, bool VEC_STORE, int BM = BM2, class LA, class LB>
__device__ __forceinline__ void tile_product2(LA &la, LB &lb, void *Cv, int ldc, int M, int N, int K, int m0,
                                              int n0, bool relu, char *smem, bool nts = true)
{
    tile_product<OUT_BF16, VEC_STORE, BM, BN2, 2, 4, 2>(la, lb, Cv, ldc, M, N, K, m0, n0, relu, smem, nts);
}

} // namespace core2
} // namespace tt
