// Sixth bf16 MFMA tile engine: launches of at most one 256 x 128 tile per CU (one row of tiles at batch 256: the forward
// products and data gradients of the classifiers, bound by streaming the weights once from HBM next to a small operand that
// every workgroup takes in from L2; products whose K is cut).
//
//   - 256 x 128 output tiles, four waves as 2 x 2, 128 x 64 per wave, one workgroup and so one wave per SIMD: nothing else
//     runs while a wave waits, so its reads, loads and MFMAs are laid out by hand (gemm_mma.h), the loads spread over the
//     whole k-step (in its second half: 8 x (256 x 3136 x 4096) 53 instead of 48 us);
//   - K tiles of 64: a lane group of eight fetches one whole 128-byte line of a K-contiguous row (the K tiles of 32 of
//     gemm_core4.h fetch half lines: 58 us);
//   - three stages of 48 KB: two tiles on their way.  More of the streamed operand on its way loses: with two stages of the
//     one and six of the other, each loaded by two waves of their own, 87 us instead of 68 where the weights come from HBM,
//     and three and four the same 68;
//   - at most 256 registers per lane: given 512, the compiler moves accumulators between the two halves of the file (75 us);
//   - LDS layouts of gemm_core2.h; the last K tile may be short.
// 8 x (256 x 3136 x 4096) A B^T, weights in the memory-side cache 64.1 -> 48.4 us, from HBM 71 -> 68 (3.0 TB/s of weights);
// 8 x (256 x 4096 x 3136) A B 58 -> 50, from HBM 72 -> 60 (gemm_core4.h before it also ran on gemm_mma.h).
#pragma once
#include <cstdint>
#include "tt_device.h"
#include "gemm_core.h"
#include "gemm_core2.h"
#include "gemm_core3.h"
#include "gemm_core4.h"
#include "gemm_mma.h"

namespace tt {
namespace core6 {

using core::bf16x8;

constexpr int kThreads6 = 256;
constexpr int BM6 = 256, BN6 = 128, BK6 = 64, NS6 = 3;
constexpr int kABytes6 = BM6 * BK6 * 2, kBBytes6 = BN6 * BK6 * 2, kStage6 = kABytes6 + kBBytes6; // 32 KB and 16 KB
constexpr size_t kSmem6 = (size_t)NS6 * kStage6;                                             // 144 KB
constexpr int kLoadsA6 = kABytes6 / 16 / kThreads6, kLoadsB6 = kBBytes6 / 16 / kThreads6;    // 8 and 4 per thread

// lane offsets of this thread's 16-byte chunks of one operand tile (ROWS x 64).  K contiguous: chunk c = tid + 256 i lies
// in row c / 8 = tid / 8 + 32 i at position c % 8 and holds k-chunk position ^ ((row >> 1) & 7), which does not depend on
// i.  Rows contiguous (the layout of gemm_core2.h / gemm_core4.h): chunk c lies in k-row c / CPR = tid / CPR + KPI i at
// position c % CPR and holds row-chunk position ^ ((k & 3) << 1); KPI is a multiple of 4, so that does not depend on i.
template <int ROWS, bool KC> __device__ __forceinline__ void chunk_offsets6(int row0, int rows, int ld, uint32_t *voff)
{
    const int tid = threadIdx.x;
    constexpr int NL = ROWS * BK6 * 2 / 16 / kThreads6;
    if constexpr (KC) {
        const int rl = tid >> 3;
        const int kc = (tid & 7) ^ ((rl >> 1) & 7);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            int r = row0 + rl + 32 * i;
            r = r < rows ? r : rows - 1; // rows past the end only feed C rows / columns that are never stored
            voff[i] = (uint32_t)r * (uint32_t)ld * 2u + (uint32_t)kc * 16u;
        }
    } else {
        constexpr int CPR = ROWS / 8;
        constexpr int KPI = kThreads6 / CPR;
        static_assert(KPI % 4 == 0 && KPI * NL == BK6, "k-rows per load");
        const int kl = tid / CPR;
        const int rc = (tid % CPR) ^ ((kl & 3) << 1);
        int r = row0 + rc * 8;
        r = r < rows ? r : rows - 8;
#pragma unroll
        for (int i = 0; i < NL; ++i) voff[i] = (uint32_t)(kl + KPI * i) * (uint32_t)ld * 2u + (uint32_t)r * 2u;
    }
}

// k of this thread's chunk i inside its tile
template <int ROWS, bool KC> __device__ __forceinline__ int k_of(int i)
{
    if constexpr (KC) return (int)((threadIdx.x & 7) ^ ((threadIdx.x >> 4) & 7)) * 8;
    else return (int)threadIdx.x / (ROWS / 8) + kThreads6 / (ROWS / 8) * i;
}

// C tile (m0, n0) of C = A B over K = klen (TAIL: no multiple of 64, what is missing is read as zeros) starting at the operands' k = 0 as given by abase / bbase;
// A is M x K with pitch lda (A_KC) or K x M, B is N x K with pitch ldb (B_KC) or K x N (rows contiguous: fragments through
// LDS transpose reads).  256 threads; smem: kSmem6 bytes, 16-byte aligned.  STAGED: rows of C take 16-byte stores.
template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL>
__device__ __forceinline__ void tile_product6(const char *abase, int lda, const char *bbase, int ldb, void *Cv, int ldc, int M,
                                              int N, int klen, int m0, int n0, bool relu, char *smem, bool nts = true)
{
    constexpr int TM = 8, TN = 4, WN = 2; // 2 x 2 waves, 128 x 64 per wave
    constexpr int LPS = kLoadsA6 + kLoadsB6;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave / WN) * (TM * 16), wn0 = (wave % WN) * (TN * 16);
    const uint32_t lds0 = dev::lds_addr(smem);

    uint32_t voa[kLoadsA6], vob[kLoadsB6];
    chunk_offsets6<BM6, A_KC>(m0, M, lda, voa);
    chunk_offsets6<BN6, B_KC>(n0, N, ldb, vob);
    const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 1024u;
    const uint64_t astep = A_KC ? (uint64_t)BK6 * 2 : (uint64_t)BK6 * (uint64_t)lda * 2;
    const uint64_t bstep = B_KC ? (uint64_t)BK6 * 2 : (uint64_t)BK6 * (uint64_t)ldb * 2;
    const int nk = (klen + BK6 - 1) / BK6, tail = klen - (nk - 1) * BK6; // K tiles, values of K in the last one

    // Rows contiguous and a tail, whose selects need registers: one lane offset per operand, a chunk's k-row is part of the scalar base
    // (with an offset per chunk A^T B spilled, and a reload's wait is one for every load on its way: 8 x (1024 x 1024 x 2056) 58 us, now
    // 44, 8 x (512 x 1024 x 4104) 98, now 68)
    constexpr bool ONE_A = TAIL && !A_KC, ONE_B = TAIL && !B_KC;
    const uint64_t arow = ONE_A ? (uint64_t)(kThreads6 / (BM6 / 8)) * (uint64_t)lda * 2 : 0;
    const uint64_t brow = ONE_B ? (uint64_t)(kThreads6 / (BN6 / 8)) * (uint64_t)ldb * 2 : 0;

    // K tile to ask for next; past the end the last one is fetched again, so that the wait counts stay the same
    uint64_t ab = core2::uniform64(abase), bb = core2::uniform64(bbase);
    int left = nk - 1;
    auto issue_one = [&](int i, uint32_t stage) {
        // (a select per lane in every tile, not a branch in front of the last: branches cut the k-step's schedule up)
        const int in = TAIL && left <= 0 ? tail : BK6;
        if (i < kLoadsA6) core2::chunk_or_zero(voa[ONE_A ? 0 : i], ab + i * arow, !TAIL || k_of<BM6, A_KC>(i) < in, TAIL,
                                               stage + wave_lds + (uint32_t)i * (kThreads6 * 16u));
        else core2::chunk_or_zero(vob[ONE_B ? 0 : i - kLoadsA6], bb + (i - kLoadsA6) * brow, !TAIL || k_of<BN6, B_KC>(i - kLoadsA6) < in, TAIL,
                                  stage + kABytes6 + wave_lds + (uint32_t)(i - kLoadsA6) * (kThreads6 * 16u));
    };
    auto advance = [&]() {
        if (left > 0) {
            ab += astep;
            bb += bstep;
        }
        --left;
    };
#pragma unroll
    for (int st = 0; st < NS6; ++st) {
#pragma unroll
        for (int i = 0; i < LPS; ++i) issue_one(i, lds0 + (uint32_t)st * kStage6);
        advance();
    }

    mma::Reader<BM6, A_KC, TM> ra;
    mma::Reader<BN6, B_KC, TN> rb;
    ra.init(wm0, lane);
    rb.init(wn0, lane);
    mma::Frags<TM, TN> f0, f1;
    core::f32x4 acc[TM][TN];
    mma::clear(acc);
    __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm((NS6 - 1) * LPS)); // this wave's chunks of the first tiles have landed
    __syncthreads();                                                // everyone's have
    mma::read_frags(f0, ra, rb, smem, smem + kABytes6, 0);

    int cs = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const char *At = smem + cs * kStage6;
        mma::k_step<0, true>(acc, f0, f1, ra, rb, At, At + kABytes6, 1, [](int) {});
        // this wave has read the item and its chunks of the next one have landed; then everyone's
        __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm_lds((NS6 - 2) * LPS));
        __syncthreads();
        const uint32_t lds_free = lds0 + (uint32_t)cs * kStage6;
        cs = cs + 1 == NS6 ? 0 : cs + 1;
        const char *nA = smem + cs * kStage6;
        mma::k_step<LPS, true>(acc, f1, f0, ra, rb, nA, nA + kABytes6, 0, [&](int i) { issue_one(i, lds_free); });
        advance();
    }
    // the re-fetches issued past the end have landed and every wave is done with the ring: it can be reused / given up
    __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm_lds(0));
    __syncthreads();
    mma::store_block<OUT_BF16, STAGED>(acc, smem + wave * mma::kStripBytes, Cv, ldc, m0 + wm0, n0 + wn0, M, N, relu, lane, nts);
}

} // namespace core6
} // namespace tt
