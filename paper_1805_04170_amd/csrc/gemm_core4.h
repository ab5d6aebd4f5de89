// Fourth bf16 MFMA tile engine: 256 x 128 output tiles, four waves, TWO workgroups resident per CU.
//
// The engines with one 256 x 256 workgroup per CU run their phases one after the other on a CU: fill the pipeline,
// multiply, write the tile out.  For products with a short K loop and a large output (the weight gradients at batch
// 256: four 64-deep K tiles per 128 KB output tile) the write-out is as long as the multiplication.  Here a workgroup
// needs half the registers and less than half the LDS of a CU, so two of them share it and the hardware interleaves
// them: while one stores its tile the other one multiplies.
//
//   - four waves as 2 x 2, 128 x 64 per wave (the same wave tile as the 256 x 256 engines);
//   - K tiles of 32; a stage is 16 KB of A and 8 KB of B; three stages (72 KB) fetched global -> LDS with
//     global_load_lds_dwordx4 two tiles ahead (inline assembly, see gemm_core2.h for why);
//   - LDS layouts: K-contiguous operands as [row][4 chunks of 8 k], chunk position p of row r holds k-chunk
//     p ^ (-(r >> 2) & 3) (LDS serves a 16-byte read of lanes 0-3, 12-15 and 20-27 together: p ^ ((r >> 2) & 3) conflicts, 307
//     instead of 466 GB/s); row-contiguous operands as [k][ROWS / 8 chunks of 8 rows], swizzled and read with LDS
//     transpose reads as in gemm_core2.h;
//   - fragments, k-steps and write-out of gemm_mma.h, a K tile being one k-step.  8 x (256 x 4608 x 1024) A B^T, 288 tiles:
//     32.9 -> 30.3 us (31.3 on gemm_core6.h); where tiles leave CUs empty gemm_core6.h is the faster one;
//   - the last K tile may be short; a workgroup computes one tile and ends (the other resident workgroup and the next
//     one queued cover its start-up and wind-down).
#pragma once
#include <cstdint>
#include "tt_device.h"
#include "gemm_core.h"
#include "gemm_core2.h"
#include "gemm_core3.h"
#include "gemm_mma.h"

namespace tt {
namespace core4 {

constexpr int kThreads4 = 256;
constexpr int BM4 = 256, BN4 = 128, BK4 = 32, NS4 = 3;
constexpr int kABytes = BM4 * BK4 * 2, kBBytes = BN4 * BK4 * 2, kStage4 = kABytes + kBBytes; // 16 KB + 8 KB
constexpr size_t kSmem4 = (size_t)NS4 * kStage4;                                              // 72 KB
constexpr int kLoadsA = kABytes / 16 / kThreads4, kLoadsB = kBBytes / 16 / kThreads4;        // 4 and 2 per thread

using core2::uniform64;

// lane offsets of this thread's 16-byte chunks of one operand tile (ROWS x 32), see the layouts above
template <int ROWS, bool KC> __device__ __forceinline__ void chunk_offsets(int row0, int rows, int ld, uint32_t *voff)
{
    const int tid = threadIdx.x;
    constexpr int NL = ROWS * BK4 * 2 / 16 / kThreads4;
    if constexpr (KC) {
        // chunk c = tid + 256 i: row c / 4 = tid / 4 + 64 i, position c % 4
        const int rl = tid >> 2;
        const int kc = (tid & 3) ^ (-(rl >> 2) & 3);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            int r = row0 + rl + 64 * i;
            r = r < rows ? r : rows - 1; // rows past the end only feed C rows / columns that are never stored
            voff[i] = (uint32_t)r * (uint32_t)ld * 2u + (uint32_t)kc * 16u;
        }
    } else {
        // chunk c = tid + 256 i: k-row c / CPR, position c % CPR holds row-chunk position ^ ((k & 3) << 1)
        constexpr int CPR = ROWS / 8;           // 32 or 16 chunks per k-row
        constexpr int KPI = kThreads4 / CPR;    // k-rows covered per i: 8 or 16 (multiples of 4: k & 3 does not depend on i)
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
    if constexpr (KC) return (int)((threadIdx.x & 3) ^ (-(threadIdx.x >> 4) & 3)) * 8;
    else return (int)threadIdx.x / (ROWS / 8) + kThreads4 / (ROWS / 8) * i;
}

// TAIL: klen is no multiple of 32, what is missing is read as zeros
template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL = false>
__device__ __forceinline__ void tile_product4(const char *abase, int lda, const char *bbase, int ldb, void *Cv, int ldc, int M,
                                              int N, int klen, int m0, int n0, bool relu, char *smem, bool nts = true)
{
    constexpr int TM = 8, TN = 4, WN = 2; // 2 x 2 waves, 128 x 64 per wave
    constexpr int LPS = kLoadsA + kLoadsB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave / WN) * (TM * 16), wn0 = (wave % WN) * (TN * 16);
    const uint32_t lds0 = dev::lds_addr(smem);

    uint32_t voa[kLoadsA], vob[kLoadsB];
    chunk_offsets<BM4, A_KC>(m0, M, lda, voa);
    chunk_offsets<BN4, B_KC>(n0, N, ldb, vob);
    const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 1024u;
    const uint64_t astep = A_KC ? BK4 * 2u : (uint64_t)BK4 * (uint64_t)lda * 2u, bstep = B_KC ? BK4 * 2u : (uint64_t)BK4 * (uint64_t)ldb * 2u;
    const int nk = (klen + BK4 - 1) / BK4, tail = klen - (nk - 1) * BK4; // K tiles, values of K in the last one

    // K tile to ask for next; past the end the last one is fetched again, so that the wait counts stay the same
    uint64_t ab = uniform64(abase), bb = uniform64(bbase);
    int left = nk - 1;
    auto issue_one = [&](int i, uint32_t stage) {
        // (a select per lane in every tile, not a branch in front of the last: branches cut the k-step's schedule up)
        const int in = TAIL && left <= 0 ? tail : BK4;
        if (i < kLoadsA) core2::chunk_or_zero(voa[i], ab, !TAIL || k_of<BM4, A_KC>(i) < in, TAIL, stage + wave_lds + (uint32_t)i * (kThreads4 * 16u));
        else core2::chunk_or_zero(vob[i - kLoadsA], bb, !TAIL || k_of<BN4, B_KC>(i - kLoadsA) < in, TAIL,
                                  stage + kABytes + wave_lds + (uint32_t)(i - kLoadsA) * (kThreads4 * 16u));
    };
    auto advance = [&]() {
        if (left > 0) {
            ab += astep;
            bb += bstep;
        }
        --left;
    };
#pragma unroll
    for (int st = 0; st < NS4; ++st) {
#pragma unroll
        for (int i = 0; i < LPS; ++i) issue_one(i, lds0 + (uint32_t)st * kStage4);
        advance();
    }

    mma::Reader<BM4, A_KC, TM, BK4> ra;
    mma::Reader<BN4, B_KC, TN, BK4> rb;
    ra.init(wm0, lane);
    rb.init(wn0, lane);
    mma::Frags<TM, TN> f0, f1;
    core::f32x4 acc[TM][TN];
    mma::clear(acc);
    __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm((NS4 - 1) * LPS)); // this wave's chunks of the first tiles have landed
    __syncthreads();                                                // everyone's have
    mma::read_frags(f0, ra, rb, smem, smem + kABytes, 0);

    int cs = 0;
    // multiplies the fragments cur of K tile kt, reads those of the next tile and asks for the one that takes this one's stage
    auto item = [&](const mma::Frags<TM, TN> &cur, mma::Frags<TM, TN> &nxt) {
        // this wave has read its fragments and its chunks of the next tile have landed; then everyone's
        __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm_lds((NS4 - 2) * LPS));
        __syncthreads();
        const uint32_t lds_free = lds0 + (uint32_t)cs * kStage4;
        cs = cs + 1 == NS4 ? 0 : cs + 1;
        const char *nA = smem + cs * kStage4;
        mma::k_step<LPS, true>(acc, cur, nxt, ra, rb, nA, nA + kABytes, 0, [&](int i) { issue_one(i, lds_free); });
        advance();
    };
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        item(f0, f1);
        item(f1, f0);
    }
    if (kt < nk) item(f0, f1);
    // the re-fetches issued past the end have landed and every wave is done with the ring: it can be reused / given up
    __builtin_amdgcn_s_waitcnt(core3::waitcnt_vm_lds(0));
    __syncthreads();
    mma::store_block<OUT_BF16, STAGED>(acc, smem + wave * mma::kStripBytes, Cv, ldc, m0 + wm0, n0 + wn0, M, N, relu, lane, nts);
}

} // namespace core4
} // namespace tt
