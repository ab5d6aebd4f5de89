// Third bf16 MFMA tile engine: persistent and software-pipelined, operand tiles straight into LDS.
//
// One workgroup of eight waves stays on its CU and walks a list of 256 x 256 output tiles.  The K tiles (64 deep) of ALL its
// output tiles form one stream of work items; operand tiles are fetched global -> LDS (global_load_lds_dwordx4) through a
// ring of two LDS stages, so the first K tiles of the next output tile are already on their way while the current one is
// finished and written out.  An item is two k-steps of 32 (gemm_mma.h): the first multiplies the fragments read last and reads
// the item's other half; then the next item's tiles must have landed (the one s_waitcnt + barrier of an item), and the
// second reads its first half and fetches the item after it into the stage that everyone has now read.
//
// What bounds it: power.  One product of 2048 x 8192 x 8192 takes 184 us on random values and 157 on zeros; with 32 x 32 x 16
// MFMAs, fragments read where they are used, it took 218.
//
// Ring shape: two stages of 64 measured best; thinner, deeper rings (BK = 32, four or five stages) fetch half lines of a
// K-contiguous operand and lose 10 % (gemm_mma.h).
//
// LDS layouts follow gemm_core2.h, and so do the loads (inline assembly, a scalar base and a 32-bit lane offset, computed once per
// output tile; the builtin form makes the compiler put s_waitcnt vmcnt(0) in front of every fragment read).  Differences:
//   - K must be a multiple of 64 (no tail handling in the K direction; the launcher falls back otherwise);
//   - results go through a small wave-private LDS strip that lies outside the ring, so the epilogue needs no workgroup
//     barrier and never touches a stage that a prefetch may be filling.
#pragma once
#include <cstdint>
#include "tt_device.h"
#include "gemm_core.h"
#include "gemm_core2.h"
#include "gemm_mma.h"

namespace tt {
namespace core3 {

using core::bf16x8;
using core::f32x4;

constexpr int kThreads3 = 512;
constexpr int BM3 = 256, BN3 = 256;

constexpr int kOpBytes3 = 256 * 64 * 2, kStage3 = 2 * kOpBytes3; // one operand's tile, one stage
constexpr int kLoads3 = kOpBytes3 / 16 / kThreads3;             // 16-byte chunks per thread and operand

template <int BK, int NS, bool STAGED> constexpr size_t smem_bytes3() { return (size_t)NS * kStage3 + 8 * mma::kStripBytes; }

struct Params3 {
    const void *A[64];
    const void *B[64];
    void *C[64];
    int32_t M, N, K;
    int32_t lda, ldb, ldc;
    int32_t tiles_m, tiles_n;
    int32_t per_xcd;     // logical output tiles per XCD
    int32_t wg_per_xcd;  // resident workgroups per XCD (grid = 8 * wg_per_xcd)
    int32_t total;       // tiles_m * tiles_n * count * ksplit
    int32_t relu;
    int32_t nts;         // non-temporal stores
    int32_t ksplit, kchunk;
    int32_t nred, parts; // RUNS (below): shards per output block, runs their K tiles are cut into
};

// position of one output tile
struct TilePos {
    int vshard, shard, m0, n0, kbeg, klen;
};

// j-th output tile of this workgroup; false when the list is exhausted
//   RUNS = false: one item per shard (and K chunk of it).
//   RUNS = true: shards blk * nred .. + nred - 1 add up into output block blk.  Their K tiles, one shard's after the
//   other's, are cut into `parts` runs of equal length (to a tile) that need not end where a shard does; run c of block b
//   writes C[b * parts + c].
template <bool RUNS = false> __device__ __forceinline__ bool tile_of(const Params3 &p, int j, TilePos *t)
{
    const int bid = blockIdx.x;
    const int li = bid / core::kXcds + j * p.wg_per_xcd;
    const int logical = (bid % core::kXcds) * p.per_xcd + li;
    if (li >= p.per_xcd || logical >= p.total) return false;
    const int tiles = p.tiles_m * p.tiles_n;
    t->vshard = logical / tiles;
    const int r = logical - t->vshard * tiles;
    int tm, tn;
    core::grouped_tile(r, p.tiles_m, p.tiles_n, &tm, &tn);
    t->m0 = tm * BM3;
    t->n0 = tn * BN3;
    if constexpr (RUNS) {
        const int seg = p.K / 64, all = seg * p.nred; // K tiles of a shard, of a block
        const int blk = t->vshard / p.parts, part = t->vshard - blk * p.parts;
        const int first = part * all / p.parts, end = (part + 1) * all / p.parts, q = first / seg;
        t->shard = blk * p.nred + q;
        t->kbeg = (first - q * seg) * 64;
        t->klen = (end - first) * 64;
        return true;
    }
    t->shard = t->vshard / p.ksplit;
    t->kbeg = (t->vshard - t->shard * p.ksplit) * p.kchunk;
    t->klen = p.K - t->kbeg < p.kchunk ? p.K - t->kbeg : p.kchunk;
    return true;
}

// Stream of operand tiles of one operand over the whole work list of the workgroup.
//   KC = true : operand rows (m for A, n for B) have K contiguous (leading dimension ld = K extent of the matrix)
//   KC = false: K rows of the matrix are contiguous over the operand's rows (ld = row extent)
template <bool KC, bool IS_A, bool RUNS = false> struct Feeder {
    static constexpr int NL = kLoads3;
    uint32_t voff[NL];  // lane part of the address of this thread's chunks
    const char *base;   // wave-uniform part: start of the current K tile
    uint32_t kstep;     // bytes from one K tile to the next
    int kt, nk, j;      // K tile inside the output tile, their number, ordinal of the output tile
    int left, shard;    // RUNS: K tiles of the current shard from the current one on, the shard
    bool live;

    __device__ __forceinline__ void bind(const Params3 &p, const TilePos &t)
    {
        const int tid = threadIdx.x;
        const void *mat = IS_A ? p.A[t.shard] : p.B[t.shard];
        const int ld = IS_A ? p.lda : p.ldb;
        const int rows = IS_A ? p.M : p.N;
        const int row0 = IS_A ? t.m0 : t.n0;
        if constexpr (KC) {
            // chunk c = tid + 512 i of the tile: row c / 8, position c % 8; the position holds k-chunk position ^ swizzle(row)
            base = reinterpret_cast<const char *>(mat) + (size_t)t.kbeg * 2;
            kstep = 64 * 2;
            const int rl = tid >> 3; // row of chunk i = rl + 64 i
            const int kc = (tid & 7) ^ ((rl >> 1) & 7);
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                int r = row0 + rl + 64 * i;
                r = r < rows ? r : rows - 1; // rows past the end only feed C rows that are never stored
                voff[i] = (uint32_t)r * (uint32_t)ld * 2u + (uint32_t)kc * 16u;
            }
        } else {
            // chunk c: k-row c / 32, position c % 32 holds row-chunk position ^ ((k & 3) << 1)
            base = reinterpret_cast<const char *>(mat) + (size_t)t.kbeg * (size_t)ld * 2;
            kstep = 64u * (uint32_t)ld * 2u;
            const int rc = (tid & 31) ^ (((tid >> 5) & 3) << 1);
            int r = row0 + rc * 8;
            r = r < rows ? r : rows - 8;
#pragma unroll
            for (int i = 0; i < NL; ++i)
                voff[i] = (uint32_t)((tid >> 5) + 16 * i) * (uint32_t)ld * 2u + (uint32_t)r * 2u;
        }
        kt = 0;
        nk = t.klen / 64;
        if constexpr (RUNS) {
            left = (p.K - t.kbeg) / 64;
            shard = t.shard;
        }
    }

    __device__ __forceinline__ void start(const Params3 &p)
    {
        TilePos t;
        j = 0;
        live = tile_of<RUNS>(p, 0, &t);
        if (live) bind(p, t);
    }

    // Fetch chunk i (of NL) of the current K tile into the stage at LDS address lds (wave-uniform).
    __device__ __forceinline__ void issue_one(int i, uint32_t lds) const
    {
        const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // the base is wave-uniform by construction; say so, or the "s" operand may be handed a vector register pair
        // (readfirstlane returns a signed int: go through uint32_t so the low half is not sign-extended)
        const uint64_t b64 = reinterpret_cast<uint64_t>(base);
        const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b64);
        const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b64 >> 32));
        const uint64_t sbase = ((uint64_t)b_hi << 32) | (uint64_t)b_lo;
        const uint32_t dst = lds + (wave * 64u + (uint32_t)i * kThreads3) * 16u;
        dev::lds_dma16(voff[i], sbase, dst);
    }

    // Move on to the next K tile.  Past the end of the list the last K tile stays current and is fetched again (into a
    // stage nobody reads), so every item issues the same number of loads and the wait count of the main loop stays
    // constant.
    __device__ __forceinline__ void advance(const Params3 &p)
    {
        if (!live) return;
        if (kt + 1 < nk) {
            ++kt;
            base += kstep;
            if constexpr (RUNS)
                if (--left == 0) { // the run goes on in the next shard: same rows, same pitch, another matrix
                    ++shard;
                    base = reinterpret_cast<const char *>(IS_A ? p.A[shard] : p.B[shard]);
                    left = p.K / 64;
                }
            return;
        }
        TilePos t;
        if (tile_of<RUNS>(p, j + 1, &t)) {
            ++j;
            bind(p, t);
        } else {
            live = false; // keep pointing at the last K tile
        }
    }

    __device__ __forceinline__ void issue_and_advance(const Params3 &p, uint32_t lds)
    {
#pragma unroll
        for (int i = 0; i < NL; ++i) issue_one(i, lds);
        advance(p);
    }
};

using mma::waitcnt_vm;
using mma::waitcnt_vm_lds;

// SPREAD: loads over the whole second k-step of an item instead of its second half
template <int BK, int NS, bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool SPREAD, bool RUNS = false>
__device__ __forceinline__ void run_tiles(const Params3 &p, char *smem)
{
    static_assert(NS == 2 && BK == 64, "ring shape");
    constexpr int TM = 8, TN = 4, WN = 4; // 2 x 4 waves, 128 x 64 per wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave / WN) * (TM * 16), wn0 = (wave % WN) * (TN * 16);
    const uint32_t lds0 = dev::lds_addr(smem);

    Feeder<A_KC, true, RUNS> fa;
    Feeder<B_KC, false, RUNS> fb;
    fa.start(p);
    fb.start(p);
    TilePos cur;
    int jc = 0;
    if (!tile_of<RUNS>(p, 0, &cur)) return; // no work for this workgroup (uniform)
    fa.issue_and_advance(p, lds0);
    fb.issue_and_advance(p, lds0 + kOpBytes3);
    fa.issue_and_advance(p, lds0 + kStage3);
    fb.issue_and_advance(p, lds0 + kStage3 + kOpBytes3);

    mma::Reader<256, A_KC, TM> ra;
    mma::Reader<256, B_KC, TN> rb;
    ra.init(wm0, lane);
    rb.init(wn0, lane);
    mma::Frags<TM, TN> f0, f1;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoads3)); // this wave's chunks of the first item have landed
    __syncthreads();                                     // everyone's have
    mma::read_frags(f0, ra, rb, smem, smem + kOpBytes3, 0);

    int cs = 0; // stage of the item being multiplied
    const bool relu = p.relu != 0;
    for (;;) {
        f32x4 acc[TM][TN];
        mma::clear(acc);
        const int nk = cur.klen / 64;
        for (int kt = 0; kt < nk; ++kt) {
            const char *At = smem + cs * kStage3;
            mma::k_step<0, false>(acc, f0, f1, ra, rb, At, At + kOpBytes3, 1, [](int) {});
            // this wave has read the item and its chunks of the next one have landed; then everyone's
            __builtin_amdgcn_s_waitcnt(waitcnt_vm_lds(0));
            __syncthreads();
            const uint32_t lds_free = lds0 + (uint32_t)cs * kStage3;
            cs ^= 1;
            const char *nA = smem + cs * kStage3;
            mma::k_step<2 * kLoads3, SPREAD>(acc, f1, f0, ra, rb, nA, nA + kOpBytes3, 0, [&](int i) {
                if (i < kLoads3) fa.issue_one(i, lds_free);
                else fb.issue_one(i - kLoads3, lds_free + kOpBytes3);
            });
            fa.advance(p);
            fb.advance(p);
        }
        mma::store_block<OUT_BF16, STAGED>(acc, smem + NS * kStage3 + wave * mma::kStripBytes, p.C[cur.vshard], p.ldc, cur.m0 + wm0,
                                           cur.n0 + wn0, p.M, p.N, relu, lane, p.nts != 0);
        ++jc;
        if (!tile_of<RUNS>(p, jc, &cur)) break;
    }
    // the re-fetches issued past the end of the list must have landed before the workgroup gives up its LDS
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
}

} // namespace core3
} // namespace tt
