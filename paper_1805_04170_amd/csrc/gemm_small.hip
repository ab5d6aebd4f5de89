// Shard products that the MFMA tile engines do not take: fp32, and bf16 whose rows are not whole 16-byte vectors, whose
// addresses are not multiples of 16 bytes, or of which one operand has 2^31 elements or more.  gemm_small_kernel
// (gemm_small.h): K cut over the waves of a workgroup.  gemm_ordered_kernel: K walked in order; short K, most of fp32, and the
// forward layout of bf16.
// One launch covers all shards (Sec. 5.2 step 2 of arXiv 1805.04170).
#include "tt_device.h"
#include <cstdint>
#include <type_traits>
#include "gemm_small.h"
#include "tt_internal.h"

namespace tt {
namespace {

using core::kXcds;

template <bool BF, bool A_KC, bool B_KC, int T, class OFF>
__global__ __launch_bounds__(small::waves_of<T>() * 64, T == 1 ? 2 : 1) void gemm_small_kernel(const small::ParamsS p)
{
    __shared__ __attribute__((aligned(16))) char lds[small::waves_of<T>() * small::lds_per_wave<BF, A_KC, B_KC, T>()];
    small::run_small<BF, A_KC, B_KC, T, OFF>(p, lds);
}

// Ordered products: every result is a chain of fp32 fused multiply-adds with K increasing, on fp32 matrix instructions.  Only
// bf16 A B, the forward layout, is one chain; elsewhere K is dealt out to four or eight chains in turn that are added pairwise
// at the end, since one chain of K terms rounds worse than the waves of gemm_small_kernel.  Relative error of fp32 results, there / here:
// fp32 K = 17, 129, 511, 1023 7.6e-8 / 5.6e-8, 1.5e-7 / 8.8e-8, 1.6e-7 / 1.5e-7, 2.1e-7 / 2.1e-7; bf16 A B^T and A^T B K = 33, 129, 255, 511 3.0e-8 /
// 3.0e-8, 6.0e-8 / 4.9e-8, 6.6e-8 / 5.8e-8, 7.2e-8 / 6.9e-8 (as one chain 3.6e-8, 7.3e-8, 1.1e-7, 1.6e-7).
// v_mfma_f32_16x16x4_f32 and v_mfma_f32_32x32x2_f32 add their four or two products to the accumulator one after the other,
// k increasing, each rounded like fmaf (compared bit for bit with chains of fmaf: normal, widely spread, subnormal operands;
// a bf16 value is an fp32 value), so the bits do not depend on the tile.
//
// Four waves, one block of S x S results each.  S = 16 is the shorter chain: a result waits 8 cycles per value of K (the
// instruction takes 32 for four), S = 32 32 cycles; per flop both cost the matrix unit the same, and the larger tile takes in
// half the operands.  KB values of K per step: global -> registers four steps ahead (pairs at any boundary of an element,
// untouched until their step, so that no load is waited for early), registers -> LDS as fp32, one barrier per step.
// bf16 A B, us, on 64 x 64 tiles of vector multiply-adds (or 32 x 32 ones, whose loads were waited for step by step) / so:
// 4 x (100 x 225 x 1500) 53 / 20, 1023^3 79 / 33, 8 x (257 x 255 x 255) 17.0 / 8.5, 4095 x 4093 x 2047 1312 / 669 (103 TFLOP/s of
// the unit's 157).
template <bool BF, bool KC, int S, int KB> struct OrderedSide {
    static constexpr int T = 2 * S, KM = 64 / S;                         // rows of the tile, K per instruction
    static constexpr int PT = T * KB / 2 / 256, W = BF ? 1 : 2;          // pairs per thread and step, words per pair
    static constexpr int ES = BF ? 2 : 4;
    // LDS: as stored, rows of K values or K rows of row values; the 64 values of a fragment lie in 64 banks
    static constexpr int PITCH = KC ? KB + KM : (S == 16 ? 48 : 96);
    static constexpr int LDS = (KC ? T : KB) * PITCH;
    static constexpr int PER = (KC ? KB : T) / 2, STEP = 256 / PER;      // pairs along the contiguous side, lines per round of the workgroup
    int c, line;        // this thread's pair (its first value) along the contiguous side; its first line along the other
    int row0, rows;
    int64_t pitch;      // bytes
    const char *base[KC ? PT : 1];

    __device__ __forceinline__ void init(const void *mat, int64_t ld, int r0, int n)
    {
        c = 2 * (threadIdx.x % PER);
        line = threadIdx.x / PER;
        row0 = r0;
        rows = n;
        pitch = ld * ES;
        if constexpr (KC) {
#pragma unroll
            for (int u = 0; u < PT; ++u) {
                const int r = row0 + line + u * STEP;
                base[u] = reinterpret_cast<const char *>(mat) + (int64_t)(r < rows ? r : rows - 1) * pitch;
            }
        } else {
            base[0] = reinterpret_cast<const char *>(mat) + (int64_t)(row0 + c < rows - 1 ? row0 + c : rows - 2) * ES;
        }
    }
    // clamped addresses; what does not exist is zeroed in store().  (The contiguous side has two values at least.)
    // Values of K are counted unsigned: a step's end lies up to a round of steps past K, which may be 2^31 - 1.
    __device__ __forceinline__ void fetch(uint32_t k0, uint32_t kend, uint32_t (&x)[PT][W]) const
    {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const uint32_t k = KC ? (k0 + c < kend - 1 ? k0 + c : kend - 2) : (k0 + line + u * STEP < kend ? k0 + line + u * STEP : kend - 1);
            const char *const p = KC ? base[u] + (int64_t)k * ES : base[0] + (int64_t)k * pitch;
            if constexpr (BF) x[u][0] = reinterpret_cast<const small::Pair16 *>(p)->w;
            else {
                const small::Pair32 v = *reinterpret_cast<const small::Pair32 *>(p);
                x[u][0] = v.w[0];
                x[u][1] = v.w[1];
            }
        }
    }
    __device__ __forceinline__ void store(uint32_t k0, uint32_t kend, const uint32_t (&x)[PT][W], float *lds) const
    {
        // of a pair that was moved back by one value at the end of an odd side, the second value is this thread's first
        const int left = KC ? (int)(kend - (k0 + c)) : rows - (row0 + c);
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const bool line_in = KC ? row0 + line + u * STEP < rows : k0 + line + u * STEP < kend;
            const uint32_t keep0 = line_in && left > 0 ? 0xffffffffu : 0u, keep1 = line_in && left > 1 ? 0xffffffffu : 0u;
            const uint32_t first = BF ? x[u][0] << 16 : x[u][0], second = BF ? x[u][0] & 0xffff0000u : x[u][W - 1];
            float *const d = lds + (line + u * STEP) * PITCH + c;
            d[0] = __uint_as_float((left == 1 ? second : first) & keep0);
            d[1] = __uint_as_float(second & keep1);
        }
    }
    // where this lane's value of the first instruction lies (block w0 of the tile), and the distance to the next one's
    __device__ __forceinline__ static int frag(int w0, int lane) { return KC ? (w0 + lane % S) * PITCH + lane / S : lane / S * PITCH + w0 + lane % S; }
    static constexpr int NEXT = KC ? KM : KM * PITCH;
};

template <bool BF, bool A_KC, bool B_KC, int S, int KB> constexpr int ordered_lds()
{
    return 2 * (OrderedSide<BF, A_KC, S, KB>::LDS + OrderedSide<BF, B_KC, S, KB>::LDS);
}

template <bool BF, bool A_KC, bool B_KC, int S, int KB, class P> __device__ __forceinline__ void run_ordered(const P &p, int block, float *lds)
{
    using OA = OrderedSide<BF, A_KC, S, KB>;
    using OB = OrderedSide<BF, B_KC, S, KB>;
    constexpr int T = OA::T, KM = OA::KM, PD = 4;
    constexpr bool ONE_CHAIN = BF && A_KC && !B_KC;
    constexpr int CHAINS = ONE_CHAIN ? 1 : KB / KM < 8 ? 4 : S == 16 ? 8 : 4;
    float *const As = lds, *const Bs = lds + 2 * OA::LDS; // two tiles each
    using acc_t = std::conditional_t<S == 16, core::f32x4, core::f32x16>;
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = block / tiles, t = block - vshard * tiles;
    const int m0 = (t % p.tiles_m) * T, n0 = (t / p.tiles_m) * T;
    const int shard = vshard / p.ksplit;
    const uint32_t kbeg = (uint32_t)(vshard - shard * p.ksplit) * (uint32_t)p.kchunk;
    const uint32_t kend = kbeg + (uint32_t)p.kchunk < (uint32_t)p.K ? kbeg + (uint32_t)p.kchunk : (uint32_t)p.K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave >> 1) * S, wn0 = (wave & 1) * S;
    OA a;
    OB b;
    a.init(p.A[shard], p.lda, m0, p.M);
    b.init(p.B[shard], p.ldb, n0, p.N);
    uint32_t ra[PD][OA::PT][OA::W], rb[PD][OB::PT][OB::W];
    acc_t acc[CHAINS];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int e = 0; e < S * S / 64; ++e) acc[c][e] = 0.0f;
#pragma unroll
    for (int d = 0; d < PD; ++d)
        if (kbeg + d * KB < kend) {
            a.fetch(kbeg + d * KB, kend, ra[d]);
            b.fetch(kbeg + d * KB, kend, rb[d]);
        }
    for (uint32_t k0 = kbeg; k0 < kend; k0 += PD * KB) {
#pragma unroll
        for (int d = 0; d < PD; ++d) { // (unrolled: the register ring is indexed by constants; two LDS tiles in turn)
            const uint32_t kd = k0 + d * KB;
            if (kd >= kend) break;
            a.store(kd, kend, ra[d], As + (d & 1) * OA::LDS);
            b.store(kd, kend, rb[d], Bs + (d & 1) * OB::LDS);
            __syncthreads();
            if (kd + PD * KB < kend) {
                a.fetch(kd + PD * KB, kend, ra[d]);
                b.fetch(kd + PD * KB, kend, rb[d]);
            }
            const float *const as = As + (d & 1) * OA::LDS + OA::frag(wm0, lane), *const bs = Bs + (d & 1) * OB::LDS + OB::frag(wn0, lane);
#pragma unroll
            for (int i = 0; i < KB / KM; ++i) {
                acc_t &x = acc[i % CHAINS];
                if constexpr (S == 16) x = __builtin_amdgcn_mfma_f32_16x16x4f32(as[i * OA::NEXT], bs[i * OB::NEXT], x, 0, 0, 0);
                else x = __builtin_amdgcn_mfma_f32_32x32x2f32(as[i * OA::NEXT], bs[i * OB::NEXT], x, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int n = CHAINS / 2; n >= 1; n /= 2)
#pragma unroll
        for (int c = 0; c < n; ++c) acc[c] += acc[c + n];
    void *const C = p.C[vshard];
    const int col = n0 + wn0 + lane % S;
    if (col >= p.N) return;
#pragma unroll
    for (int e = 0; e < S * S / 64; ++e) { // a lane holds one column and rows 4 (lane / S) + e % 4 of every 256 / S
        const int row = m0 + wm0 + (e >> 2) * 4 * KM + lane / S * 4 + (e & 3);
        if (row >= p.M) continue;
        float v = acc[0][e];
        if (p.relu) v = v > 0.0f ? v : 0.0f;
        if (p.out_bf16) reinterpret_cast<uint16_t *>(C)[(size_t)row * p.ldc + col] = (uint16_t)core::f32_to_bf16_bits(v);
        else reinterpret_cast<float *>(C)[(size_t)row * p.ldc + col] = v;
    }
}

template <bool BF, bool A_KC, bool B_KC, int S, int KB> __global__ __launch_bounds__(256) void gemm_ordered_kernel(const small::ParamsS p)
{
    __shared__ __attribute__((aligned(16))) float lds[ordered_lds<BF, A_KC, B_KC, S, KB>()];
    run_ordered<BF, A_KC, B_KC, S, KB>(p, (int)blockIdx.x, lds);
}

// A B^T and A^T B of a backward step in one launch.  Both are bound by their launch and a few trips to memory, and together
// take what the longer one takes alone: 3.8 + 3.7, 6.9 + 3.4 and 5.6 + 3.5 us of the 68 us of kernels in the fp32 step 256-512-256-10.
struct OrderedPair {
    small::ParamsT<8> dgrad, wgrad;
    int32_t first; // workgroups of the data gradient
};
template <bool BF, int KD, int KW> __global__ __launch_bounds__(256) void gemm_ordered_pair_kernel(const OrderedPair p)
{
    constexpr int D = ordered_lds<BF, true, true, 16, KD>(), W = ordered_lds<BF, false, false, 16, KW>();
    __shared__ __attribute__((aligned(16))) float lds[D > W ? D : W];
    const int block = (int)blockIdx.x;
    if (block < p.first) run_ordered<BF, true, true, 16, KD>(p.dgrad, block, lds);
    else run_ordered<BF, false, false, 16, KW>(p.wgrad, block - p.first, lds);
}

constexpr int64_t kMostGroups = (int64_t(1) << 24) - 1; // workgroups of 256 threads in a launch of fewer than 2^32 threads

int64_t tiles_of(int64_t M, int64_t N, int64_t outs, int64_t T) { return ((M + T - 1) / T) * ((N + T - 1) / T) * outs; }
int64_t tiles_of(const small::ParamsS &p, int count, int64_t T) { return tiles_of(p.M, p.N, (int64_t)count * p.ksplit, T); }

template <bool BF, int S, int KB> tt_status launch_ordered_tile(small::ParamsS &p, int count, bool a_kc, bool b_kc, hipStream_t s)
{
    const int64_t total = tiles_of(p, count, 2 * S);
    if (total > kMostGroups) return TT_EUNSUPPORTED;
    p.tiles_m = (int32_t)(((int64_t)p.M + 2 * S - 1) / (2 * S));
    p.tiles_n = (int32_t)(((int64_t)p.N + 2 * S - 1) / (2 * S));
    const dim3 grid((uint32_t)total), block(256);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_ordered_kernel<BF, true, true, S, KB>), grid, block, 0, s, p);
    else if (a_kc) hipLaunchKernelGGL((gemm_ordered_kernel<BF, true, false, S, KB>), grid, block, 0, s, p);
    else if (b_kc) hipLaunchKernelGGL((gemm_ordered_kernel<BF, false, true, S, KB>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_ordered_kernel<BF, false, false, S, KB>), grid, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// 64 x 64 tiles where they fill one round of the CUs or come in more than one and a half, while neither side is a strip that
// would leave half of them empty.  32 x 32 / 64 x 64 tiles, us, bf16 A B at K = 1023: 8 x (257 x 255) (200 tiles of 64 x 64) 26.8 / 31.7,
// 1023 x 1023 (256) 37.4 / 32.8, 1023 x 1535 (384) 49.4 / 50.9, 1023 x 1791 (448) 56.4 / 50.5, 1023 x 2047 (512) 63.8 / 52.5,
// 4095 x 4093 (4096) 450 / 342;  strips 20001 x 31 26.1 / 49.5, 31 x 100001 107 / 153.  One step of A B: 1023 x 1023 x 16 3.7 / 4.4.
// Steps of 16 while K is little more than one of the longer ones, whose idle part costs more than a few more barriers; on few
// tiles sooner, as there each step's wait shows.  Longer step / 16, us: 31 x 100001 x 7 bf16 13.9 / 7.6, K = 65 / 58 per cent of the time
// on A^T B fp32 50001 x 9, 1023 x 1535 0.83 of it at K = 96, 0.99 at 127; 4 x (101 x 225) 1.01 and 1.16; 4 x (2047 x 4095) 0.92 at 127.
struct OrderedTile {
    bool large, small_step; // 64 x 64 tiles; steps of 16
};
OrderedTile pick_ordered(bool nn_bf16, int64_t M, int64_t N, int64_t K, int64_t outs)
{
    const int64_t tiles = tiles_of(M, N, outs, 64);
    const int t64 = tuning_int("TT_FWD_T64", -1); // development builds: 64 x 64 from that many tiles on
    const bool one_round = tiles > 224 && tiles <= 256 && !(nn_bf16 && K <= 32);
    const bool large = (M > 32 && N > 32 && (t64 >= 0 ? tiles >= t64 : one_round || tiles > 384)) || tiles_of(M, N, outs, 32) > kMostGroups;
    return {large, K <= (tiles < 512 ? 96 : 160)};
}

template <bool BF> tt_status launch_ordered(small::ParamsS &p, int count, bool a_kc, bool b_kc, hipStream_t s)
{
    const OrderedTile t = pick_ordered(BF && a_kc && !b_kc, p.M, p.N, p.ksplit > 1 ? p.kchunk : p.K, (int64_t)count * p.ksplit);
    if (t.large)
        return t.small_step ? launch_ordered_tile<BF, 32, 16>(p, count, a_kc, b_kc, s) : launch_ordered_tile<BF, 32, 32>(p, count, a_kc, b_kc, s);
    return t.small_step ? launch_ordered_tile<BF, 16, 16>(p, count, a_kc, b_kc, s) : launch_ordered_tile<BF, 16, 64>(p, count, a_kc, b_kc, s);
}

// Whether the ordered kernel is the faster one.  gemm_small_kernel cuts K over waves whose chunks (64 values, fp32 32) need K to
// be worth cutting and whose write-out goes through LDS once more; its bf16 instructions multiply eight times as fast.  So
// bf16 crosses over at K of 200 to 500, fp32 only where K is long enough for eight waves to walk it sooner than one (few
// tiles), or where its 64 x 64 blocks fill the CUs better.  (tiles: of 64 x 64.)  Small / ordered kernel, us:
//   bf16 A B^T  257 x 255 (20 tiles)  K 63 6.1 / 3.8, 255 6.2 / 5.5, 319 6.7 / 6.2, 383 6.7 / 7.0;  511 x 767 (96)  319 8.4 / 7.8, 383 8.4 / 8.8;
//     767 x 1153 (228)  223 9.9 / 10.0, 255 9.9 / 10.8;  1023 x 1535 (384)  319 19.1 / 17.5, 447 21.2 / 21.7;  8 x (511 x 513) (576)  447 38.9 / 33.3, 511
//     40.2 / 37.5;  2047 x 4095 (2048)  159 45.1 / 38.7, 223 49.0 / 46.7, 255 49.6 / 52.4;  4 x (2047 x 4095) (8192)  191 173 / 152, 255 189 / 192
//   bf16 A^T B  257 x 255  255 9.4 / 5.6, 511 9.1 / 8.5;  511 x 767  447 14.5 / 10.1, 511 10.9 / 11.0;  767 x 1153  191 14.0 / 9.2;  1023 x 1535  191
//     20.5 / 12.8, 223 14.7 / 15.6;  2047 x 4095  159 39.6 / 37.2, 191 40.3 / 41.3, 223 43.3 / 46.5;  4 x (2047 x 4095)  191 153 / 152
//   fp32 A B^T  4 x (32 x 128) (8)  1535 20.3 / 20.8;  1023 x 1023 (256)  1023 29.6 / 33.1;  2047 x 4095  1023 186 / 202;  fp32 A^T B  4 x (101 x 225) (32)
//     1023 15.1 / 16.3;  fp32 A B  64 x (65 x 67) (256)  255 12.6 / 12.0, 511 18.1 / 20.0;  4095 x 4093 (4096) ahead up to K = 4095 (1385 / 1310)
// (fp32 A B^T on few tiles with K a little over one chunk keeps its kernel, whose one trip to memory takes it in.)
bool ordered_is_faster(bool bf, bool a_kc, bool b_kc, int64_t K, int64_t tiles)
{
    const int forced = tuning_int("TT_PLAIN_K", -1);
    if (forced >= 0) return K <= forced;
    const bool nt = a_kc && b_kc, tn = !a_kc && !b_kc;
    if (!bf) {
        if (tiles < 128 && nt && K > 32 && K <= 48) return false;
        if (tiles <= 256) return K <= (tiles < 72 ? 768 : tiles <= 224 ? 1536 : 320);
        return K <= (nt ? 768 : b_kc ? 1536 : 4096);
    }
    if (tiles <= 224) return K <= (nt ? 320 : tn ? 512 : 448);
    if (tiles <= 256) return K <= (nt ? 224 : tn ? 192 : 256);
    return K <= (tiles < 2048 ? (nt ? 448 : tn ? 192 : 256) : (nt ? 224 : 192));
}

template <bool BF, int KD, int KW> tt_status launch_ordered_pair_steps(const OrderedPair &p, int64_t total, hipStream_t s)
{
    hipLaunchKernelGGL((gemm_ordered_pair_kernel<BF, KD, KW>), dim3((uint32_t)total), dim3(256), 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}
template <bool BF> tt_status launch_ordered_pair_type(const OrderedPair &p, int64_t total, bool short_d, bool short_w, hipStream_t s)
{
    if (short_d) return short_w ? launch_ordered_pair_steps<BF, 16, 16>(p, total, s) : launch_ordered_pair_steps<BF, 16, 64>(p, total, s);
    return short_w ? launch_ordered_pair_steps<BF, 64, 16>(p, total, s) : launch_ordered_pair_steps<BF, 64, 64>(p, total, s);
}

template <bool BF, int T, class OFF> tt_status launch_small_layout(const small::ParamsS &p, bool a_kc, bool b_kc, hipStream_t s)
{
    const dim3 grid(p.per_xcd > 0 ? (uint32_t)p.per_xcd * kXcds : (uint32_t)p.total), block(p.wm * p.wn * p.wk * 64);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, true, true, T, OFF>), grid, block, 0, s, p);
    else if (a_kc) {
        if constexpr (BF) return TT_EINVAL; // (the ordered kernel's)
        else hipLaunchKernelGGL((gemm_small_kernel<BF, true, false, T, OFF>), grid, block, 0, s, p);
    }
    else if (b_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, false, true, T, OFF>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_small_kernel<BF, false, false, T, OFF>), grid, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// Block size and the waves' split between K and N (gemm_small.h); count * ksplit outputs of M x N.
template <bool BF> tt_status launch_small(small::ParamsS &p, int count, bool a_kc, bool b_kc, hipStream_t s)
{
    const int64_t outs = (int64_t)count * p.ksplit;
    // 64 x 64 blocks halve what a product reads through L2; they pay once they give every CU a workgroup.  32 x 32 / 64 x 64
    // blocks, us, K = 1023: bf16 A^T B 255 x 2047 (128 blocks of 64 x 64) 14.6 / 16.5, 1001 x 1007 (256) 22.8 / 16.6, 2047 x 2047
    // (1024) 76 / 53;  fp32 A B 24.8 / 27.5, 42.8 / 31.3, 146 / 110.  (The line is not sharp: 511 x 1535, 192 blocks, 23.8 / 16.7
    // and 41 / 29; and bf16 A B^T, whose staged rows need no more loads with the small block, stays ahead with it up to
    // 1024 blocks: 1001 x 1007 17.7 / 18.7, 8 x (511 x 513) 38.6 / 52.3, 2047 x 2047 55 / 59, K = 2047 99 / 94.)
    const int64_t pitch32 = tuning_int("TT_SMALL_PITCH", 1 << 24); // a lane's offset inside a block must fit 32 bits
    const bool big_pitch = p.lda >= pitch32 || p.ldb >= pitch32;
    const int64_t blocks64 = tiles_of(p, count, 64);
    const int T = !big_pitch && p.M > 32 && p.N > 32 && blocks64 >= tuning_int("TT_SMALL_T2", 256) ? 2 : 1;
    // Waves along K: as many as leave each of them two chunks (both on their way at once: a wave alone would not be done
    // sooner with one), while the output blocks alone do not give every CU eight waves.  Four waves at least: what K does
    // not take lies side by side along N, then M.
    const int S = 32 * T, KU = small::chunk_k<BF>(), W = T == 1 ? small::waves_of<1>() : small::waves_of<2>();
    const int64_t chunks = ((int64_t)(p.ksplit > 1 ? p.kchunk : p.K) + KU - 1) / KU;
    p.wk = 1;
    const int64_t blocks = T == 2 ? blocks64 : tiles_of(p, count, 32);
    while (p.wk < W && 4 * p.wk <= chunks && blocks * p.wk < 2048) p.wk *= 2;
    p.wn = p.wk <= 2 ? 2 : 1;
    p.wm = p.wk == 1 ? 2 : 1;
    // (fewer side by side where that leaves CUs without a workgroup: the fp32 step of tiny_mlp 98.8 -> 92.6 us)
    if ((((int64_t)p.M + p.wm * S - 1) / (p.wm * S)) * (((int64_t)p.N + p.wn * S - 1) / (p.wn * S)) * outs < 256) {
        p.wm = 1;
        p.wn = T == 1 && p.wk == 1 ? 2 : 1;
    }
    p.tiles_m = (int32_t)(((int64_t)p.M + p.wm * S - 1) / (p.wm * S));
    p.tiles_n = (int32_t)(((int64_t)p.N + p.wn * S - 1) / (p.wn * S));
    const int64_t total = (int64_t)p.tiles_m * p.tiles_n * outs;
    if (total > kMostGroups - kXcds) return TT_EUNSUPPORTED; // (launches of more than 2048 blocks have four waves or fewer)
    p.total = (int32_t)total;
    p.per_xcd = total < 8 * kXcds ? 0 : (int32_t)((total + kXcds - 1) / kXcds); // (a handful of workgroups: any order will do)
    if (big_pitch) return launch_small_layout<BF, 1, uint64_t>(p, a_kc, b_kc, s);
    return T == 2 ? launch_small_layout<BF, 2, uint32_t>(p, a_kc, b_kc, s) : launch_small_layout<BF, 1, uint32_t>(p, a_kc, b_kc, s);
}

} // namespace

// C_s = op(A_s) op(B_s); lda, ldb: elements between rows of the stored matrices; a_kc / b_kc: the operand has K contiguous
tt_status launch_gemm_small(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N, int64_t K,
                            int64_t lda, int64_t ldb, bool a_kc, bool b_kc, int in_dtype, int out_dtype, int relu, int ksplit,
                            int64_t kchunk, void *stream)
{
    if (count < 1 || count * ksplit > kMaxShards) return TT_EINVAL;
    small::ParamsS g;
    for (int i = 0; i < kMaxShards; ++i) {
        g.A[i] = i < count ? A[i] : nullptr;
        g.B[i] = i < count ? B[i] : nullptr;
        g.C[i] = i < count * ksplit ? C[i] : nullptr;
    }
    g.M = (int32_t)M; g.N = (int32_t)N; g.K = (int32_t)K;
    g.lda = lda;
    g.ldb = ldb;
    g.ldc = (int32_t)N;
    g.ksplit = ksplit;
    g.kchunk = (int32_t)kchunk;
    g.relu = relu;
    g.out_bf16 = out_dtype == TT_BF16;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const bool bf = in_dtype == TT_BF16;
    // bf16 A B, the forward layout: K increasing on every size, so that one shard product stores the same activations whatever
    // its size, tile and split, and with them the ReLU gates of the backward pass.  (F3 cuts and ksplit still add their partial
    // sums per shard, and aligned sizes add in MFMA order.)  An activation next to zero that falls on the other side moves that
    // row's gradients: on one of 12 drawn inputs by 1.2e-2 of a 1500-900-300-20 chain's gradients.
    const bool ordered = (bf && a_kc && !b_kc) || ordered_is_faster(bf, a_kc, b_kc, ksplit > 1 ? kchunk : K, tiles_of(g, count, 64));
    // The ordered kernel loads pairs along an operand's contiguous side.  A matrix of one row or one column is as well stored
    // the other way round; one that is a single value has no pair.
    if (ordered && (K == 0 || ((K > 1 || M > 1) && (K > 1 || N > 1)))) { // (K = 0: nothing is loaded, zeros are stored)
        if (a_kc ? K == 1 : M == 1) { a_kc = !a_kc; g.lda = a_kc ? K : M; }
        if (b_kc ? K == 1 : N == 1) { b_kc = !b_kc; g.ldb = b_kc ? K : N; }
        return bf ? launch_ordered<true>(g, count, a_kc, b_kc, s) : launch_ordered<false>(g, count, a_kc, b_kc, s);
    }
    if (K == 1 && N == 1) b_kc = true;      // (either way round: the layouts that exist below)
    else if (K == 1 && M == 1) a_kc = false;
    return bf ? launch_small<true>(g, count, a_kc, b_kc, s) : launch_small<false>(g, count, a_kc, b_kc, s);
}

// Both on the ordered kernel with 32 x 32 tiles (what is larger fills the chip by itself), up to eight shards.
tt_status launch_ordered_pair(const GemmCall &d, const GemmCall &w, void *stream)
{
    const GemmCall *const g[2] = {&d, &w};
    bool small_step[2];
    int64_t tiles[2];
    for (int i = 0; i < 2; ++i) {
        const GemmCall &c = *g[i];
        const bool bf = c.in_dtype == TT_BF16, nt = i == 0;
        if (c.in_dtype != d.in_dtype || c.ksplit != 1 || c.count < 1 || c.count > 8) return TT_EUNSUPPORTED;
        if (nt ? c.K < 2 : c.K < 1 || c.M < 2 || c.N < 2) return TT_EUNSUPPORTED; // pairs along the contiguous sides
        if (!ordered_is_faster(bf, nt, nt, c.K, tiles_of(c.M, c.N, c.count, 64))) return TT_EUNSUPPORTED;
        const OrderedTile t = pick_ordered(false, c.M, c.N, c.K, c.count);
        if (t.large) return TT_EUNSUPPORTED;
        small_step[i] = t.small_step;
        tiles[i] = tiles_of(c.M, c.N, c.count, 32);
    }
    if (tiles[0] + tiles[1] > kMostGroups) return TT_EUNSUPPORTED;
    OrderedPair p;
    for (int i = 0; i < 2; ++i) {
        const GemmCall &c = *g[i];
        small::ParamsT<8> &q = i == 0 ? p.dgrad : p.wgrad;
        for (int s = 0; s < 8; ++s) {
            q.A[s] = s < c.count ? c.A[s] : nullptr;
            q.B[s] = s < c.count ? c.B[s] : nullptr;
            q.C[s] = s < c.count ? c.C[s] : nullptr;
        }
        q.M = (int32_t)c.M; q.N = (int32_t)c.N; q.K = (int32_t)c.K;
        q.lda = i == 0 ? c.K : c.M;
        q.ldb = i == 0 ? c.K : c.N;
        q.ldc = (int32_t)c.N;
        q.tiles_m = (int32_t)((c.M + 31) / 32);
        q.tiles_n = (int32_t)((c.N + 31) / 32);
        q.per_xcd = 0;
        q.total = (int32_t)tiles[i];
        q.ksplit = 1;
        q.kchunk = (int32_t)c.K;
        q.wm = q.wn = q.wk = 1;
        q.relu = 0;
        q.out_bf16 = c.out_dtype == TT_BF16;
    }
    p.first = (int32_t)tiles[0];
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    ProfileScope scope(stream, TT_K_GEMM_PAIR, d.count, d.M, d.N, d.K, d.bytes() + w.bytes(), d.flops() + w.flops());
    if (d.in_dtype == TT_BF16) return launch_ordered_pair_type<true>(p, tiles[0] + tiles[1], small_step[0], small_step[1], s);
    return launch_ordered_pair_type<false>(p, tiles[0] + tiles[1], small_step[0], small_step[1], s);
}

} // namespace tt
