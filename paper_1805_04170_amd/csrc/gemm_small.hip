// Shard products that the MFMA tile engines do not take: fp32, and bf16 whose rows are not whole 16-byte vectors, whose
// addresses are not multiples of 16 bytes, or of which one operand has 2^31 elements or more.  gemm_small_kernel
// (gemm_small.h): matrix instructions.  gemm_plain_kernel, gemm_ordered_kernel: fused multiply-adds in the order of
// increasing K; short K, and the forward layout of bf16.
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

// Plain products: one 64 x 64 tile per workgroup, fp32 fused multiply-adds in the order of increasing K, any layout.  16
// values of K per step through LDS, 4 x 4 results per thread, operands fetched into registers four steps ahead.  Bound by
// LDS reads and the vector unit (two LDS values per four multiply-adds).
template <bool BF, bool A_KC, bool B_KC, bool OUT_BF16> __global__ __launch_bounds__(256) void gemm_plain_kernel(const small::ParamsS p)
{
    using E = std::conditional_t<BF, uint16_t, uint32_t>; // an element's bits
    constexpr int T = 64, KB = 16;
    __shared__ float As[KB][T + 1];
    __shared__ float Bs[KB][T + 1];
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = blockIdx.x / tiles, t = blockIdx.x - vshard * tiles;
    const int m0 = (t % p.tiles_m) * T, n0 = (t / p.tiles_m) * T;
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int kend = kbeg + p.kchunk < p.K ? kbeg + p.kchunk : p.K;
    const E *A = reinterpret_cast<const E *>(p.A[shard]), *B = reinterpret_cast<const E *>(p.B[shard]);
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    float acc[4][4] = {};
    constexpr int PT = T * KB / 256, PD = 4;
    float ra[PD][PT], rb[PD][PT];
    // all loads of a step in flight together: clamped addresses, the out-of-range values zeroed afterwards
    auto fetch = [&](int k0, float (&xa)[PT], float (&xb)[PT]) {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int i = threadIdx.x + u * 256;
            const int gm = m0 + (A_KC ? i / KB : i % T), gka = k0 + (A_KC ? i % KB : i / T);
            const int gn = n0 + (B_KC ? i / KB : i % T), gkb = k0 + (B_KC ? i % KB : i / T);
            const int64_t am = gm < p.M ? gm : p.M - 1, ak = gka < kend ? gka : kend - 1;
            const int64_t bn = gn < p.N ? gn : p.N - 1, bk = gkb < kend ? gkb : kend - 1;
            const uint32_t va = A[A_KC ? am * p.lda + ak : ak * p.lda + am], vb = B[B_KC ? bn * p.ldb + bk : bk * p.ldb + bn];
            xa[u] = gm < p.M && gka < kend ? __uint_as_float(BF ? va << 16 : va) : 0.0f;
            xb[u] = gn < p.N && gkb < kend ? __uint_as_float(BF ? vb << 16 : vb) : 0.0f;
        }
    };
#pragma unroll
    for (int d = 0; d < PD; ++d)
        if (kbeg + d * KB < kend) fetch(kbeg + d * KB, ra[d], rb[d]);
    for (int k0 = kbeg; k0 < kend; k0 += PD * KB) {
#pragma unroll
        for (int d = 0; d < PD; ++d) { // (unrolled: the register ring is indexed by constants)
            const int kd = k0 + d * KB;
            if (kd >= kend) break;
#pragma unroll
            for (int u = 0; u < PT; ++u) {
                const int i = threadIdx.x + u * 256;
                As[A_KC ? i % KB : i / T][A_KC ? i / KB : i % T] = ra[d][u];
                Bs[B_KC ? i % KB : i / T][B_KC ? i / KB : i % T] = rb[d][u];
            }
            __syncthreads();
            if (kd + PD * KB < kend) fetch(kd + PD * KB, ra[d], rb[d]);
#pragma unroll
            for (int kk = 0; kk < KB; ++kk) {
                float a[4], b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { a[i] = As[kk][ty * 4 + i]; b[i] = Bs[kk][tx * 4 + i]; }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
            }
            __syncthreads();
        }
    }
    void *const C = p.C[vshard];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = m0 + ty * 4 + i, col = n0 + tx * 4 + j;
            if (row >= p.M || col >= p.N) continue;
            float v = acc[i][j];
            if (p.relu) v = v > 0.0f ? v : 0.0f;
            if (OUT_BF16) reinterpret_cast<uint16_t *>(C)[(size_t)row * p.ldc + col] = (uint16_t)core::f32_to_bf16_bits(v);
            else reinterpret_cast<float *>(C)[(size_t)row * p.ldc + col] = v;
        }
}

// bf16 C = A B, both row-major as stored (the forward layout): the same multiply-adds in the same order, hence the same
// bits, on 32 x 32 tiles.  Bound by latency: 2 x 2 results per thread, operands fetched into registers four K tiles ahead.
// With 64 x 64 tiles 4 x (100 x 225 x 1500) took 138 us, so 53; the step of a 1500-900-300-20 chain at batch 100 went from
// 327 to 181 us.  Why K increases here and the MFMA kernel does not take this layout: one shard product then stores the
// same activations on every size, tile and split of the waves, and with them the ReLU gates of the backward pass.  (F3 cuts
// and ksplit still add their partial sums per shard, and aligned sizes add in MFMA order.)  An activation next to zero that
// falls on the other side moves that row's gradients: on one of 12 drawn inputs by 1.2e-2 of such a chain's gradients.
constexpr int kOrdTile = 32, kOrdK = 16;
template <bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_ordered_kernel(const small::ParamsS p)
{
    constexpr int T = kOrdTile, KB = kOrdK, PT = T * KB / 256, PD = 4;
    __shared__ float As[2][KB][T + 2];
    __shared__ float Bs[2][KB][T + 2];
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = blockIdx.x / tiles, t = blockIdx.x - vshard * tiles;
    const int m0 = (t % p.tiles_m) * T, n0 = (t / p.tiles_m) * T;
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int kend = kbeg + p.kchunk < p.K ? kbeg + p.kchunk : p.K;
    const uint16_t *A = reinterpret_cast<const uint16_t *>(p.A[shard]), *B = reinterpret_cast<const uint16_t *>(p.B[shard]);
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    float acc[2][2] = {};
    uint32_t ra[PD][PT], rb[PD][PT];
    // clamped addresses, out-of-range values zeroed by AND (a load under a branch would be waited for by itself)
    auto fetch = [&](int k0, uint32_t (&xa)[PT], uint32_t (&xb)[PT]) {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int i = threadIdx.x + u * 256;
            const int gka = k0 + i % KB, gm = m0 + i / KB, gkb = k0 + i / T, gn = n0 + i % T;
            const uint32_t va = A[(int64_t)(gm < p.M ? gm : p.M - 1) * p.lda + (gka < kend ? gka : kend - 1)];
            const uint32_t vb = B[(int64_t)(gkb < kend ? gkb : kend - 1) * p.ldb + (gn < p.N ? gn : p.N - 1)];
            xa[u] = (va << 16) & (gm < p.M && gka < kend ? 0xffffffffu : 0u);
            xb[u] = (vb << 16) & (gn < p.N && gkb < kend ? 0xffffffffu : 0u);
        }
    };
#pragma unroll
    for (int d = 0; d < PD; ++d)
        if (kbeg + d * KB < kend) fetch(kbeg + d * KB, ra[d], rb[d]);
    for (int k0 = kbeg; k0 < kend; k0 += PD * KB) {
#pragma unroll
        for (int d = 0; d < PD; ++d) { // (unrolled: the register ring is indexed by constants; two LDS tiles in turn, one barrier each)
            const int kd = k0 + d * KB;
            if (kd >= kend) break;
#pragma unroll
            for (int u = 0; u < PT; ++u) {
                const int i = threadIdx.x + u * 256;
                As[d & 1][i % KB][i / KB] = __uint_as_float(ra[d][u]);
                Bs[d & 1][i / T][i % T] = __uint_as_float(rb[d][u]);
            }
            __syncthreads();
            if (kd + PD * KB < kend) fetch(kd + PD * KB, ra[d], rb[d]);
#pragma unroll
            for (int kk = 0; kk < KB; ++kk) {
                const float a0 = As[d & 1][kk][ty * 2], a1 = As[d & 1][kk][ty * 2 + 1];
                const float b0 = Bs[d & 1][kk][tx * 2], b1 = Bs[d & 1][kk][tx * 2 + 1];
                acc[0][0] = fmaf(a0, b0, acc[0][0]); acc[0][1] = fmaf(a0, b1, acc[0][1]);
                acc[1][0] = fmaf(a1, b0, acc[1][0]); acc[1][1] = fmaf(a1, b1, acc[1][1]);
            }
        }
    }
    void *const C = p.C[vshard];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = m0 + ty * 2 + i, col = n0 + tx * 2 + j;
            if (row >= p.M || col >= p.N) continue;
            float v = acc[i][j];
            if (p.relu) v = v > 0.0f ? v : 0.0f;
            if (OUT_BF16) reinterpret_cast<uint16_t *>(C)[(size_t)row * p.ldc + col] = (uint16_t)core::f32_to_bf16_bits(v);
            else reinterpret_cast<float *>(C)[(size_t)row * p.ldc + col] = v;
        }
}

constexpr int64_t kMostGroups = (int64_t(1) << 24) - 1; // workgroups of 256 threads in a launch of fewer than 2^32 threads

int64_t tiles_of(const small::ParamsS &p, int count, int64_t T) { return ((p.M + T - 1) / T) * ((p.N + T - 1) / T) * count * p.ksplit; }

template <bool BF, bool A_KC, bool B_KC> tt_status launch_plain_layout(small::ParamsS &p, int count, hipStream_t s)
{
    const int64_t total = tiles_of(p, count, 64);
    if (total > kMostGroups) return TT_EUNSUPPORTED;
    p.tiles_m = (int32_t)(((int64_t)p.M + 63) / 64);
    p.tiles_n = (int32_t)(((int64_t)p.N + 63) / 64);
    const dim3 grid((uint32_t)total), block(256);
    if (p.out_bf16) hipLaunchKernelGGL((gemm_plain_kernel<BF, A_KC, B_KC, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_plain_kernel<BF, A_KC, B_KC, false>), grid, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <bool BF> tt_status launch_plain(small::ParamsS &p, int count, bool a_kc, bool b_kc, hipStream_t s)
{
    if (a_kc && b_kc) return launch_plain_layout<BF, true, true>(p, count, s);
    if (a_kc) return launch_plain_layout<BF, true, false>(p, count, s);
    return b_kc ? launch_plain_layout<BF, false, true>(p, count, s) : launch_plain_layout<BF, false, false>(p, count, s);
}

// The forward layout of bf16.  64 x 64 tiles once there are about three for every two CUs, while neither side is a strip
// that would leave half of them empty: the larger tile reads half as much LDS per multiply-add and half the operands.
// 32 x 32 / 64 x 64 tiles, us, at K = 33 and 1023: 1023 x 1279 (320 tiles of 64 x 64) 6.9 / 8.4 and 91 / 100, 1023 x 1535 (384)
// 7.4 / 8.4 and 107 / 101, 1023 x 1663 (416) 8.2 / 8.4 and 123 / 102, 33 x 25001 (391) 8.5 / 8.3 and 129 / 110, 1023 x 2047 (512)
// 9.1 / 8.5 and 139 / 108; 4095 x 4093 (4096) at K = 2047 2027 / 1307.  Strips: 31 x 100001 at K = 1023 223 / 314.
tt_status launch_forward(small::ParamsS &p, int count, hipStream_t s)
{
    const int64_t total = tiles_of(p, count, kOrdTile);
    if ((p.M > 32 && p.N > 32 && tiles_of(p, count, 64) >= tuning_int("TT_FWD_T64", 400)) || total > kMostGroups)
        return launch_plain<true>(p, count, true, false, s);
    p.tiles_m = (int32_t)(((int64_t)p.M + kOrdTile - 1) / kOrdTile);
    p.tiles_n = (int32_t)(((int64_t)p.N + kOrdTile - 1) / kOrdTile);
    const dim3 grid((uint32_t)total), block(256);
    if (p.out_bf16) hipLaunchKernelGGL(gemm_ordered_kernel<true>, grid, block, 0, s, p);
    else hipLaunchKernelGGL(gemm_ordered_kernel<false>, grid, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// Short K: whether the plain kernel is the faster one.  gemm_small_kernel's waves take K in chunks (64 values, fp32 32), of
// which a short K gives them one or two, and its write-out goes through LDS once more; the longer K is, the more the matrix
// instructions win, the sooner the more often every CU gets a tile (tiles: of 64 x 64).  Between 128 and 192 values of K (fp32
// between 64 and 96) the chunks are not yet cut over two waves.  Plain / small kernel, us:
//   bf16 A B^T  1023 x 1535 (384 tiles)  K 15 5.5 / 14.5, 95 12.9 / 20.1, 175 20.3 / 22.0, 223 24.7 / 17.1;  767 x 769 (156)  47 7.1 / 9.0,
//     63 8.2 / 8.1;  257 x 255 (20)  15 4.6 / 5.9, 47 6.8 / 6.3;  8 x (511 x 513) (576)  191 28.6 / 41.6, 223 32.6 / 30.8;
//     2047 x 4095 (2048)  63 26.4 / 37.2, 95 36.7 / 42.1, 127 47.0 / 42.6;  strips 31 x 100001 (1563)  47 19.1 / 25.3, 63 23.2 / 22.4
//   fp32 A B  1023 x 1535  15 6.4 / 13.2, 95 13.1 / 19.9, 111 14.7 / 13.7;  767 x 769  95 10.6 / 11.7, 127 12.9 / 12.7;  257 x 255  15 4.2 / 4.9,
//     31 5.4 / 4.9, 47 6.7 / 7.5, 111 11.4 / 6.9;  8 x (511 x 513)  159 25.6 / 30.4, 191 30.1 / 30.5;  2047 x 4095  111 44.9 / 47.4,
//     143 54.6 / 52.6;  strips 31 x 100001  63 25.3 / 33.2, 111 38.8 / 40.1
bool plain_is_faster(bool bf, bool a_kc, bool b_kc, int64_t M, int64_t N, int64_t K, int64_t tiles)
{
    const int forced = tuning_int("TT_PLAIN_K", -1);
    if (forced >= 0) return K <= forced;
    const bool nt = a_kc && b_kc;
    if (M <= 32 || N <= 32) { // a strip: half of each 64 x 64 tile is empty, while the other kernel's blocks are 32 x 32
        if (!bf) return K <= (tiles < 512 ? 16 : tiles < 1024 ? 64 : a_kc || b_kc ? 96 : 144);
        return K <= (tiles < 256 ? 16 : nt || tiles >= 1024 ? 48 : tiles < 512 ? 16 : 32);
    }
    if (tiles < 128) return bf ? K <= 32 : K <= 16 || (K > 32 && K <= 48 && !nt); // (fp32 up to 32: a single chunk)
    if (tiles < 256) return K <= (bf ? 48 : 96);
    if (M <= 64 || N <= 64) return K <= 192; // half of the other kernel's waves have no rows or columns of their own
    if (tiles < 512) return K <= (bf ? 176 : 96);
    if (tiles < 1024) return K <= (bf ? 192 : 160);
    if (tiles < 2048) return K <= 144;
    return K <= (bf ? 96 : 128);
}

template <bool BF, int T, class OFF> tt_status launch_small_layout(const small::ParamsS &p, bool a_kc, bool b_kc, hipStream_t s)
{
    const dim3 grid(p.per_xcd > 0 ? (uint32_t)p.per_xcd * kXcds : (uint32_t)p.total), block(p.wm * p.wn * p.wk * 64);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, true, true, T, OFF>), grid, block, 0, s, p);
    else if (a_kc) {
        if constexpr (BF) return TT_EINVAL; // (launch_forward's)
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
    if (bf && a_kc && !b_kc) return launch_forward(g, count, s);
    if (plain_is_faster(bf, a_kc, b_kc, M, N, ksplit > 1 ? kchunk : K, tiles_of(g, count, 64)))
        return bf ? launch_plain<true>(g, count, a_kc, b_kc, s) : launch_plain<false>(g, count, a_kc, b_kc, s);
    return bf ? launch_small<true>(g, count, a_kc, b_kc, s) : launch_small<false>(g, count, a_kc, b_kc, s);
}

} // namespace tt
