// The step between a convolution and a fully-connected layer: the image tensor [batch][channel][pixel] changes from
// the convolutions' storage (per shard a row-major (batch * pixels) x channels matrix) to the fully-connected layers'
// storage (per shard a row-major batch x (channels * pixels) matrix, channel-major columns), or back for the gradient.
//
// Sec. 4.5 of arXiv 1805.04170 cuts a convolution's tensors along batch and channel only; with channel-major columns a
// column cut of the flattened matrix is a channel cut, so the k-cut tilings of both sides are tilings of the same
// [batch][channel] grid and the step is a tiling conversion (Sec. 5.2) whose pieces are also transposed per image.
// One launch covers all shards; a workgroup moves a square tile of pixels x channels of one image through LDS so that both
// sides are accessed along their contiguous dimension.  Small tensors are bound by latency: all of a thread's loads go out
// before the first one is used, where an element lies is worked out per row and column of the tile and not per element, and
// a tensor that gives few 64 x 64 tiles is cut into 32 x 32 ones.
#include <cstdint>
#include <type_traits>
#include "tt_device.h"
#include "tt_internal.h"

namespace tt {
namespace {

constexpr int kFlatThreads = 256;

struct SideGrid {
    uint32_t maskR, maskC, maskX;
    uint32_t simgs;  // images per shard
    uint32_t schans; // channels per shard
};

struct FlattenParams {
    const void *src[kMaxShards];
    void *dst[kMaxShards];
    uint8_t rep_ids[kMaxShards]; // id bits of the r-th destination replica
    SideGrid S, D;
    uint32_t k, nrep;
    uint32_t channels, pixels;
    uint32_t cchunks; // 64-channel chunks per image
};

__device__ __forceinline__ uint32_t deposit_dev(uint32_t v, uint32_t mask, uint32_t k)
{
    uint32_t out = 0;
    int n = __popc(mask);
    for (int b = (int)k - 1; b >= 0; --b)
        if (mask & (1u << b)) { --n; if ((v >> n) & 1u) out |= 1u << b; }
    return out;
}

// Where element (image n, channel c, pixel px) lies under a side's grid: base(n, c) + px * pitch; IMAGE: (images * pixels) x
// channels rows, otherwise images x (channels * pixels).
struct ChanLoc { uint32_t shard; uint64_t base; };
template <bool IMAGE>
__device__ __forceinline__ ChanLoc locate_chan(const SideGrid &g, uint32_t k, uint32_t pixels, uint32_t n, uint32_t c)
{
    const uint32_t rb = n / g.simgs, ni = n - rb * g.simgs;
    const uint32_t cb = c / g.schans, ci = c - cb * g.schans;
    ChanLoc e;
    e.shard = deposit_dev(rb, g.maskR, k) | deposit_dev(cb, g.maskC, k);
    e.base = IMAGE ? (uint64_t)ni * pixels * g.schans + ci : ((uint64_t)ni * g.schans + ci) * pixels;
    return e;
}

// TO_MATRIX: source is the image side.  Lanes run along channels on the image side and along pixels on the matrix side.
// TILE x TILE elements per workgroup.  A 32 x 64 x 14 x 14 tensor: 21-24 us -> 7 us (before: 64 x 64 tiles, one element
// after the other).
template <typename T, bool TO_MATRIX, int TILE>
__global__ __launch_bounds__(kFlatThreads) void flatten_kernel(const FlattenParams p)
{
    constexpr int STEP = kFlatThreads / TILE, PER = TILE / STEP; // rows a pass of the workgroup covers, passes
    __shared__ T tile[TILE][TILE + 1]; // [pixel][channel]
    const uint32_t n = blockIdx.y;
    const uint32_t cc = blockIdx.x % p.cchunks, pc = blockIdx.x / p.cchunks;
    const uint32_t c0 = cc * TILE, p0 = pc * TILE;
    const uint32_t lane = threadIdx.x % TILE, grp = threadIdx.x / TILE;
    const uint32_t clast = p.channels - 1, plast = p.pixels - 1;
    // elements past the end are loaded from the last channel or pixel and not stored
    T v[PER];
    if (TO_MATRIX) {
        const uint32_t c = c0 + lane < clast ? c0 + lane : clast;
        const ChanLoc e = locate_chan<true>(p.S, p.k, p.pixels, n, c);
        const T *src = reinterpret_cast<const T *>(p.src[e.shard]) + e.base; // replica with all other id bits zero
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t px = p0 + grp + i * STEP;
            v[i] = src[(uint64_t)(px < plast ? px : plast) * p.S.schans];
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) tile[grp + i * STEP][lane] = v[i];
    } else {
        // few channels leave passes of the workgroup without one (the same passes for all its threads): these would load for
        // nothing, each with its own search for the shard (256 x 3 x 1024: 26.6 us with them, 18.9 without)
        const uint32_t rows = p.channels - c0, px = p0 + lane < plast ? p0 + lane : plast;
        const auto move = [&](auto every_pass) {
            constexpr bool ALL = decltype(every_pass)::value;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (!ALL && (uint32_t)(i * STEP) >= rows) break;
                const uint32_t c = c0 + grp + i * STEP;
                const ChanLoc e = locate_chan<false>(p.S, p.k, p.pixels, n, c < clast ? c : clast);
                v[i] = reinterpret_cast<const T *>(p.src[e.shard])[e.base + px];
            }
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (!ALL && (uint32_t)(i * STEP) >= rows) break;
                tile[lane][grp + i * STEP] = v[i];
            }
        };
        if (rows > (uint32_t)((PER - 1) * STEP)) move(std::true_type());
        else move(std::false_type());
    }
    __syncthreads();
    if (TO_MATRIX) {
        const uint32_t px = p0 + lane;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t c = c0 + grp + i * STEP;
            if (c >= p.channels || px >= p.pixels) continue;
            const ChanLoc e = locate_chan<false>(p.D, p.k, p.pixels, n, c);
            const T x = tile[lane][grp + i * STEP];
            for (uint32_t r = 0; r < p.nrep; ++r) reinterpret_cast<T *>(p.dst[e.shard | p.rep_ids[r]])[e.base + px] = x;
        }
    } else {
        const uint32_t c = c0 + lane;
        if (c >= p.channels) return;
        const ChanLoc e = locate_chan<true>(p.D, p.k, p.pixels, n, c);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t px = p0 + grp + i * STEP;
            if (px >= p.pixels) continue;
            const T x = tile[grp + i * STEP][lane];
            for (uint32_t r = 0; r < p.nrep; ++r)
                reinterpret_cast<T *>(p.dst[e.shard | p.rep_ids[r]])[e.base + (uint64_t)px * p.D.schans] = x;
        }
    }
}

bool side_grid(const tt_tiling &t, int k, int64_t batch, int64_t channels, SideGrid *out, Grid *g)
{
    if (!make_grid(t.cut, k, batch, channels, g)) return false;
    out->maskR = g->maskR;
    out->maskC = g->maskC;
    out->maskX = g->maskX;
    out->simgs = (uint32_t)g->srows;
    out->schans = (uint32_t)g->scols;
    return true;
}

template <typename T, int TILE> tt_status launch_flatten_t(FlattenParams &p, int64_t batch, bool to_matrix, hipStream_t s)
{
    p.cchunks = (p.channels + TILE - 1) / TILE;
    const uint64_t gx = (uint64_t)p.cchunks * (((uint64_t)p.pixels + TILE - 1) / TILE);
    if (gx >= (uint64_t(1) << 31)) return TT_EUNSUPPORTED;
    const dim3 grid((uint32_t)gx, (uint32_t)batch);
    if (to_matrix) hipLaunchKernelGGL((flatten_kernel<T, true, TILE>), grid, dim3(kFlatThreads), 0, s, p);
    else hipLaunchKernelGGL((flatten_kernel<T, false, TILE>), grid, dim3(kFlatThreads), 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

} // namespace
} // namespace tt

extern "C" tt_status tt_flatten(void *const *dst, tt_tiling B, const void *const *src, tt_tiling A, int k, int64_t batch,
                                int64_t channels, int64_t pixels, int elem_bytes, int to_matrix, void *stream)
{
    using namespace tt;
    if (!dst || !src || !valid_k(k) || !valid_tiling(A, k) || !valid_tiling(B, k)) return TT_EINVAL;
    if (batch < 0 || channels < 0 || pixels < 0 || (elem_bytes != 2 && elem_bytes != 4)) return TT_EINVAL;
    Grid ga, gb;
    FlattenParams p;
    if (!side_grid(A, k, batch, channels, &p.S, &ga) || !side_grid(B, k, batch, channels, &p.D, &gb)) return TT_EINFEASIBLE;
    if (batch == 0 || channels == 0 || pixels == 0) return TT_OK;
    // grid.y carries the image number; per-shard offsets are 64-bit, the coordinates themselves 32-bit
    if (batch > 65535 || channels >= (int64_t(1) << 31) || pixels >= (int64_t(1) << 31) ||
        batch * pixels >= (int64_t(1) << 32))
        return TT_EUNSUPPORTED;
    const int n = 1 << k;
    for (int s = 0; s < kMaxShards; ++s) {
        p.src[s] = s < n ? src[s] : nullptr;
        p.dst[s] = s < n ? dst[s] : nullptr;
        p.rep_ids[s] = 0;
        if (s < n && (!src[s] || !dst[s] || reinterpret_cast<uintptr_t>(src[s]) % elem_bytes ||
                      reinterpret_cast<uintptr_t>(dst[s]) % elem_bytes))
            return TT_EINVAL;
    }
    p.k = (uint32_t)k;
    p.nrep = 1u << gb.kX;
    for (uint32_t r = 0; r < p.nrep; ++r) p.rep_ids[r] = (uint8_t)deposit(r, gb.maskX, k);
    p.channels = (uint32_t)channels;
    p.pixels = (uint32_t)pixels;
    // 64 x 64 tiles (whole cache lines on both sides) where they give every CU four workgroups, else 32 x 32; those also
    // where the pixels, or on the way to images the channels, of an image fit in one (the larger tile's passes would mostly
    // be empty).  64 x 64 / 32 x 32 tiles, us: to matrix 2048 x 64 x 4 14.2 / 9.4, 4096 x 8 x 16 8.0 / 5.4, but 8 x 1 x 65536 11.4 / 12.9
    // and 512 x 20 x 400 12.3 / 12.5; to images 256 x 3 x 1024 18.9 / 12.5, 512 x 20 x 400 18.2 / 15.2.
    const uint64_t tiles64 = (((uint64_t)channels + 63) / 64) * (((uint64_t)pixels + 63) / 64) * (uint64_t)batch;
    const uint64_t bytes = (uint64_t)batch * channels * pixels * elem_bytes;
    ProfileScope scope(stream, TT_K_CONVERT, n, batch * pixels, channels, elem_bytes, bytes * (1u + p.nrep), 0);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (tiles64 >= 1024 && pixels > 32 && (to_matrix || channels > 32))
        return elem_bytes == 2 ? launch_flatten_t<uint16_t, 64>(p, batch, to_matrix != 0, s)
                               : launch_flatten_t<uint32_t, 64>(p, batch, to_matrix != 0, s);
    return elem_bytes == 2 ? launch_flatten_t<uint16_t, 32>(p, batch, to_matrix != 0, s)
                           : launch_flatten_t<uint32_t, 32>(p, batch, to_matrix != 0, s);
}
