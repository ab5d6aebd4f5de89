// Host build of the shard-product entry point WITH its launch code (csrc/gemm.hip and csrc/gemm3.hip compiled as they
// are: tt_shard_gemm picks the engine, the tile and the in-launch K split exactly as in the library, on a device with
// 256 compute units) for checking memory accesses without a GPU.  Operands are zero, outputs start as 0x5a bytes and
// have exactly the product's size; the stand-in MFMA multiplies nothing.  Checked: no access outside a buffer or
// outside the launch's LDS (address sanitizer and explicit ranges), every output byte written.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <sys/mman.h>
#include <vector>

#define TT_HOST_EMULATION 1
#include <cstdint>
namespace tt {
namespace {
// what the kernels' `extern __shared__` arrays refer to here (one name per kernel family)
alignas(16) thread_local uint16_t smem[80 * 1024];
alignas(16) thread_local char smem2[160 * 1024], smem3[160 * 1024], smem4[160 * 1024];
}
} // namespace tt
#include "gemm.hip"
#include "gemm3.hip"
#include "gemm_small.hip"
#include "exec_common.h"

namespace tt {
ProfileScope::ProfileScope(void *, int, int, int64_t, int64_t, int64_t, uint64_t, uint64_t) : slot(-1), stream(nullptr) {}
ProfileScope::~ProfileScope() {}
} // namespace tt

static bool read_file(const char *dir, const char *name, int s, std::vector<char> &into)
{
    char path[512];
    std::snprintf(path, sizeof(path), "%s/%s%d.bin", dir, name, s);
    FILE *f = std::fopen(path, "rb");
    if (!f) return false;
    const size_t got = std::fread(into.data(), 1, into.size(), f);
    const bool at_end = std::fgetc(f) == EOF;
    std::fclose(f);
    return got == into.size() && at_end;
}

// The last chunk of a 2 x 2 product with K = 2^31 - 2 on the ordered kernel: of operands of 2^32 values only what that chunk
// may read can be read at all.
struct HugeOperand {
    char *base;
    size_t bytes;
    HugeOperand(bool k_contiguous, size_t es, size_t K, size_t kbeg) : bytes(2 * K * es)
    {
        base = static_cast<char *>(mmap(nullptr, bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
        if (base == MAP_FAILED) { std::perror("mmap"); std::exit(66); }
        for (size_t r = 0; r < (k_contiguous ? 2 : 1); ++r) { // (whole pages)
            const size_t lo = (k_contiguous ? (r * K + kbeg) * es : 2 * kbeg * es) & ~size_t(4095);
            const size_t hi = ((k_contiguous ? (r + 1) * K * es : bytes) + 4095) & ~size_t(4095);
            if (mprotect(base + lo, hi - lo, PROT_READ) != 0) { std::perror("mprotect"); std::exit(66); }
        }
    }
    ~HugeOperand() { munmap(base, bytes); }
};
struct OneResult {
    float c[4];
    void *operator[](int) const { return const_cast<float *>(c); }
};
struct LastChunk { // (what small::ParamsT has, with the one result buffer that this chunk writes)
    const void *A[1], *B[1];
    OneResult C;
    int32_t M, N, K;
    int64_t lda, ldb;
    int32_t ldc, tiles_m, tiles_n, ksplit, kchunk, relu, out_bf16;
};
template <bool BF, bool A_KC, bool B_KC, int S, int KB> static void run_last_chunk()
{
    const size_t K = 0x7ffffffe, kchunk = 662, chunks = K / kchunk, es = BF ? 2 : 4;
    static_assert(K % kchunk == 0, "chunks that end where K does");
    HugeOperand a(A_KC, es, K, K - kchunk), b(B_KC, es, K, K - kchunk);
    LastChunk p;
    std::memset(&p, 0, sizeof(p));
    p.A[0] = a.base; p.B[0] = b.base;
    for (float &v : p.C.c) v = 1.0f;
    p.M = p.N = p.ldc = 2;
    p.K = (int32_t)K;
    p.lda = A_KC ? (int64_t)K : 2; p.ldb = B_KC ? (int64_t)K : 2;
    p.tiles_m = p.tiles_n = 1;
    p.ksplit = (int32_t)chunks;
    p.kchunk = (int32_t)kchunk;
    static float lds[tt::ordered_lds<BF, A_KC, B_KC, S, KB>()];
    for (unsigned t = 0; t < 256; ++t) {
        threadIdx = {t, 0, 0};
        tt::run_ordered<BF, A_KC, B_KC, S, KB>(p, (int)chunks - 1, lds);
    }
    for (float v : p.C.c) if (v != 0.0f) { std::printf("a result of zeros is not zero\n"); std::exit(1); }
}
template <bool BF, bool A_KC, bool B_KC> static void run_last_chunks()
{
    run_last_chunk<BF, A_KC, B_KC, 16, 16>();
    run_last_chunk<BF, A_KC, B_KC, 16, 64>();
    run_last_chunk<BF, A_KC, B_KC, 32, 16>();
    run_last_chunk<BF, A_KC, B_KC, 32, 32>();
}

int main(int argc, char **argv)
{
    // emu_shard_gemm count M N K trans_a trans_b in_bf16 out_bf16 relu ksplit
    // (ksplit 1: the exported entry point; above 1: the in-launch K split the layer-chain code asks launch_gemm for,
    // which writes count * ksplit partial products)
    // With a directory as one more argument (lock-step build): operands are read from a<s>.bin / b<s>.bin there and the
    // results written to c<s>.bin, for the caller to compare with the oracle's.
    // emu_shard_gemm ahead outputs M N K trans_a: how many K tiles of 64 the 128 x 128 tile keeps on their way
    if (argc == 7 && std::strcmp(argv[1], "ahead") == 0) {
        std::printf("%d\n", tt::two_tiles_ahead(std::atol(argv[3]), std::atol(argv[4]), std::atol(argv[5]), std::atol(argv[2]), std::atoi(argv[6]) == 0) ? 2 : 1);
        return 0;
    }
    // emu_shard_gemm panel M N K: whether the panel engine takes such a product (1) or leaves it to the others (0)
    if (argc == 5 && std::strcmp(argv[1], "panel") == 0) {
        tt::core5::Params5 p;
        void *none[64] = {};
        const int64_t M = std::atol(argv[2]), N = std::atol(argv[3]), K = std::atol(argv[4]);
        std::printf("%d\n", tt::fill_params5(&p, 256, 1, none, none, none, M, N, K, M, N, N, 0) == TT_OK);
        return 0;
    }
    // emu_shard_gemm store row_bytes all_bytes: whether results leave with non-temporal stores
    if (argc == 4 && std::strcmp(argv[1], "store") == 0) {
        std::printf("%d\n", tt::non_temporal_results(std::atol(argv[2]), std::atol(argv[3])));
        return 0;
    }
    // emu_shard_gemm runs M N K blocks shards_per_block: into how many runs their K tiles are cut
    if (argc == 7 && std::strcmp(argv[1], "runs") == 0) {
        std::printf("%d\n", tt::pick_runs(std::atol(argv[2]), std::atol(argv[3]), std::atol(argv[4]), std::atoi(argv[5]), std::atoi(argv[6])));
        return 0;
    }
    // emu_shard_gemm last_chunk
    if (argc == 2 && std::strcmp(argv[1], "last_chunk") == 0) {
        run_last_chunks<true, true, true>(); run_last_chunks<true, true, false>(); run_last_chunks<true, false, true>(); run_last_chunks<true, false, false>();
        run_last_chunks<false, true, true>(); run_last_chunks<false, true, false>(); run_last_chunks<false, false, true>(); run_last_chunks<false, false, false>();
        std::printf("ok last_chunk\n");
        return 0;
    }
    if (argc != 11 && argc != 12) { std::fprintf(stderr, "usage: emu_shard_gemm count M N K trans_a trans_b in_bf16 out_bf16 relu ksplit [dir]\n"); return 64; }
    const char *dir = argc == 12 ? argv[11] : nullptr;
    emu_register_lds(tt::smem, sizeof(tt::smem));
    emu_register_lds(tt::smem2, sizeof(tt::smem2));
    emu_register_lds(tt::smem3, sizeof(tt::smem3));
    emu_register_lds(tt::smem4, sizeof(tt::smem4));
    const int count = std::atoi(argv[1]);
    const long M = std::atol(argv[2]), N = std::atol(argv[3]), K = std::atol(argv[4]);
    const int ta = std::atoi(argv[5]), tb = std::atoi(argv[6]), in_bf = std::atoi(argv[7]), out_bf = std::atoi(argv[8]), relu = std::atoi(argv[9]);
    const int ksplit = std::atoi(argv[10]);
    const size_t ib = in_bf ? 2 : 4, ob = out_bf ? 2 : 4;
    std::vector<std::vector<char>> A(count), B(count), C((size_t)count * ksplit);
    std::vector<const void *> Ap, Bp;
    std::vector<void *> Cp;
    tt::dev::g_n_readable = 0;
    tt::dev::g_readable[tt::dev::g_n_readable++] = {reinterpret_cast<const char *>(tt::core2::g_zero_chunk),
                                                    reinterpret_cast<const char *>(tt::core2::g_zero_chunk) + 16};
    for (int s = 0; s < count; ++s) {
        A[s].assign((size_t)M * K * ib, 0);
        B[s].assign((size_t)K * N * ib, 0);
        if (dir && (!read_file(dir, "a", s, A[s]) || !read_file(dir, "b", s, B[s]))) { std::fprintf(stderr, "cannot read operand %d\n", s); return 65; }
        // (operands of no elements: an address behind which nothing can be read)
        alignas(16) static char none[16];
        Ap.push_back(K ? A[s].data() : none + 16); Bp.push_back(K ? B[s].data() : none + 16);
        tt::dev::g_readable[tt::dev::g_n_readable++] = {A[s].data(), A[s].data() + A[s].size()};
        tt::dev::g_readable[tt::dev::g_n_readable++] = {B[s].data(), B[s].data() + B[s].size()};
    }
    for (auto &c : C) { c.assign((size_t)M * N * ob, (char)0x5a); Cp.push_back(c.data()); }
    const int in_dt = in_bf ? TT_BF16 : TT_F32, out_dt = out_bf ? TT_BF16 : TT_F32, act = relu ? TT_ACT_RELU : TT_ACT_NONE;
    const tt_status st = ksplit == 1 ? tt_shard_gemm(count, Ap.data(), Bp.data(), Cp.data(), M, N, K, ta, tb, in_dt, out_dt, act, nullptr)
                                     : tt::launch_gemm(count, Ap.data(), Bp.data(), Cp.data(), M, N, K, ta, tb, in_dt, out_dt, act, ksplit, nullptr);
    if (st != TT_OK) { std::printf("status %d\n", (int)st); return 2; }
    if (dir) {
        for (size_t s = 0; s < C.size(); ++s) {
            char path[512];
            std::snprintf(path, sizeof(path), "%s/c%zu.bin", dir, s);
            FILE *f = std::fopen(path, "wb");
            if (!f || std::fwrite(C[s].data(), 1, C[s].size(), f) != C[s].size()) { std::fprintf(stderr, "cannot write %s\n", path); return 66; }
            std::fclose(f);
        }
        std::printf("ok shard_gemm values: %llu threads run, launched by %s\n", g_emu_threads_run, g_emu_launched_by);
        return 0;
    }
    for (size_t s = 0; s < C.size(); ++s)
        for (size_t i = 0; i < C[s].size(); ++i)
            if (C[s][i] != 0) { std::printf("output %zu byte %zu never written\n", s, i); return 1; }
    std::printf("ok shard_gemm: %llu threads run, %llu bytes global -> LDS, %zu bytes of LDS\n", g_emu_threads_run, tt::dev::g_dma_bytes, g_emu_last_lds);
    return 0;
}
