// Union path for large batches (prefill-like): LDS-tiled bf16 MFMA gather-GEMMs over an
// explicit list of the union's slots.
//
// The computation is the one of the union path (Selective Computation section; see
// k_union.hip): with U = A_1 u ... u A_B,
//   H[b][u] = SiLU(x_b . gate_c[U_u]) * (x_b . up_c[U_u]) * [U_u in A_b],   Y = H . down_c[U].
// For many tokens the weights are reused across the batch, so both products are compute
// bound and are tiled for MFMA throughput instead of streamed:
//  - or_blocks / union_scan: the OR of the token bitmaps per block of 64 tokens, then one
//    work-group ORs the blocks and turns the union into the ascending list of its slots;
//  - gemm1_pipe: H for a tile of tokens x union slots, K = d. The tile's weight rows are
//    ordered so that gate and up of one (token, slot) land in one lane, and the SiLU*up*mask
//    epilogue needs no data exchange. H is written as bf16(h), and with SI_FLAG_EXACT_H also
//    lo = bf16(h - hi) as a second plane;
//  - gemm2_pipe: Y for a tile of tokens x columns over one of KS chunks of the union, K =
//    union position. H rows are K-contiguous; the down rows are row segments, read back
//    transposed into the MFMA layout with ds_read_b64_tr_b16. H enters the MFMA as one 16-bit
//    value (about 8 significant bits of h for bf16) unless SI_FLAG_EXACT_H asks for the hi +
//    lo pair (about 16 bits, twice the MFMA work). The first chunk's sums go to y, the others'
//    to partials that add_partials adds in a fixed order.
// Both GEMMs are one pipeline. Operand tiles go straight from memory to LDS (pipe.h), K in
// steps of 64, two to four stages of them; a wave's fragments are read half a step ahead of
// their MFMAs, and there is one barrier a step, met by every wave with half a step of MFMAs in
// registers. What it is bound by, and what each part gave (GEMM1 of 512 tokens x 9677 slots,
// d = 5120; of 2048 x 7706, d = 4096; of 512 x 14336, d = 4096; weights in the Infinity Cache):
//  - staging through registers, two barriers a step (256 x 160 and 128 x 160 tiles): 111, 310
//    and 133 us;
//  - this pipeline, LDS reads and loads spread over the MFMAs by scheduling groups between
//    scheduling barriers: 83, 188 and 90 us (1220, 1377 and 1336 TFLOP/s; the vendor library
//    reaches 1383 on an 8192-cubed bf16 product). The same code scheduled by the compiler alone
//    takes 92, 200 and 97 us; scheduling groups without the barriers spill. Raising the waves'
//    priority around the MFMAs gave nothing.
//  - With the weights read from HBM a step's loads need more than one step (1.0 to 1.4 us) of
//    flight: 256 x 160 tiles take 122 us with two stages and 97 us with three. 256 x 256 tiles
//    have room for three stages of the weights and two of x, which stays in L2.
// A microbenchmark of the load path alone takes 75 to 113 GB/s a CU from L2 into LDS, three
// times what these kernels need; LDS reads run at about 240 bytes a cycle.
#include <hip/hip_ext.h>

#include <atomic>

#include "common.h"
#include "launch.h"
#include "gemm_pipe.h"
#include "selectinfer.h"

namespace si {

namespace {

// part[c][w] = OR of bits[b][w] over the 64 tokens b of block c. Work-group (wx, c): 64 words
// x 64 tokens; each wave ORs 16 tokens of the 64 words, then the 4 waves meet in LDS.
__global__ __launch_bounds__(256) void or_blocks(const uint32_t* __restrict__ bits, int64_t B,
                                                 int64_t W, uint32_t* __restrict__ part) {
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t w = (int64_t)blockIdx.x * 64 + lane;
    const int64_t b0 = (int64_t)blockIdx.y * 64 + 16 * wv;
    // range-checked buffer loads, issued together (a load behind each token's condition made
    // the compiler wait for it before the next)
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(bits, B * W * 4);
    uint32_t v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        v[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
            rb, (w < W && b0 + i < B) ? (int)(((b0 + i) * W + w) * 4) : kOOB, 0, 0);
    uint32_t u = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) u |= v[i];
    __shared__ uint32_t red[4][64];
    red[wv][lane] = u;
    __syncthreads();
    if (wv == 0 && w < W) part[(int64_t)blockIdx.y * W + w] = red[0][lane] | red[1][lane] |
                                                               red[2][lane] | red[3][lane];
}

// One work-group: the union of the nb block bitmaps part[0..nb)[W], its set bits in ascending
// order -> ulist, their number -> *ucount. The union words are formed once into LDS (thread t
// takes words t, t + 1024, ...; the block rows of a word are read eight at a time with
// range-checked loads issued together, so a word costs one memory round trip per eight
// blocks). Thread t then owns a contiguous run of words; an exclusive scan of the runs' counts
// (wave scans, then the 16 wave totals) gives each run its first position. Dynamic LDS: W
// words (W <= 16368).
__global__ __launch_bounds__(1024) void union_scan(const uint32_t* __restrict__ part, int64_t nb,
                                                   int64_t W, int32_t* __restrict__ ulist,
                                                   int* __restrict__ ucount) {
    extern __shared__ uint32_t uw[];
    __shared__ int wtot[16];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wv = t >> 6;
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(part, nb * W * 4);
    for (int64_t w = t; w < W; w += 1024) {
        uint32_t u = 0u;
        for (int64_t c0 = 0; c0 < nb; c0 += 8) {
            uint32_t v[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                v[c] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rp, c0 + c < nb ? (int)(((c0 + c) * W + w) * 4) : kOOB, 0, 0);
#pragma unroll
            for (int c = 0; c < 8; ++c) u |= v[c];
        }
        uw[w] = u;
    }
    __syncthreads();
    const int64_t per = (W + 1023) / 1024;
    const int64_t w0 = (int64_t)t * per;
    const int64_t w1 = (w0 + per < W) ? w0 + per : W;
    int c = 0;
    for (int64_t w = w0; w < w1; ++w) c += __popc(uw[w]);
    const int incl = wave_incl_scan(c);
    if (lane == kWave - 1) wtot[wv] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        before += q < wv ? wtot[q] : 0;
        all += wtot[q];
    }
    int pos = before + incl - c;
    for (int64_t w = w0; w < w1; ++w) {
        uint32_t u = uw[w];
        while (u) {
            const int j = __ffs(u) - 1;
            ulist[pos++] = (int32_t)(w * 32 + j);
            u &= u - 1u;
        }
    }
    if (t == 0) *ucount = all;
}

// ---- tile choice ---------------------------------------------------------------------------
// Time of one K step (64) of a work-group that has a CU to itself, in units of 10 ns, measured
// over whole GEMMs with the weights in HBM (kernel time / rounds of work-groups / steps): the
// larger tile does more per byte it takes in and per barrier, the smaller one fills the CUs
// where the product is small. By least (rounds x time) the choice was the fastest, or within 3%
// of it, at each of 18 sizes from 128 to 2048 tokens; e.g. with 256 x 256, 256 x 192, 256 x 160,
// 128 x 256 and 128 x 160 tiles 512 tokens x 11000 slots, d = 5120 take 114, 104, 172, 156 and
// 180 us, 512 x 7706, d = 4096 85, 76, 69, 65 and 100, 200 x 8602, d = 4096 85, 77, 67, 63 and 51.
struct G1Tile {
    int bm, bn, cost;
};
constexpr G1Tile kG1Tiles[] = {
    {256, 256, 145}, {256, 192, 128}, {256, 160, 115}, {128, 256, 105}, {128, 160, 82}};
constexpr int kG1Count = 5;
struct G2Tile {
    int bm, bn, cost;
};
constexpr G2Tile kG2Tiles[] = {{256, 256, 160}, {256, 128, 90}, {128, 128, 52}};  // one 16-bit h
constexpr int kG2Count = 3;
// (128 x 256 against 128 x 128, 200 tokens, d = 4096: 34 / 40 us, rows from HBM 44 / 56 us)
constexpr G2Tile kG2Exact[] = {{128, 256, 190}, {128, 128, 116}};  // hi + lo pair
constexpr int kG2ExactCount = 2;

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// GEMM1 tile for T tokens over L slots: least (rounds of work-groups) x (time of a step)
int gemm1_pick(int64_t T, int64_t L, int num_cu) {
    int best = 0;
    int64_t bc = INT64_MAX;
    for (int c = 0; c < kG1Count; ++c) {
        const int64_t tiles = cdiv(T, kG1Tiles[c].bm) * cdiv(L, kG1Tiles[c].bn / 2);
        const int64_t cost = cdiv(tiles, num_cu) * kG1Tiles[c].cost;
        if (cost < bc) bc = cost, best = c;
    }
    return best;
}

struct TPlan {
    int64_t W, Lp, Up;
    int g1, ntm1, nst;       // GEMM1: tile (kG1Tiles), token tiles, slot tiles (of all L slots)
    int g2, ntm2, ntn2, KS;  // GEMM2: tile (kG2Tiles), token tiles, column tiles, K chunks
    int64_t nb;              // blocks of 64 tokens
    int scan;                // GEMM1 forms the union list itself
    size_t off_bits, off_words, off_ulist, off_count, off_hhi, off_hlo, off_part, total;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Partial rows a workspace has room for (per token): what fills the CUs once with 256-token
// tiles of 128 columns (160 and 192 where d needs more than 32 of them). Keeps the workspace
// bounded whatever tile GEMM2 takes.
int64_t partial_rows(int64_t B, int64_t L, int64_t d, int num_cu) {
    int64_t cols = 128;
    while (cols < 192 && cdiv(d, cols) > 32) cols += 32;
    int64_t r = num_cu / (cdiv(B, 256) * cdiv(d, cols));
    const int64_t kmax = cdiv(L, kBK);
    if (r > kmax) r = kmax;
    if (r > 64) r = 64;
    return r < 1 ? 1 : r;
}

// The tiles, and the K chunks (at most `rows`), for a union of at most U slots
void pick_tiles(TPlan& p, int64_t B, int64_t U, int64_t d, int num_cu, bool exact, int64_t rows) {
    p.g1 = gemm1_pick(B, U, num_cu);
    p.ntm1 = (int)cdiv(B, kG1Tiles[p.g1].bm);
    p.nst = (int)cdiv(U, kG1Tiles[p.g1].bn / 2);
    // GEMM2: tile and K chunks of least time, where every chunk past the first writes and the
    // reducer reads one float32 partial of Y (about 4 TB/s both ways: 2 B d / 10^7 units of
    // 10 ns a chunk)
    const int64_t steps = cdiv(U, kBK);
    double bc = 1e300;
    for (int c = 0; c < (exact ? kG2ExactCount : kG2Count); ++c) {
        const G2Tile& tl = exact ? kG2Exact[c] : kG2Tiles[c];
        const int64_t tiles = cdiv(B, tl.bm) * cdiv(d, tl.bn);
        // (the pair's 256-column tile sums a chunk in one run, for want of registers: it is taken
        // with the most chunks only, so that no run is longer than it has to be. Distance from the
        // 64-bit result in such runs and with 128 columns in runs of about the square root: 512
        // half tokens x 9677 slots, d = 5120, 3 chunks 8.6e-7 and 7.1e-7; 2048 x 7706, d = 4096,
        // where one chunk is all there is, 9.9e-7 and 6.5e-7 in half, 2.62e-6 and 2.53e-6 in bf16,
        // 417 and 445 us, 393 and 433 us)
        for (int64_t ks = exact && c == 0 ? rows : 1; ks <= rows && ks <= steps; ++ks) {
            const double cost = (double)(cdiv(tiles * ks, num_cu) * cdiv(steps, ks) * tl.cost) +
                                2e-4 * (double)(B * d) * (double)(ks - 1) + (ks > 1 ? 300. : 0.);
            if (cost < bc) bc = cost, p.g2 = c, p.KS = (int)ks;
        }
    }
    const G2Tile& t2 = exact ? kG2Exact[p.g2] : kG2Tiles[p.g2];
    p.ntm2 = (int)cdiv(B, t2.bm);
    p.ntn2 = (int)cdiv(d, t2.bn);
}

// exact: H as a hi + lo pair (SI_FLAG_EXACT_H), else one 16-bit value (no lo plane)
TPlan make_tplan(int64_t B, int64_t L, int64_t d, int num_cu, bool exact) {
    TPlan p;
    p.W = (L + 31) / 32;
    p.Lp = p.W * 32;
    p.Up = (L + kBK - 1) / kBK * kBK;
    pick_tiles(p, B, L, d, num_cu, exact, partial_rows(B, L, d, num_cu));
    size_t o = 0;
    p.off_bits = o;
    o = align256(o + (size_t)B * p.W * 4);
    // Up to 2048 tokens and 32768 slots every GEMM1 work-group ORs the blocks and scans the
    // union words in its prologue (about 1 us) instead of a launch of one work-group before it
    // (8 us). More tokens would make its reads as long as that launch's.
    p.scan = p.W <= kScanWords && B <= 2048;
    p.nb = (B + 63) / 64;
    p.off_words = o;
    o = align256(o + (size_t)p.nb * p.W * 4);
    p.off_ulist = o;
    o = align256(o + (size_t)p.Lp * 4);
    p.off_count = o;
    o = align256(o + 4);
    p.off_hhi = o;
    o = align256(o + (size_t)B * p.Up * 2);
    p.off_hlo = o;
    if (exact) o = align256(o + (size_t)B * p.Up * 2);
    p.off_part = o;
    o = align256(o + (size_t)(p.KS - 1) * B * part_chunks(d) * kChunk * 4);
    p.total = o;
    return p;
}

// The plan a call takes. Its nnz ids are at most nnz slots of the union: with fewer than a third
// as many ids as slots the tiles are chosen for those, in the workspace of all (446 half tokens
// with 3 ids each of 28190 slots, d = 2048: 82.3 us with the tiles for all, 51.8 so; 622 x 3 of
// 26818, d = 512 57.7 / 43.2). Of random sets with fewer, a half is over 4% faster and 1 in 500
// slower; from 0.4 on the ids say less of the union (often half of them), and 1 in 25 is slower, by
// up to a quarter, where the rounds of work-groups for it fall badly.
TPlan launch_tplan(int64_t B, int64_t nnz, int64_t L, int64_t d, int num_cu, bool exact) {
    TPlan p = make_tplan(B, L, d, num_cu, exact);
    if (3 * nnz < L) pick_tiles(p, B, nnz > 0 ? nnz : 1, d, num_cu, exact, p.KS);
    return p;
}

}  // namespace

hipError_t launch_bits_to_list(const uint32_t* bits, int64_t W, int32_t* list, int* count,
                               hipStream_t s) {
    hipLaunchKernelGGL(union_scan, dim3(1), dim3(1024), (unsigned)(W * 4), s, bits, (int64_t)1, W,
                       list, count);
    return hipGetLastError();
}

// compute units of the current device, looked up once per device
int current_cu_count() {
    static std::atomic<int> cache[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

int activation_tiles(int64_t T, int64_t L) {
    return (int)cdiv(T, kG1Tiles[gemm1_pick(T, L, current_cu_count())].bm);
}
int activation_tiles_max(int64_t T) { return (int)((T + 127) / 128); }
void activation_tile(int64_t T, int64_t L, int32_t* tile) {
    const G1Tile& t = kG1Tiles[gemm1_pick(T, L, current_cu_count())];
    tile[0] = t.bm;
    tile[1] = t.bn;
}

bool tiled_supported(int64_t B, int64_t L, int64_t d) {
    const int64_t Up = (L + kBK - 1) / kBK * kBK;
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit buffer offsets; the token bitmaps are built in LDS (at most 64 KB), and the union
    // scan keeps the union words and its 16 wave totals there (W * 4 + 64 <= 64 KB)
    return L * 2 * d * 2 < lim && B * d * 2 < lim && B * Up * 2 < lim && L <= 523776;
}

// The tiled path is compute bound: by default H enters GEMM2 as one 16-bit value (about 8
// significant bits for bf16; GEMM2 then does half the MFMA work); SI_FLAG_EXACT_H asks for the
// hi + lo pair, SI_FLAG_FAST_H for the single value explicitly.
bool tiled_exact_h(int flags) { return (flags & SI_FLAG_EXACT_H) && !(flags & SI_FLAG_FAST_H); }

size_t tiled_workspace(int64_t B, int64_t L, int64_t d, int num_cu, int flags) {
    return make_tplan(B, L, d, num_cu, tiled_exact_h(flags)).total;
}

void tiled_tiles(int64_t B, int64_t nnz, int64_t L, int64_t d, int num_cu, int flags,
                 int32_t* plan) {
    const bool exact = tiled_exact_h(flags);
    const TPlan p = launch_tplan(B, nnz, L, d, num_cu, exact);
    const G1Tile& g1 = kG1Tiles[p.g1];
    const G2Tile& g2 = exact ? kG2Exact[p.g2] : kG2Tiles[p.g2];
    const int32_t out[6] = {2, g1.bm, g1.bn, g2.bm, g2.bn, p.KS};
    for (int i = 0; i < 6; ++i) plan[i] = out[i];
}

template <typename ET>
hipError_t launch_union_tiled_t(const void* x, int64_t B, int64_t d, const int32_t* offsets,
                                const int32_t* idx, int64_t nnz, const void* gate_up_c,
                                const void* down_c, int64_t L, float* y, void* ws, int flags,
                                int num_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const bool fast = !tiled_exact_h(flags);
    const TPlan p = launch_tplan(B, nnz, L, d, num_cu, !fast);
    uint8_t* base = static_cast<uint8_t*>(ws);
    uint32_t* bits = reinterpret_cast<uint32_t*>(base + p.off_bits);
    uint32_t* words = reinterpret_cast<uint32_t*>(base + p.off_words);
    int32_t* ulist = reinterpret_cast<int32_t*>(base + p.off_ulist);
    int* ucount = reinterpret_cast<int*>(base + p.off_count);
    uint16_t* hhi = reinterpret_cast<uint16_t*>(base + p.off_hhi);
    uint16_t* hlo = fast ? nullptr : reinterpret_cast<uint16_t*>(base + p.off_hlo);
    float* part = reinterpret_cast<float*>(base + p.off_part);
    const uint16_t* xx = static_cast<const uint16_t*>(x);
    const uint16_t* gu = static_cast<const uint16_t*>(gate_up_c);
    const uint16_t* dc = static_cast<const uint16_t*>(down_c);

    hipError_t e = launch_token_bitmaps(offsets, idx, nnz, B, L, p.W, bits, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(or_blocks, dim3((unsigned)((p.W + 63) / 64), (unsigned)p.nb), dim3(256), 0,
                       s, bits, B, p.W, words);
    if (!p.scan)
        hipLaunchKernelGGL(union_scan, dim3(1), dim3(1024), (unsigned)(p.W * 4), s, words, p.nb,
                           p.W, ulist, ucount);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nb1 = p.scan ? (int)p.nb : 0;
    const dim3 g1((unsigned)((int64_t)p.nst * p.ntm1 + 7) / 8 * 8);
#define SI_G1(BM, BN, WT, WW, NX, NWT)                                                                \
    hipExtLaunchKernelGGL((gemm1_pipe<ET, kUnion, BM, BN, WT, WW, NX, NWT>), g1, dim3(64 * WT * WW),  \
                          0, s, ev0, nullptr, 0, xx, B, d, gu, L, ulist, ucount, words, nb1, bits, p.W, hhi, \
                          hlo, p.Up, p.ntm1, nullptr, nullptr)
    switch (p.g1) {
        case 0: SI_G1(256, 256, 2, 4, 2, 3); break;
        case 1: SI_G1(256, 192, 2, 4, 2, 3); break;
        case 2: SI_G1(256, 160, 4, 2, 3, 3); break;
        case 3: SI_G1(128, 256, 2, 4, 3, 3); break;
        default: SI_G1(128, 160, 2, 2, 4, 4); break;
    }
#undef SI_G1
    const dim3 g2((unsigned)((int64_t)p.ntm2 * p.ntn2 * p.KS + 7) / 8 * 8);
#define SI_G2(PL, BM, BN, WT, WW, NH, ND)                                                            \
    hipExtLaunchKernelGGL((gemm2_pipe<ET, true, PL, BM, BN, WT, WW, NH, ND>), g2,               \
                          dim3(64 * WT * WW), 0, s, nullptr, ev1, 0, hhi, hlo, p.Up, B, dc, d, L, \
                          ulist, ucount, nullptr, (int64_t)0, y, part, p.KS, p.ntm2, p.ntn2)
    if (!fast && p.g2 == 0)
        SI_G2(2, 128, 256, 2, 4, 2, 3);
    else if (!fast)
        SI_G2(2, 128, 128, 4, 2, 3, 3);
    else if (p.g2 == 0)
        SI_G2(1, 256, 256, 2, 4, 2, 3);
    else if (p.g2 == 1)
        SI_G2(1, 256, 128, 2, 4, 3, 3);
    else
        SI_G2(1, 128, 128, 2, 2, 4, 4);
#undef SI_G2
    return launch_add_partials(part, p.KS - 1, B, d, y, s);
}

template <typename ET>
hipError_t launch_activations_mfma_t(const void* x, int64_t T, int64_t d, const void* gate_up_c,
                                     int64_t L, float* out, int64_t ldo, int score, hipStream_t s,
                                     hipEvent_t ev0, hipEvent_t ev1) {
    if (T == 0 || L == 0) return hipSuccess;
    const int c = gemm1_pick(T, L, current_cu_count());
    const int ntm = (int)cdiv(T, kG1Tiles[c].bm);
    const int64_t nst = cdiv(L, kG1Tiles[c].bn / 2);
    const uint16_t* xx = static_cast<const uint16_t*>(x);
    const uint16_t* gu = static_cast<const uint16_t*>(gate_up_c);
#define SI_ACT_LAUNCH(MODE, BM, BN, WT, WW, NX, NWT)                                                 \
    hipExtLaunchKernelGGL((gemm1_pipe<ET, MODE, BM, BN, WT, WW, NX, NWT>),                           \
                          dim3((unsigned)(nst * ntm + 7) / 8 * 8), dim3(64 * WT * WW), 0, s, ev0, \
                          ev1, 0, xx, T, d, gu, L, nullptr, nullptr, nullptr, 0, nullptr, (int64_t)0, \
                          nullptr, nullptr, ldo, ntm, out, nullptr)
#define SI_ACT_TILES(MODE)                                                \
    switch (c) {                                                          \
        case 0: SI_ACT_LAUNCH(MODE, 256, 256, 2, 4, 2, 3); break;            \
        case 1: SI_ACT_LAUNCH(MODE, 256, 192, 2, 4, 2, 3); break;            \
        case 2: SI_ACT_LAUNCH(MODE, 256, 160, 4, 2, 3, 3); break;            \
        case 3: SI_ACT_LAUNCH(MODE, 128, 256, 2, 4, 3, 3); break;            \
        default: SI_ACT_LAUNCH(MODE, 128, 160, 2, 2, 4, 4); break;           \
    }
    if (score) {
        SI_ACT_TILES(kScore)
    } else {
        SI_ACT_TILES(kAct)
    }
#undef SI_ACT_TILES
#undef SI_ACT_LAUNCH
    return hipGetLastError();
}

hipError_t launch_union_tiled(const void* x, int64_t B, int64_t d, const int32_t* offsets,
                              const int32_t* idx, int64_t nnz, const void* gate_up_c,
                              const void* down_c, int64_t L, int et, float* y, void* ws,
                              int flags, int num_cu, hipStream_t s, hipEvent_t ev0,
                              hipEvent_t ev1) {
    if (et == 2)
        return launch_union_tiled_t<f16_t>(x, B, d, offsets, idx, nnz, gate_up_c, down_c, L, y,
                                           ws, flags, num_cu, s, ev0, ev1);
    return launch_union_tiled_t<bf16_t>(x, B, d, offsets, idx, nnz, gate_up_c, down_c, L, y, ws,
                                        flags, num_cu, s, ev0, ev1);
}

hipError_t launch_activations_mfma(const void* x, int64_t T, int64_t d, const void* gate_up_c,
                                   int64_t L, int et, float* out, int64_t ldo, int score,
                                   hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (et == 2)
        return launch_activations_mfma_t<f16_t>(x, T, d, gate_up_c, L, out, ldo, score, s, ev0,
                                                ev1);
    return launch_activations_mfma_t<bf16_t>(x, T, d, gate_up_c, L, out, ldo, score, s, ev0, ev1);
}

}  // namespace si
