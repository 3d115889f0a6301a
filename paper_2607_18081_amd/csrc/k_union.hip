// Union path of the selective SwiGLU FFN for a batch of B >= 2 tokens with bf16 weights and x.
//
// Each token b has its own active set A_b (Selective Computation section). Reading every
// token's rows separately would fetch a row once per token that uses it; instead the rows of
// the union U = A_1 u ... u A_B are read once and both projections become dense bf16 MFMA
// gather-GEMMs over U, with each token's h masked to its own set:
//
//   G, Uu = X[B][d] . gate_c[U]^T, X . up_c[U]^T         (GEMM1, fp32 accumulate)
//   H[b][n] = SiLU(G[b][n]) * Uu[b][n] * [U[n] in A_b]   (fused epilogue, fp32)
//   Y = H[B][|U|] . down_c[U]                             (GEMM2, fp32 accumulate)
//
// H enters GEMM2's bf16 MFMA as a pair hi = bf16(H), lo = bf16(H - hi), so the product keeps
// about 16 significant bits of H (SI_FLAG_FAST_H uses hi only).
//
// Kernels (the GEMMs are gemm_pipe.h's, without a union list):
//  - token bitmaps: one work-group per token marks its active slots in an L-bit bitmap;
//  - gemm1_pipe in its kWord mode: one work-group per tile of 32, 40, 48 or 64 slots and tile of
//    tokens. It ORs the slots' bitmap words over its tokens; rows of slots that none of them has
//    load nothing (their loads are out of range), and a tile without any writes zeros and ends. H
//    is written by slot, zero outside the tokens' sets;
//  - gemm2_pipe over K = slot: a tile of tokens x 128 or 256 columns, one of KS chunks of slots,
//    down rows outside the union again without memory traffic, steps of 64 slots without any
//    passed over. The KS sums are added in a fixed order (chunk 0 goes to y itself).
// For so few tokens both GEMMs stream the union's rows: they are bound by how much of HBM's
// latency the loads in flight cover, so the tiles are small and the stages many (60 to 160 KB
// of LDS a CU), and the row loads carry the non-temporal policy while one token tile reads each
// row (128 tokens x 524288 slots, d = 512 556 us, default policy 575; with several tiles the
// others then find fewer rows in L2: 300 tokens x 523900, d = 680 2267 / 2156 us).
#include <hip/hip_ext.h>

#include "common.h"
#include "gemm_pipe.h"
#include "launch.h"
#include "selectinfer.h"

namespace si {

namespace {

// Token tile by batch size: the smallest of 16, 32, 64 and 128 that holds the batch, since each
// token tile streams the union's rows again (more than 128 tokens take tiles of 128; few slots
// two of 64, see make_plan).

struct Plan {
    int64_t W;      // 32-bit words per token bitmap (slot s is bit s % 32 of word s / 32)
    int64_t Up;     // row stride of H, indexed by slot
    int bm;         // token tile
    int bn1;        // GEMM1 weight rows per work-group (two per slot)
    int bn2;        // GEMM2 columns per work-group
    int ntm, ntn;   // token and column tiles
    int KS;         // GEMM2 split-K chunks
    size_t off_bits, off_words, off_hhi, off_hlo, off_part, total;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

Plan make_plan(int64_t B, int64_t L, int64_t d, int num_cu) {
    Plan p;
    p.W = (L + 31) / 32;
    p.Up = (L + kBK - 1) / kBK * kBK;
    p.bm = B > 64 ? 128 : (B > 32 ? 64 : (B > 16 ? 32 : 16));
    // Where 32-slot work-groups of a 128-token tile would leave half the CUs idle, two tiles of 64
    // tokens: twice the work-groups at half the work, and the second reading of a row is from L2
    // (112 half tokens x 18 slots, d = 6224: 46 us with such tiles before the pipelined GEMMs, 57
    // with 128; 127 tokens x 1250 slots, d = 5120 63.3 us with 128 and 48.1 with 64, x 4096 73.5
    // and 58.9). Past 4096 slots it depends (65 and 127 tokens x 6000, d = 4096: 58.1 and 65.3 us
    // with 128, 60.2 and 62.4 with 64).
    if (p.bm == 128 && 2 * p.W <= num_cu) p.bm = 64;
    p.ntm = (int)((B + p.bm - 1) / p.bm);
    // GEMM1 slot tile: a work-group takes in (its tokens + its weight rows) x d, and a CU has
    // one at a time, so the least (rounds of work-groups) x (tokens + rows): with 303
    // work-groups of 32 slots, 47 CUs had two, and 45 tokens of a 13B layer took 57 us against
    // 39 us with 242 of 40 slots (198 MB of rows: 3.5 and 5.1 TB/s)
    p.bn1 = 64;
    int64_t best = INT64_MAX;
    for (int bn : {64, 80, 96, 128}) {
        const int64_t wgs = p.ntm * ((p.W * 32 + bn / 2 - 1) / (bn / 2));
        const int64_t cost = (wgs + num_cu - 1) / num_cu * (p.bm + bn);
        if (cost < best) best = cost, p.bn1 = bn;
    }
    // GEMM2 column tile: 256 (512 bytes of a down row), but 128 where the token tile's H is small
    // or where d has so few tiles of 256 that the partials of the many K chunks count (whole
    // call: 16 tokens, d = 4096 43.7 / 42.9 us; 12 and 100 tokens, d = 2048 25.4 / 23.3 and
    // 45.0 / 42.4 us; the other way 45 tokens, d = 5120 75.3 / 79.0 us, 100 tokens 92.2 / 96.8)
    p.bn2 = p.bm == 16 || d <= 2048 ? 128 : 256;
    p.ntn = (int)((d + p.bn2 - 1) / p.bn2);
    // chunks that fill the CUs once, each of at least one K step
    int64_t ks = num_cu / ((int64_t)p.ntm * p.ntn);
    if (ks > p.Up / kBK) ks = p.Up / kBK;
    if (ks > 64) ks = 64;
    if (ks < 1) ks = 1;
    p.KS = (int)ks;
    size_t o = 0;
    p.off_bits = o;
    o = align256(o + (size_t)B * p.W * 4);
    p.off_words = o;
    o = align256(o + (size_t)p.ntm * p.W * 4);
    p.off_hhi = o;
    o = align256(o + (size_t)B * p.Up * 2);
    p.off_hlo = o;
    o = align256(o + (size_t)B * p.Up * 2);
    p.off_part = o;
    // Where that many chunks' partials alone would take the call past si_selective_ffn_noalloc's
    // scratch, as few less as fit, down to half (127 tokens x 71117 slots, d = 4264: 67.7 MB with
    // 15 chunks; a batch of 65 to 127 tokens once had two token tiles and half the chunks, and is
    // taken as it was then)
    const size_t row = (size_t)B * part_chunks(d) * kChunk * 4;  // partials of a chunk
    const size_t room = o < SI_NOALLOC_SCRATCH_BYTES ? SI_NOALLOC_SCRATCH_BYTES - o : 0;
    const int64_t fit = (int64_t)(room / row) + 1;  // (chunk 0 has none)
    if (o <= SI_NOALLOC_SCRATCH_BYTES && fit < p.KS && fit >= (p.KS + 1) / 2) p.KS = (int)fit;
    o = align256(o + (size_t)(p.KS - 1) * row);
    p.total = o;
    return p;
}

__device__ __forceinline__ void clamp_range(const int32_t* offsets, int64_t b, int64_t nnz,
                                            int64_t& lo, int64_t& hi) {
    lo = offsets[b];
    hi = offsets[b + 1];
    lo = lo < 0 ? 0 : (lo > nnz ? nnz : lo);
    hi = hi < lo ? lo : (hi > nnz ? nnz : hi);
}

// Token b's active slots as a bitmap (LDS), written to bits[b][0..W). The ids are read 4096
// at a time, four range-checked loads per thread issued together, so a token's list costs one
// memory round trip per 4096 ids rather than one per 256.
constexpr int kBmThreads = 1024;
__global__ __launch_bounds__(kBmThreads) void token_bitmaps(const int32_t* __restrict__ offsets,
                                                            const int32_t* __restrict__ idx,
                                                            int64_t nnz, int64_t L, int64_t W,
                                                            uint32_t* __restrict__ bits) {
    extern __shared__ uint32_t bm[];
    constexpr int U = 4;
    const int64_t b = blockIdx.x;
    for (int64_t q = threadIdx.x; q < W; q += kBmThreads) bm[q] = 0u;
    int64_t lo, hi;
    clamp_range(offsets, b, nnz, lo, hi);
    __syncthreads();
    for (int64_t r0 = lo; r0 < hi; r0 += (int64_t)kBmThreads * U) {
        const int64_t nr = hi - r0 < (int64_t)kBmThreads * U ? hi - r0 : (int64_t)kBmThreads * U;
        const __amdgpu_buffer_rsrc_t ri = make_rsrc(idx + r0, nr * 4);
        int32_t sv[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            sv[u] = __builtin_amdgcn_raw_buffer_load_b32(ri, (u * kBmThreads + (int)threadIdx.x) * 4,
                                                         0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t sl = sv[u];
            if (u * kBmThreads + (int)threadIdx.x < nr && sl >= 0 && sl < L)
                atomicOr(&bm[sl >> 5], 1u << (sl & 31));
        }
    }
    __syncthreads();
    for (int64_t q = threadIdx.x; q < W; q += kBmThreads) bits[b * W + q] = bm[q];
}

}  // namespace

hipError_t launch_token_bitmaps(const int32_t* offsets, const int32_t* idx, int64_t nnz,
                                int64_t B, int64_t L, int64_t W, uint32_t* bits, hipStream_t s) {
    hipLaunchKernelGGL(token_bitmaps, dim3((unsigned)B), dim3(kBmThreads), (size_t)W * 4, s,
                       offsets, idx, nnz, L, W, bits);
    return hipGetLastError();
}

// Batches from which the LDS-tiled GEMMs (k_tiled.hip) take over, and with them h as one 16-bit
// value, half of H's workspace. Past 128 tokens the row-word kernels read every row once per token
// tile: 129 tokens x 7706 slots, d = 4096 78 us tiled and 86 by words, x 9677, d = 5120 101 and 147.
// 128 tokens fit one token tile and would be faster by words (88 and 71 us, 110 and 95, with the
// hi + lo pair), as would up to 256 tokens over 2000 slots (d = 4096: 71 and 46 us), but the form of
// h from 128 tokens on, and what fits a given scratch there, are part of the interface.
constexpr int64_t kTiledMinB = 128;

static bool use_tiled(int64_t B, int64_t L, int64_t d) {
    return B >= kTiledMinB && tiled_supported(B, L, d);
}

bool union_supported(int64_t B, int64_t L, int64_t d) {
    // buffer loads take 32-bit byte offsets
    return L * 2 * d * 2 < ((int64_t)1 << 31) && B * d * 2 < ((int64_t)1 << 31) &&
           L <= 524288 && B * ((L + 31) / 32) * 4 < ((int64_t)1 << 31);
}

size_t union_workspace(int64_t B, int64_t L, int64_t d, int num_cu, int flags) {
    if (use_tiled(B, L, d)) return tiled_workspace(B, L, d, num_cu, flags);
    return make_plan(B, L, d, num_cu).total;
}

void union_tiles(int64_t B, int64_t nnz, int64_t L, int64_t d, int num_cu, int flags,
                 int32_t* plan) {
    if (use_tiled(B, L, d)) return tiled_tiles(B, nnz, L, d, num_cu, flags, plan);
    const Plan p = make_plan(B, L, d, num_cu);
    const int32_t out[6] = {1, p.bm, p.bn1, p.bm, p.bn2, p.KS};
    for (int i = 0; i < 6; ++i) plan[i] = out[i];
}

namespace {

template <typename ET>
hipError_t launch_union_t(const void* x, int64_t B, int64_t d, const int32_t* offsets,
                          const int32_t* idx, int64_t nnz, const void* gate_up_c,
                          const void* down_c, int64_t L, float* y, void* ws, int flags,
                          int num_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const Plan p = make_plan(B, L, d, num_cu);
    uint8_t* base = static_cast<uint8_t*>(ws);
    uint32_t* bits = reinterpret_cast<uint32_t*>(base + p.off_bits);
    uint32_t* words = reinterpret_cast<uint32_t*>(base + p.off_words);
    uint16_t* hhi = reinterpret_cast<uint16_t*>(base + p.off_hhi);
    const bool fast = (flags & SI_FLAG_FAST_H) != 0;  // h as one 16-bit value: no lo plane
    uint16_t* hlo = fast ? nullptr : reinterpret_cast<uint16_t*>(base + p.off_hlo);
    float* part = reinterpret_cast<float*>(base + p.off_part);
    const uint16_t* xx = static_cast<const uint16_t*>(x);
    const uint16_t* gu = static_cast<const uint16_t*>(gate_up_c);
    const uint16_t* dc = static_cast<const uint16_t*>(down_c);

    hipError_t e = launch_token_bitmaps(offsets, idx, nnz, B, L, p.W, bits, s);
    if (e != hipSuccess) return e;
    const dim3 g2((unsigned)((int64_t)p.ntm * p.ntn * p.KS + 7) / 8 * 8);
    const dim3 g1((unsigned)(p.ntm * ((p.W * 32 + p.bn1 / 2 - 1) / (p.bn1 / 2)) + 7) / 8 * 8);
    // (token tiles below 64 hold the whole batch, and so do those of 64 with slot tiles over 32)
    const bool once = p.ntm == 1;
#define SI_G1(BM, BN, WT, WW, NX, ONCE)                                                          \
    hipExtLaunchKernelGGL((gemm1_pipe<ET, kWord, BM, BN, WT, WW, NX, NX, ONCE>), g1,             \
                          dim3(64 * WT * WW), 0, s, ev0, nullptr, 0, xx, B, d, gu, L, nullptr,   \
                          nullptr, nullptr, 0, bits, p.W, hhi, hlo, p.Up, p.ntm, nullptr, words)
#define SI_G1_TILES(BM, BN, WT, WW, NX)                                                          \
    if (once) SI_G1(BM, BN, WT, WW, NX, true); else SI_G1(BM, BN, WT, WW, NX, false)
#define SI_G2_PL(PL, BM, BN, WT, WW, NH, ND, ONCE)                                               \
    hipExtLaunchKernelGGL((gemm2_pipe<ET, false, PL, BM, BN, WT, WW, NH, ND, ONCE>), g2,         \
                          dim3(64 * WT * WW), 0, s, nullptr, ev1, 0, hhi, hlo, p.Up, B, dc, d, L, \
                          nullptr, nullptr, words, p.W, y, part, p.KS, p.ntm, p.ntn)
#define SI_G2(BM, BN, WT, WW, NH, ND, ONCE)                                                      \
    if (fast) SI_G2_PL(1, BM, BN, WT, WW, NH, ND, ONCE);                                         \
    else SI_G2_PL(2, BM, BN, WT, WW, NH, ND, ONCE)
#define SI_G2_TILES(BM, BN, WT, WW, NH, ND)                                                      \
    if (once) {                                                                                  \
        SI_G2(BM, BN, WT, WW, NH, ND, true);                                                     \
    } else {                                                                                     \
        SI_G2(BM, BN, WT, WW, NH, ND, false);                                                    \
    }
    switch (p.bm * 1000 + p.bn1) {
        case 16064: SI_G1(16, 64, 1, 2, 8, true); break;
        case 16080: SI_G1(16, 80, 1, 1, 5, true); break;
        case 16096: SI_G1(16, 96, 1, 2, 8, true); break;
        case 16128: SI_G1(16, 128, 1, 2, 7, true); break;
        case 32064: SI_G1(32, 64, 2, 2, 8, true); break;
        case 32080: SI_G1(32, 80, 2, 1, 8, true); break;
        case 32096: SI_G1(32, 96, 2, 2, 8, true); break;
        case 32128: SI_G1(32, 128, 2, 2, 7, true); break;
        case 64064: SI_G1_TILES(64, 64, 2, 2, 8); break;
        case 64080: SI_G1(64, 80, 4, 1, 8, true); break;
        case 64096: SI_G1(64, 96, 2, 2, 7, true); break;
        case 64128: SI_G1(64, 128, 2, 2, 6, true); break;
        case 128064: SI_G1_TILES(128, 64, 2, 2, 6); break;
        case 128080: SI_G1_TILES(128, 80, 4, 1, 6); break;
        case 128096: SI_G1_TILES(128, 96, 2, 2, 5); break;
        default: SI_G1_TILES(128, 128, 2, 2, 4); break;
    }
    switch (p.bm * 1000 + p.bn2) {
        // (three stages: eight, and no wait for the union words to hold them back, read HBM more
        // slowly. 16 tokens x 7706 slots, d = 4096 45.3 / 44.6 / 44.4 / 43.7 / 48.4 us with 8, 6, 4,
        // 3 and 2 stages, x 28672, d = 5120 172.2 / 171.2 / 170.2 / 169.0 with 8, 6, 4 and 3)
        case 16128: SI_G2(16, 128, 1, 4, 3, 3, true); break;
        case 32128: SI_G2(32, 128, 1, 4, 6, 6, true); break;
        case 32256: SI_G2(32, 256, 1, 4, 4, 4, true); break;
        case 64128: SI_G2_TILES(64, 128, 2, 2, 5, 5); break;
        case 64256: SI_G2_TILES(64, 256, 2, 4, 3, 3); break;
        case 128128: SI_G2_TILES(128, 128, 4, 2, 3, 3); break;
        default: SI_G2_TILES(128, 256, 2, 4, 2, 3); break;
    }
#undef SI_G1_TILES
#undef SI_G2_TILES
#undef SI_G1
#undef SI_G2
#undef SI_G2_PL
    return launch_add_partials(part, p.KS - 1, B, d, y, s);
}

}  // namespace

hipError_t launch_union(const void* x, int64_t B, int64_t d, const int32_t* offsets,
                        const int32_t* idx, int64_t nnz, const void* gate_up_c,
                        const void* down_c, int64_t L, int et, float* y, void* ws, int flags,
                        int num_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (use_tiled(B, L, d))
        return launch_union_tiled(x, B, d, offsets, idx, nnz, gate_up_c, down_c, L, et, y, ws,
                                  flags, num_cu, s, ev0, ev1);
    if (et == 2)
        return launch_union_t<f16_t>(x, B, d, offsets, idx, nnz, gate_up_c, down_c, L, y, ws,
                                     flags, num_cu, s, ev0, ev1);
    return launch_union_t<bf16_t>(x, B, d, offsets, idx, nnz, gate_up_c, down_c, L, y, ws, flags,
                                  num_cu, s, ev0, ev1);
}

}  // namespace si
