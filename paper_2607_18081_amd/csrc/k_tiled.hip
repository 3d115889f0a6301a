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
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "mfma.h"
#include "pipe.h"
#include "selectinfer.h"

namespace si {

namespace {

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;

constexpr int kBK = 64;          // K step (elements)

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

// ---- GEMM1 ---------------------------------------------------------------------------------
// MODE selects what the epilogue produces (the product itself is the same):
//   kUnion:  h masked by the token bitmaps, over the union list, as 16-bit hi (and lo) planes;
//   kAct:    the activation of every slot (the union list is the identity, no mask), float32
//            out[tok * Up + slot];
//   kScore:  Eq. 1 for this work-group's tokens: sum over its BM tokens of |a| per slot, added
//            in a fixed order, float32 out[tm * Up + slot] (one partial row per token tile; the
//            host-side reducer adds the rows in order).
enum { kUnion = 0, kAct = 1, kScore = 2 };

// Token bitmap words a work-group keeps in LDS for the mask (per token; pitch odd so that 16
// tokens' words lie in different banks)
constexpr int kWin = 16, kWinP = kWin + 1;

// BM tokens x BN weight rows (BN / 2 union slots); WT x WW waves of FT x FW 16x16 MFMA tiles,
// the weight rows as the M operand, so a lane ends up with 4 consecutive weight rows of one
// token. Those are 2 gate and 2 up rows of the same two slots, so SiLU * up needs no data
// exchange. NX LDS stages of x and NWT of the weight rows, which come from HBM and are given
// the longer flight where the LDS cannot hold a third stage of both (256 x 256).
template <typename ET, int MODE, int BM, int BN, int WT, int WW, int NX, int NWT>
__global__ __launch_bounds__(64 * WT * WW) void gemm1_pipe(
    const uint16_t* __restrict__ x, int64_t B, int64_t d, const uint16_t* __restrict__ gu, int64_t L,
    const int32_t* __restrict__ ulist, const int* __restrict__ ucount,
    const uint32_t* __restrict__ bits, int64_t W, uint16_t* __restrict__ Hhi,
    uint16_t* __restrict__ Hlo, int64_t Up, int ntm, float* __restrict__ out) {
    constexpr int NW = WT * WW, kThr = 64 * NW;
    constexpr int FT = BM / (16 * WT), FW = BN / (16 * WW);
    constexpr int kS = BN / 2;
    // 1 KB pieces (8 rows) of a stage, and how many of them a wave loads (the last of a
    // wave's weight pieces may be left to the lower waves: kPart of them)
    constexpr int RX = BM / 8, RW = BN / 8, LX = RX / NW, LW = RW / NW, kPart = RW % NW;
    constexpr bool kSplit = NWT > NX;
    constexpr int kPer = kSplit ? NX * NWT : NX;  // steps after which the stages come round
    static_assert(RX % NW == 0 && NX >= 2 && NX <= 4, "tile");
    static_assert(NWT == NX || (NX == 2 && NWT == 3 && kPart == 0), "stages");
    typedef typename Mfma<ET>::vec8 vec8;
    // one array per stage: the compiler then sees that a stage's reads do not touch the stages
    // being loaded, and waits for nothing between them
    __shared__ __align__(1024) char x0[RX * 1024];
    __shared__ __align__(1024) char x1[RX * 1024];
    __shared__ __align__(1024) char x2[NX > 2 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x3[NX > 3 ? RX * 1024 : 16];
    __shared__ __align__(1024) char w0[RW * 1024];
    __shared__ __align__(1024) char w1[RW * 1024];
    __shared__ __align__(1024) char w2[NWT > 2 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w3[NWT > 3 ? RW * 1024 : 16];

    const int nU = MODE == kUnion ? *ucount : (int)L;
    int tm, st;
    if (!xcd_tile((int)blockIdx.x, ntm, (nU + kS - 1) / kS, tm, st)) return;  // uniform
    const int64_t m0 = (int64_t)tm * BM, u0 = (int64_t)st * kS;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nn = lane & 15;
    const int g = lane >> 4;
    const int wt = w % WT, ww = w / WT;

    // slot of union position u0 + p, -1 past the union
    const __amdgpu_buffer_rsrc_t rul = make_rsrc(ulist, MODE == kUnion ? (int64_t)nU * 4 : 0);
    auto union_slot = [&](int p) -> int32_t {
        const int u = (int)u0 + p;
        int32_t sl = u;
        if constexpr (MODE == kUnion)
            sl = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rul, u * 4, 0, 0);
        return (u < nU && (unsigned)sl < (unsigned)L) ? sl : -1;
    };
    // weight row 16 f + 4 q + e of the tile (e < 4): plane e / 2 (gate, up) of slot
    // slot_of(f, q, e % 2). A wave's tiles f come in pairs, over which a lane's slots are four
    // consecutive ones (an odd last tile: two), for wide stores of h.
    auto slot_of = [&](int f, int q, int e) {
        const int i = f % FW, base = (f / FW) * 8 * FW;
        return i < (FW & ~1) ? base + 16 * (i / 2) + 4 * q + 2 * (i & 1) + e
                             : base + 8 * i + 2 * q + e;
    };
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(x, B * d * 2);
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(gu, L * 2 * d * 2);
    // Piece p: rows 8 p + lane / 8, 128 bytes (a K step) each. The 16-byte chunk c of row r is
    // kept at position c ^ (r % 8), so that the fragment reads of 16 rows at one chunk meet no
    // bank conflicts; the loads place it so by what each lane reads.
    const int cb = ((lane & 7) ^ (lane >> 3)) * 16;
    int xoff[LX], woff[LW + 1];
#pragma unroll
    for (int j = 0; j < LX; ++j) {
        const int64_t tok = m0 + 8 * (j * NW + w) + (lane >> 3);
        xoff[j] = tok < B ? (int)(tok * d * 2) + cb : kOOB;
    }
#pragma unroll
    for (int j = 0; j < LW + (kPart ? 1 : 0); ++j) {
        const int r = 8 * (j * NW + w) + (lane >> 3);  // (past the tile: not loaded)
        const int32_t sl = union_slot(slot_of(r / 16, (r % 16) / 4, r & 1));
        woff[j] = sl >= 0 ? (int)(((int64_t)sl * 2 + ((r >> 1) & 1)) * d * 2) + cb : kOOB;
    }
    // the mask's window: kWin bitmap words from the first slot's on, unless the tile's slots
    // span more
    int win0 = 0;
    bool in_win = false;
    if constexpr (MODE == kUnion) {
        const int last = (int)(nU - u0 < kS ? nU - u0 : kS) - 1;
        win0 = __builtin_amdgcn_readfirstlane(ulist[u0] >> 5);
        in_win = __builtin_amdgcn_readfirstlane(ulist[u0 + last] >> 5) - win0 < kWin;
    }

    const int nk = (int)((d + kBK - 1) / kBK);
    // loads of step k into stage s: what lies past d reads as zeros (d % 8 == 0: a chunk is all
    // in or all out)
    auto load_x = [&](int k, char* s) {
        const bool ok = k * 128 + cb < (int)(d * 2);
#pragma unroll
        for (int j = 0; j < LX; ++j)
            load_lds16(rx, s + (j * NW + w) * 1024, ok ? xoff[j] : kOOB, k * 128);
    };
    auto load_w = [&](int k, char* s) {
        const bool ok = k * 128 + cb < (int)(d * 2);
#pragma unroll
        for (int j = 0; j < LW; ++j)
            load_lds16(rg, s + (j * NW + w) * 1024, ok ? woff[j] : kOOB, k * 128);
    };
    // the pieces that only waves below kPart have: loaded before the others of the same step,
    // so that the counted waits hold for every wave
    auto load_part = [&](int k, char* s) {
        if constexpr (kPart != 0) {
            const bool ok = k * 128 + cb < (int)(d * 2);
            if (w < kPart)
                load_lds16(rg, s + (LW * NW + w) * 1024, ok ? woff[LW] : kOOB, k * 128);
        }
    };

    f32x4_t acc[FW][FT];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < FT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // fragments of the two halves (K = 32) of a step
    vec8 ft[2][FT], fw[2][FW];
    const int to = (wt * 16 * FT + nn) * 128, wo = (ww * 16 * FW + nn) * 128;
    const int c0 = (g ^ (nn & 7)) * 16, c1 = ((4 + g) ^ (nn & 7)) * 16;
    auto frags = [&](const char* sx, const char* sw, int h) {
        const int c = h ? c1 : c0;
#pragma unroll
        for (int i = 0; i < FW; ++i) fw[h][i] = Mfma<ET>::vec(ld16(sw + wo + i * 2048 + c));
#pragma unroll
        for (int j = 0; j < FT; ++j) ft[h][j] = Mfma<ET>::vec(ld16(sx + to + j * 2048 + c));
    };
    auto mults = [&](int h) {
#pragma unroll
        for (int j = 0; j < FT; ++j)
#pragma unroll
            for (int i = 0; i < FW; ++i) acc[i][j] = Mfma<ET>::mma(fw[h][i], ft[h][j], acc[i][j]);
    };
    char* const xs[4] = {x0, x1, x2, x3};
    char* const ws[4] = {w0, w1, w2, w3};
    // One K step k = q mod kPer. The first half's fragments are in registers. The second half's
    // are read under the first half's MFMAs; then every wave has read all of step k's stages
    // and, past the barrier, they take the loads of step k + NX (k + NWT), while the next
    // step's first fragments are read under the second half's MFMAs. One barrier a step, and
    // every wave holds the fragments of half a step when it meets it. With kSplit the weight
    // loads go out in the next step's first half instead: behind the x loads, so that a wait
    // for those leaves the later weight loads in flight.
    constexpr int NM = FT * FW, NR = FT + FW;
    constexpr int LA = kSplit ? LW : 0, LB = LX + (kSplit ? 0 : LW);  // loads in each half
    auto step = [&](int k, int q) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kSplit) load_w(k - 1 + NWT, ws[(q + NWT - 1) % NWT]);
        frags(xs[q % NX], ws[q % NWT], 1);
        mults(0);
#pragma unroll
        for (int i = 0; i < NR; ++i) {  // one LDS read (and load), then its share of the MFMAs
            if (i < LA) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NM / NR, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        wait_vm_lds<kSplit ? LW : (NX - 2) * (LX + LW)>();  // the next step's loads have landed
        wg_barrier();
        load_part(k + NWT, ws[q % NWT]);
        __builtin_amdgcn_sched_barrier(0);
        load_x(k + NX, xs[q % NX]);
        if constexpr (!kSplit) load_w(k + NWT, ws[q % NWT]);
        frags(xs[(q + 1) % NX], ws[(q + 1) % NWT], 0);
        mults(1);
#pragma unroll
        for (int i = 0; i < (NR > LB ? NR : LB); ++i) {
            if (i < LB) {
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
            if (i < NR) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
        asm volatile("" ::: "memory");
    };
    // (with kSplit a step's first half issues the weights of step k + NWT - 1: those of step
    // NWT - 1 are left to step 0)
#pragma unroll
    for (int q = 0; q < NX; ++q) {
        load_part(q, ws[q]);
        load_x(q, xs[q]);
        load_w(q, ws[q]);
        __builtin_amdgcn_sched_barrier(0);  // the counted waits rely on the stages' order
    }
    wait_vm_lds<(NX - 1) * (LX + LW)>();
    wg_barrier();
    frags(x0, w0, 0);
    int k = 0;
    for (; k + kPer <= nk; k += kPer) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) step(k + q, q);
    }
#pragma unroll
    for (int q = 0; q < kPer - 1; ++q)
        if (k + q < nk) step(k + q, q);

    // The stages are done with (nothing is in flight to them either): their memory takes the
    // epilogue's tables.
    wait_vm_lds<0>();
    wg_barrier();
    int32_t* const sslot = reinterpret_cast<int32_t*>(w0);       // the tile's slots
    uint32_t* const swin = reinterpret_cast<uint32_t*>(x0);      // the mask's window
    double* const ssum = reinterpret_cast<double*>(x0);          // kScore: sums per wave row
    static_assert(BM * kWinP * 4 <= RX * 1024 && WT * kS * 8 <= RX * 1024 && kS <= kThr, "tables");
    if (t < kS) sslot[t] = union_slot(t);
    if constexpr (MODE == kUnion) {
        if (in_win) {
            const __amdgpu_buffer_rsrc_t rbm = make_rsrc(bits, B * W * 4);
            constexpr int kWinQ = BM * kWin / kThr;
            uint32_t v[kWinQ];
#pragma unroll
            for (int q = 0; q < kWinQ; ++q) {
                const int e = q * kThr + t, wi = win0 + e % kWin;
                const int64_t tok = m0 + e / kWin;
                v[q] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                    rbm, (tok < B && wi < W) ? (int)((tok * W + wi) * 4) : kOOB, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < kWinQ; ++q) {
                const int e = q * kThr + t;
                swin[(e / kWin) * kWinP + e % kWin] = v[q];
            }
        }
    }
    __syncthreads();

    // element e of acc[i][j]: plane e / 2 of slot slot_of(ww FW + i, g, e % 2) for token
    // m0 + 16 (wt FT + j) + nn
    if constexpr (MODE == kScore) {
        // |a| summed over this lane's tokens, the 16 lanes nn, then the WT waves, each in a
        // fixed order, in float64 and rounded once (a few hundred adds a work-group; float32
        // sums of 256 tokens were 6.1e-8 from the 64-bit scores, of 128 tokens 5.7e-8)
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < FT; ++j) {
                    const int64_t tok = m0 + 16 * (wt * FT + j) + nn;
                    if (tok < B) v += (double)fabsf(silu_f32(acc[i][j][e]) * acc[i][j][2 + e]);
                }
                v += __shfl_xor(v, 1, kWave);
                v += __shfl_xor(v, 2, kWave);
                v += __shfl_xor(v, 4, kWave);
                v += __shfl_xor(v, 8, kWave);
                if (nn == 0) ssum[wt * kS + slot_of(ww * FW + i, g, e)] = v;
            }
        __syncthreads();
        if (t < kS && u0 + t < nU) {
            double a = ssum[t];
#pragma unroll
            for (int q = 1; q < WT; ++q) a += ssum[q * kS + t];
            out[(int64_t)tm * Up + u0 + t] = (float)a;
        }
        return;
    }
    const __amdgpu_buffer_rsrc_t rbm = make_rsrc(bits, MODE == kUnion ? B * W * 4 : 0);
    auto finish = [&](auto win) {
        constexpr int kLast = FW & 1 ? FW - 1 : FW;
#pragma unroll
        for (int i = 0; i < FW; i += 2) {
            const int np = i == kLast ? 1 : 2;  // tiles of this pair: 2 np consecutive slots
            const int64_t u = u0 + slot_of(ww * FW + i, g, 0);
            int32_t sl[4];
#pragma unroll
            for (int e = 0; e < 2 * np; ++e) sl[e] = sslot[slot_of(ww * FW + i, g, 0) + e];
#pragma unroll
            for (int j = 0; j < FT; ++j) {
                const int row = 16 * (wt * FT + j) + nn;
                const int64_t tok = m0 + row;
                float h[4];
#pragma unroll
                for (int e = 0; e < 2 * np; ++e) {
                    const f32x4_t& c = acc[i + e / 2][j];
                    h[e] = silu_f32(c[e & 1]) * c[2 + (e & 1)];
                }
                if constexpr (MODE == kAct) {
                    float* o = out + tok * Up + u;  // Up is a multiple of 4
                    if (tok < B && np == 2 && sl[3] >= 0) {
                        *reinterpret_cast<f32x4_t*>(o) = f32x4_t{h[0], h[1], h[2], h[3]};
                    } else if (tok < B) {
#pragma unroll
                        for (int e = 0; e < 2 * np; ++e)
                            if (sl[e] >= 0) o[e] = h[e];
                    }
                } else {
                    uint32_t hb[4], lb[4];
#pragma unroll
                    for (int e = 0; e < 2 * np; ++e) {
                        // a slot past the union, or one that is not in the token's set: h = 0
                        const int wi = sl[e] >> 5;
                        uint32_t word;
                        if constexpr (decltype(win)::value)
                            word = swin[row * kWinP + ((wi - win0) & (kWin - 1))];
                        else
                            word = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                                rbm, (tok < B && sl[e] >= 0) ? (int)((tok * W + wi) * 4) : kOOB, 0,
                                0);
                        const bool act = sl[e] >= 0 && ((word >> (sl[e] & 31)) & 1u);
                        h[e] = act ? h[e] : 0.0f;
                        hb[e] = Mfma<ET>::rne(h[e]);
                        lb[e] = Mfma<ET>::rne(h[e] - Mfma<ET>::widen(hb[e]));
                    }
                    // up to the end of this tile, so that the 8-wide chunk of GEMM2 that
                    // straddles the union's end holds zeros past it (Up is a multiple of 64)
                    if (tok < B && u < Up) {
                        uint32_t* ph = reinterpret_cast<uint32_t*>(Hhi + tok * Up + u);
#pragma unroll
                        for (int e = 0; e < np; ++e) ph[e] = hb[2 * e] | (hb[2 * e + 1] << 16);
                        if (Hlo) {  // the lo plane exists only for SI_FLAG_EXACT_H
                            uint32_t* pl = reinterpret_cast<uint32_t*>(Hlo + tok * Up + u);
#pragma unroll
                            for (int e = 0; e < np; ++e) pl[e] = lb[2 * e] | (lb[2 * e + 1] << 16);
                        }
                    }
                }
            }
        }
    };
    if (MODE != kUnion || in_win)
        finish(std::true_type());
    else
        finish(std::false_type());  // the tile's slots span more than kWin bitmap words
}

// ---- GEMM2 ---------------------------------------------------------------------------------
// BM tokens x BN columns of Y over one of KS chunks of the union, K = union position in steps
// of 64; WT x WW waves of FT x FW 16x16 MFMA tiles, the columns as the M operand, so a lane ends
// up with 4 consecutive columns of one token (16-byte stores). PL planes of H (1: one 16-bit
// value, 2: hi + lo). Chunk 0 goes to y, chunk p > 0 to row p - 1 of the partials.
template <typename ET, int PL, int BM, int BN, int WT, int WW, int NH, int ND>
__global__ __launch_bounds__(64 * WT * WW) void gemm2_pipe(
    const uint16_t* __restrict__ Hhi, const uint16_t* __restrict__ Hlo, int64_t Up, int64_t B,
    const uint16_t* __restrict__ dc, int64_t d, int64_t L, const int32_t* __restrict__ ulist,
    const int* __restrict__ ucount, float* __restrict__ y, float* __restrict__ part, int KS,
    int ntm, int ntn) {
    constexpr int NW = WT * WW;
    constexpr int FT = BM / (16 * WT), FW = BN / (16 * WW);
    // 1 KB pieces of a stage and how many of them a wave loads
    constexpr int RH = PL * BM / 8, RD = BN / 8, LH = RH / NW, LD = RD / NW;
    constexpr bool kSplit = ND > NH;
    constexpr int kPer = kSplit ? NH * ND : NH;  // steps after which the stages come round
    constexpr int kRow = 2 * BN;                 // bytes of a down row segment
    constexpr int kRpp = 1024 / kRow;            // down rows per piece
    static_assert((BN == 128 || BN == 256) && RH % NW == 0 && RD % NW == 0, "tile");
    static_assert(NH >= 2 && NH <= 4 && (ND == NH || (NH == 2 && ND == 3)), "stages");
    typedef typename Mfma<ET>::vec8 vec8;
    __shared__ __align__(1024) char h0[RH * 1024];
    __shared__ __align__(1024) char h1[RH * 1024];
    __shared__ __align__(1024) char h2[NH > 2 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h3[NH > 3 ? RH * 1024 : 16];
    __shared__ __align__(1024) char d0[RD * 1024];
    __shared__ __align__(1024) char d1[RD * 1024];
    __shared__ __align__(1024) char d2[ND > 2 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d3[ND > 3 ? RD * 1024 : 16];

    int tm, sc;
    if (!xcd_tile((int)blockIdx.x, ntm, ntn * KS, tm, sc)) return;  // uniform
    const int ks = __builtin_amdgcn_readfirstlane((int)((unsigned)sc / (unsigned)ntn));
    const int ct = sc - ks * ntn;
    const int nU = *ucount;
    const int kper = __builtin_amdgcn_readfirstlane(
        ((int)((unsigned)(nU + KS - 1) / (unsigned)KS) + kBK - 1) / kBK * kBK);
    const int kb = ks * kper;
    const int ke = kb + kper < nU ? kb + kper : nU;
    const int64_t n0 = (int64_t)ct * BN;
    const int64_t m0 = (int64_t)tm * BM;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nn = lane & 15;
    const int g = lane >> 4;
    const int wt = w % WT, ww = w / WT;

    const __amdgpu_buffer_rsrc_t rh = make_rsrc(Hhi, B * Up * 2);
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(PL == 2 ? Hlo : Hhi, B * Up * 2);
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(dc, L * d * 2);
    const __amdgpu_buffer_rsrc_t ru = make_rsrc(ulist, (int64_t)(ke > 0 ? ke : 0) * 4);
    // H pieces as in GEMM1: row 8 p + lane / 8, chunk c at position c ^ (row % 8)
    const int hc = (lane & 7) ^ (lane >> 3);
    // (a token past the batch has an offset past the buffer: reads as zeros)
    const int hoff = (int)(((m0 + 8 * w + (lane >> 3)) * Up + kb) * 2) + hc * 16;
    const int hstep = (int)(8 * NW * Up * 2);  // from a wave's piece to its next
    // Down pieces: kRpp rows of BN columns. The 32-byte unit u (16 columns) of row r is kept at
    // unit u ^ f(r), f(r) = r % 4 + 4 (r / 8) mod the units of a row: the 8 (16) rows that a
    // transposing read takes at once then lie in different banks.
    constexpr int kF = kRow / 32 - 1;  // 7 or 15
    // From a wave's piece to its next the row grows by kDR, which flips at most the top bit of
    // f (256 columns: kX in the byte offset).
    constexpr int kDR = NW * kRpp, kX = BN == 256 && kDR == 16 ? 256 : 0;
    static_assert(BN == 256 ? kDR == 16 : kDR % 16 == 0, "row swizzle");
    const int drow = w * kRpp + lane / (64 / kRpp);
    const int dc0 = (lane % (64 / kRpp)) ^ ((((drow & 3) | ((drow >> 3) << 2)) & kF) << 1);
    const int dcol = (int)(n0 * 2) + 16 * dc0;
    const bool dok0 = n0 + 8 * dc0 < d, dok1 = n0 + 8 * (dc0 ^ (kX / 16)) < d;  // d % 8 == 0
    // The slots of a step's down rows are read a step ahead of the rows' loads (a position past
    // the chunk is out of the descriptor's range: reads as 0, not used).
    auto load_ids = [&](int k, int32_t(&ids)[LD]) {
#pragma unroll
        for (int j = 0; j < LD; ++j)
            ids[j] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(
                ru, (kb + k * kBK + drow + j * kDR) * 4, 0, 0);
    };
    int32_t nid[LD];  // of the step whose rows are loaded next
    int doff[LD];
    auto row_offsets = [&](int k, const int32_t(&ids)[LD]) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            // (no short circuits: each would be a branch)
            const bool ok = (drow < ke - kb - k * kBK - j * kDR) & (j & 1 ? dok1 : dok0) &
                            ((unsigned)ids[j] < (unsigned)L);
            const int o = ids[j] * (int)(d * 2) + (j & 1 ? dcol ^ kX : dcol);
            doff[j] = ok ? o : kOOB;
        }
    };
    // loads of step k into stage s (H past the chunk reads as zeros, so that what its rows hold
    // there does not matter)
    auto load_h = [&](int k, char* s) {
        const bool ok = 8 * hc < ke - kb - k * kBK;
#pragma unroll
        for (int j = 0; j < LH; ++j)
            load_lds16(PL == 2 && j * NW >= BM / 8 ? rl : rh, s + (j * NW + w) * 1024,
                       ok ? hoff + j % (BM / 8 / NW) * hstep : kOOB, k * 128);
    };
    auto load_d = [&](char* s) {  // at row_offsets()
#pragma unroll
        for (int j = 0; j < LD; ++j) load_lds16(rd, s + (j * NW + w) * 1024, doff[j], 0);
    };

    f32x4_t acc[FW][FT];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < FT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    vec8 fh[2][PL][FT], fd[2][FW];
    const int to = (wt * 16 * FT + nn) * 128;
    const int c0 = (g ^ (nn & 7)) * 16, c1 = ((4 + g) ^ (nn & 7)) * 16;
    // Down fragments: lane (nn, g) needs union positions 8 g .. 8 g + 7 of column nn of a
    // 16-column unit; ds_read_b64_tr_b16 hands lane i of a 16-lane group element i % 4 of the
    // 8-byte pieces addressed by lanes i / 4 + 4 q, so lane nn addresses position 8 g + nn / 4
    // (and + 4), columns 4 (nn % 4) .. + 3 of the unit.
    const int df = ((nn >> 2) | (g << 2)) & kF;  // f of the lane's rows, in every half
    int dadr[FW];
#pragma unroll
    for (int i = 0; i < FW; ++i)
        dadr[i] = (8 * g + (nn >> 2)) * kRow + (((ww * FW + i) ^ df) * 32) + (nn & 3) * 8;
    auto tr = [&](const char* p) {
        const s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4_t*)const_cast<char*>(p));
        return __builtin_bit_cast(u32x2_t, v);
    };
    auto frags = [&](const char* sh, const char* sd, int h) {
#pragma unroll
        for (int i = 0; i < FW; ++i) {
            const u32x2_t lo = tr(sd + dadr[i] + h * 32 * kRow);
            const u32x2_t hi = tr(sd + dadr[i] + (h * 32 + 4) * kRow);
            fd[h][i] = Mfma<ET>::vec(V16{{lo[0], lo[1], hi[0], hi[1]}});
        }
        const int c = h ? c1 : c0;
#pragma unroll
        for (int q = 0; q < PL; ++q)
#pragma unroll
            for (int j = 0; j < FT; ++j)
                fh[h][q][j] = Mfma<ET>::vec(ld16(sh + q * BM * 128 + to + j * 2048 + c));
    };
    auto mults = [&](int h) {
#pragma unroll
        for (int q = 0; q < PL; ++q)
#pragma unroll
            for (int j = 0; j < FT; ++j)
#pragma unroll
                for (int i = 0; i < FW; ++i)
                    acc[i][j] = Mfma<ET>::mma(fd[h][i], fh[h][q][j], acc[i][j]);
    };
    char* const hs[4] = {h0, h1, h2, h3};
    char* const ds[4] = {d0, d1, d2, d3};
    // A K step, as in GEMM1. The offsets of the next down loads are formed from their slots just
    // before the barrier; the slots after those are then asked for, a step ahead of their use.
    constexpr int NM = PL * FT * FW, NR = PL * FT + 2 * FW;
    constexpr int LA = kSplit ? LD : 0, LB = LH + (kSplit ? 0 : LD);
    auto step = [&](int k, int q) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kSplit) load_d(ds[(q + ND - 1) % ND]);
        frags(hs[q % NH], ds[q % ND], 1);
        mults(0);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (i < LA) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NM / NR, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the next step's loads have landed: at least these many were issued after them
        wait_vm_lds<kSplit ? LD : (NH - 2) * (LH + LD)>();
        row_offsets(k + ND, nid);
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
        load_ids(k + ND + 1, nid);
        __builtin_amdgcn_sched_barrier(0);
        load_h(k + NH, hs[q % NH]);
        if constexpr (!kSplit) load_d(ds[q % ND]);
        frags(hs[(q + 1) % NH], ds[(q + 1) % ND], 0);
        mults(1);
#pragma unroll
        for (int i = 0; i < (NR > LB ? NR : LB); ++i) {
            if (i < LB) {
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
            if (i < NR) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        }
        asm volatile("" ::: "memory");
    };
    if (kb < ke) {
        const int nk = (ke - kb + kBK - 1) / kBK;
        int32_t pid[ND][LD];
#pragma unroll
        for (int q = 0; q < ND; ++q) load_ids(q, pid[q]);
        load_ids(ND, nid);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NH; ++q) {
            row_offsets(q, pid[q]);
            load_h(q, hs[q]);
            load_d(ds[q]);
            __builtin_amdgcn_sched_barrier(0);  // the counted waits rely on the stages' order
        }
        if constexpr (kSplit) row_offsets(ND - 1, pid[ND - 1]);  // step 0 loads these rows
        wait_vm_lds<(NH - 1) * (LH + LD)>();
        wg_barrier();
        frags(h0, d0, 0);
        int k = 0;
        for (; k + kPer <= nk; k += kPer) {
#pragma unroll
            for (int q = 0; q < kPer; ++q) step(k + q, q);
        }
#pragma unroll
        for (int q = 0; q < kPer - 1; ++q)
            if (k + q < nk) step(k + q, q);
        wait_vm_lds<0>();  // nothing may land in LDS once the work-group is gone
    }

    // element e of acc[i][j]: column n0 + 16 (ww FW + i) + 4 g + e of token
    // m0 + 16 (wt FT + j) + nn
    const int64_t nch = part_chunks(d);
#pragma unroll
    for (int j = 0; j < FT; ++j) {
        const int64_t tok = m0 + 16 * (wt * FT + j) + nn;
#pragma unroll
        for (int i = 0; i < FW; ++i) {
            const int64_t col = n0 + 16 * (ww * FW + i) + 4 * g;
            if (tok < B && col < d) {
                float* p = ks == 0 ? y + tok * d + col
                                   : part + part_off(tok, ks - 1, col, KS - 1, nch);
                *reinterpret_cast<f32x4_t*>(p) = acc[i][j];
            }
        }
    }
}

// y += the P partials of chunks 1 .. KS - 1 (P = KS - 1), in order: one float4 of y a thread
__global__ __launch_bounds__(256) void add_partials(const float* __restrict__ part, int P,
                                                    int64_t n4, int64_t d, float* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const int64_t e = 4 * i;
    const int64_t b = e / d, c = e - b * d;  // d % 8 == 0: the float4 is in one row
    const f32x4_t* p = reinterpret_cast<const f32x4_t*>(part + part_off(b, 0, c, P, part_chunks(d)));
    f32x4_t s = *reinterpret_cast<const f32x4_t*>(y + e);
    int q = 0;
    for (; q + 4 <= P; q += 4) {
        f32x4_t v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = p[(q + r) * (kChunk / 4)];
#pragma unroll
        for (int r = 0; r < 4; ++r) s += v[r];
    }
    for (; q < P; ++q) s += p[q * (kChunk / 4)];
    *reinterpret_cast<f32x4_t*>(y + e) = s;
}

// ---- tile choice ---------------------------------------------------------------------------
// Time of one K step (64) of a work-group that has a CU to itself, in units of 10 ns, measured
// over whole GEMMs (kernel time / rounds of work-groups / steps): the larger tile does more per
// byte it takes in and per barrier, the smaller one fills the CUs where the product is small.
struct G1Tile {
    int bm, bn, cost;
};
constexpr G1Tile kG1Tiles[] = {{256, 256, 143}, {256, 160, 103}, {128, 160, 56}};
constexpr int kG1Count = 3;
struct G2Tile {
    int bm, bn, cost;
};
constexpr G2Tile kG2Tiles[] = {{256, 256, 143}, {256, 128, 95}, {128, 128, 55}};  // one 16-bit h
constexpr int kG2Count = 3;
constexpr G2Tile kG2Exact = {128, 128, 85};  // hi + lo pair

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

// exact: H as a hi + lo pair (SI_FLAG_EXACT_H), else one 16-bit value (no lo plane)
TPlan make_tplan(int64_t B, int64_t L, int64_t d, int num_cu, bool exact) {
    TPlan p;
    p.W = (L + 31) / 32;
    p.Lp = p.W * 32;
    p.Up = (L + kBK - 1) / kBK * kBK;
    p.g1 = gemm1_pick(B, L, num_cu);
    p.ntm1 = (int)cdiv(B, kG1Tiles[p.g1].bm);
    p.nst = (int)cdiv(L, kG1Tiles[p.g1].bn / 2);
    // GEMM2: tile and K chunks of least time, where every chunk past the first writes and the
    // reducer reads one float32 partial of Y (about 4 TB/s both ways: 2 B d / 10^7 units of
    // 10 ns a chunk)
    const int64_t rows = partial_rows(B, L, d, num_cu);
    const int64_t steps = cdiv(L, kBK);
    double bc = 1e300;
    for (int c = 0; c < (exact ? 1 : kG2Count); ++c) {
        const G2Tile& tl = exact ? kG2Exact : kG2Tiles[c];
        const int64_t tiles = cdiv(B, tl.bm) * cdiv(d, tl.bn);
        for (int64_t ks = 1; ks <= rows + 1 && ks <= steps; ++ks) {
            const double cost = (double)(cdiv(tiles * ks, num_cu) * cdiv(steps, ks) * tl.cost) +
                                2e-4 * (double)(B * d) * (double)(ks - 1) + (ks > 1 ? 300. : 0.);
            if (cost < bc) bc = cost, p.g2 = c, p.KS = (int)ks;
        }
    }
    const G2Tile& t2 = exact ? kG2Exact : kG2Tiles[p.g2];
    p.ntm2 = (int)cdiv(B, t2.bm);
    p.ntn2 = (int)cdiv(d, t2.bn);
    size_t o = 0;
    p.off_bits = o;
    o = align256(o + (size_t)B * p.W * 4);
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

template <typename ET>
hipError_t launch_union_tiled_t(const void* x, int64_t B, int64_t d, const int32_t* offsets,
                                const int32_t* idx, int64_t nnz, const void* gate_up_c,
                                const void* down_c, int64_t L, float* y, void* ws, int flags,
                                int num_cu, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const bool fast = !tiled_exact_h(flags);
    const TPlan p = make_tplan(B, L, d, num_cu, !fast);
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
    hipLaunchKernelGGL(union_scan, dim3(1), dim3(1024), (unsigned)(p.W * 4), s, words, p.nb, p.W,
                       ulist, ucount);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 g1((unsigned)((int64_t)p.nst * p.ntm1 + 7) / 8 * 8);
#define SI_G1(BM, BN, WT, WW, NX, NWT)                                                                \
    hipExtLaunchKernelGGL((gemm1_pipe<ET, kUnion, BM, BN, WT, WW, NX, NWT>), g1, dim3(64 * WT * WW),  \
                          0, s, ev0, nullptr, 0, xx, B, d, gu, L, ulist, ucount, bits, p.W, hhi, \
                          hlo, p.Up, p.ntm1, nullptr)
    switch (p.g1) {
        case 0: SI_G1(256, 256, 2, 4, 2, 3); break;
        case 1: SI_G1(256, 160, 4, 2, 3, 3); break;
        default: SI_G1(128, 160, 2, 2, 4, 4); break;
    }
#undef SI_G1
    const dim3 g2((unsigned)((int64_t)p.ntm2 * p.ntn2 * p.KS + 7) / 8 * 8);
#define SI_G2(PL, BM, BN, WT, WW, NH, ND)                                                            \
    hipExtLaunchKernelGGL((gemm2_pipe<ET, PL, BM, BN, WT, WW, NH, ND>), g2, dim3(64 * WT * WW), 0, s, \
                          nullptr, ev1, 0, hhi, hlo, p.Up, B, dc, d, L, ulist, ucount, y, part,   \
                          p.KS, p.ntm2, p.ntn2)
    if (!fast)
        SI_G2(2, 128, 128, 4, 2, 3, 3);
    else if (p.g2 == 0)
        SI_G2(1, 256, 256, 2, 4, 2, 3);
    else if (p.g2 == 1)
        SI_G2(1, 256, 128, 4, 2, 3, 3);
    else
        SI_G2(1, 128, 128, 2, 2, 4, 4);
#undef SI_G2
    if (p.KS > 1) {
        const int64_t n4 = B * d / 4;
        hipLaunchKernelGGL(add_partials, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, part,
                           p.KS - 1, n4, d, y);
    }
    return hipGetLastError();
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
                          ev1, 0, xx, T, d, gu, L, nullptr, nullptr, nullptr, (int64_t)0,        \
                          nullptr, nullptr, ldo, ntm, out)
#define SI_ACT_TILES(MODE)                                                \
    switch (c) {                                                          \
        case 0: SI_ACT_LAUNCH(MODE, 256, 256, 2, 4, 2, 3); break;            \
        case 1: SI_ACT_LAUNCH(MODE, 256, 160, 4, 2, 3, 3); break;            \
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
