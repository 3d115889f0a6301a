// The pipelined MFMA GEMMs of the union paths: GEMM1 (H, or the activations or scores of every
// slot) and GEMM2 (Y from H). k_tiled.hip and k_union.hip instantiate them with their tiles.
#pragma once

#include <type_traits>

#include "common.h"
#include "mfma.h"
#include "pipe.h"

namespace si {

namespace {

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;

constexpr int kBK = 64;  // K step (elements)

// Position of the r-th (0-based) set bit of u; requires r < popcount(u).
__device__ __forceinline__ int nth_set_bit(uint32_t u, int r) {
    int pos = 0;
#pragma unroll
    for (int half = 16; half >= 1; half >>= 1) {
        const uint32_t low = (1u << half) - 1u;
        const int c = __popc(u & low);
        if (r >= c) {
            r -= c;
            u >>= half;
            pos += half;
        } else {
            u &= low;
        }
    }
    return pos;
}

// Steps of a run, for sums of nk steps (2 MFMAs each) taken in runs whose results are then added
// up: runs of m of n MFMAs leave a squared rounding error of about n (m + n / m) / 2, least at
// m = sqrt(n). One run leaves n^2 / 2.
__device__ __forceinline__ int run_steps(int nk) {
    int r = 1;
    while (2 * (r + 1) * (r + 1) <= nk) ++r;
    return r;
}
// the end of a run: tot += acc, acc = 0
template <int M, int N>
__device__ __forceinline__ void flush_sums(f32x4_t (&tot)[M][N], f32x4_t (&acc)[M][N]) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
}

// ---- GEMM1 ---------------------------------------------------------------------------------
// MODE selects what the epilogue produces (the product itself is the same):
//   kUnion:  h masked by the token bitmaps, over the union list, as 16-bit hi (and lo) planes.
//            With nb = 0 the list is given. With nb > 0 it is formed here: part[0..nb) are
//            bitmaps whose OR is the union (W <= kScanWords words), every work-group finds its
//            own slots from them, and those of the first token tile write the list for GEMM2;
//   kAct:    the activation of every slot (the union list is the identity, no mask), float32
//            out[tok * Up + slot];
//   kScore:  Eq. 1 for this work-group's tokens: sum over its BM tokens of |a| per slot, added
//            in a fixed order, float32 out[tm * Up + slot] (one partial row per token tile; the
//            host-side reducer adds the rows in order);
//   kWord:   as kUnion, but without a union list: a slot tile is BN / 2 consecutive slots, H is
//            indexed by slot, and rows that no token of the tile has are not loaded. The tile's
//            union words go to words[tm * W ..] for GEMM2.
enum { kUnion = 0, kAct = 1, kScore = 2, kWord = 3 };

// Token bitmap words a work-group keeps in LDS for the mask (per token; pitch odd so that 16
// tokens' words lie in different banks)
constexpr int kWin = 16, kWinP = kWin + 1;

// Union words a GEMM1 work-group scans by itself (L <= 32768)
constexpr int kScanWords = 1024;

// BM tokens x BN weight rows (BN / 2 union slots); WT x WW waves of FT x FW 16x16 MFMA tiles,
// the weight rows as the M operand, so a lane ends up with 4 consecutive weight rows of one
// token. Those are 2 gate and 2 up rows of the same two slots, so SiLU * up needs no data
// exchange. NX LDS stages of x and NWT of the weight rows, which come from HBM and are given
// the longer flight where the LDS cannot hold a third stage of both (256 x 256).
// ONCE: each weight row is read by one work-group.
template <typename ET, int MODE, int BM, int BN, int WT, int WW, int NX, int NWT, bool ONCE = false>
__global__ __launch_bounds__(64 * WT * WW) void gemm1_pipe(
    const uint16_t* __restrict__ x, int64_t B, int64_t d, const uint16_t* __restrict__ gu, int64_t L,
    int32_t* __restrict__ ulist, int* __restrict__ ucount, const uint32_t* __restrict__ part,
    int nb, const uint32_t* __restrict__ bits, int64_t W, uint16_t* __restrict__ Hhi,
    uint16_t* __restrict__ Hlo, int64_t Up, int ntm, float* __restrict__ out,
    uint32_t* __restrict__ words) {
    constexpr int NW = WT * WW, kThr = 64 * NW;
    constexpr int FT = BM / (16 * WT), FW = BN / (16 * WW);
    constexpr int kS = BN / 2;
    // 1 KB pieces (8 rows) of a stage, and how many of them a wave loads (the last of a
    // wave's weight pieces may be left to the lower waves: kPart of them)
    constexpr int RX = BM / 8, RW = BN / 8, LX = RX / NW, LW = RW / NW, kPart = RW % NW;
    constexpr bool kSplit = NWT > NX;
    constexpr int kPer = kSplit ? NX * NWT : NX;  // steps after which the stages come round
    static_assert(RX % NW == 0 && NX >= 2 && NX <= 8 && (MODE != kWord || BN <= 128), "tile");
    static_assert(NX * (LX + LW + (kPart ? 1 : 0)) <= 63, "the load counter has 6 bits");
    static_assert(NWT == NX || (NX == 2 && NWT == 3 && kPart == 0), "stages");
    typedef typename Mfma<ET>::vec8 vec8;
    constexpr int kWPol = ONCE ? kNonTemporal : 0;
    // one array per stage: the compiler then sees that a stage's reads do not touch the stages
    // being loaded, and waits for nothing between them
    __shared__ __align__(1024) char x0[RX * 1024];
    __shared__ __align__(1024) char x1[RX * 1024];
    __shared__ __align__(1024) char x2[NX > 2 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x3[NX > 3 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x4[NX > 4 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x5[NX > 5 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x6[NX > 6 ? RX * 1024 : 16];
    __shared__ __align__(1024) char x7[NX > 7 ? RX * 1024 : 16];
    __shared__ __align__(1024) char w0[RW * 1024];
    __shared__ __align__(1024) char w1[RW * 1024];
    __shared__ __align__(1024) char w2[NWT > 2 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w3[NWT > 3 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w4[NWT > 4 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w5[NWT > 5 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w6[NWT > 6 ? RW * 1024 : 16];
    __shared__ __align__(1024) char w7[NWT > 7 ? RW * 1024 : 16];

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nn = lane & 15;
    const int g = lane >> 4;
    const int wt = w % WT, ww = w / WT;

    // kUnion with nb > 0: the union words and the union position of each word's first slot.
    // (The tables lie in stages that are not loaded yet.)
    int nU = (int)L;
    int* const wpos = reinterpret_cast<int*>(x0);
    uint32_t* const wtab = reinterpret_cast<uint32_t*>(x0) + kScanWords;
    static_assert(MODE != kUnion || (kScanWords % kThr == 0 && 8 * kScanWords <= RX * 1024), "scan");
    if constexpr (MODE == kUnion) {
        if (nb > 0) {
            // thread t: words kRun t .., 8 bitmaps' loads in flight
            constexpr int kRun = kScanWords / kThr;
            const __amdgpu_buffer_rsrc_t rp = make_rsrc(part, (int64_t)nb * W * 4);
            uint32_t run_word[kRun];
#pragma unroll
            for (int i = 0; i < kRun; ++i) run_word[i] = 0u;
            for (int r0 = 0; r0 < nb; r0 += 8) {
                uint32_t v[kRun][8];
#pragma unroll
                for (int i = 0; i < kRun; ++i)
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        v[i][q] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                            rp,
                            (r0 + q < nb) & (kRun * t + i < (int)W)
                                ? ((r0 + q) * (int)W + kRun * t + i) * 4
                                : kOOB,
                            0, 0);
#pragma unroll
                for (int i = 0; i < kRun; ++i)
#pragma unroll
                    for (int q = 0; q < 8; ++q) run_word[i] |= v[i][q];
            }
            // positions: a wave's counts scanned, then the waves'
            int* const wtot = reinterpret_cast<int*>(x1);
            int c = 0;
#pragma unroll
            for (int i = 0; i < kRun; ++i) c += __popc(run_word[i]);
            const int incl = wave_incl_scan(c);
            if (lane == kWave - 1) wtot[w] = incl;
            __syncthreads();
            nU = 0;
            int pos = incl - c;
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                pos += q < w ? wtot[q] : 0;
                nU += wtot[q];
            }
#pragma unroll
            for (int i = 0; i < kRun; ++i) {
                wpos[kRun * t + i] = pos;
                wtab[kRun * t + i] = run_word[i];
                pos += __popc(run_word[i]);
            }
            nU = __builtin_amdgcn_readfirstlane(nU);
            if (blockIdx.x == 0 && t == 0) *ucount = nU;
        } else {
            nU = *ucount;
        }
    }
    // (kWord: the whole of the last word, so that GEMM2 finds H defined over every step)
    const int nst = ((MODE == kWord ? (int)W * 32 : nU) + kS - 1) / kS;
    int tm, st;
    if (!xcd_tile((int)blockIdx.x, ntm, nst, tm, st)) return;  // uniform
    const int64_t m0 = (int64_t)tm * BM, u0 = (int64_t)st * kS;

    const __amdgpu_buffer_rsrc_t rbm =
        make_rsrc(bits, MODE == kUnion || MODE == kWord ? B * W * 4 : 0);
    // kWord: the two bitmap words that hold the tile's slots (a multiple of 8, at most 64, from
    // bit wsh of word wd on), ORed over its tokens
    const int wd = (int)(u0 >> 5), wsh = (int)(u0 & 31);
    static_assert(MODE != kWord || (kS % 8 == 0 && (kS == 64 || kS <= 48)), "mask words");
    auto token_words = [&](int64_t tok, bool in) -> uint64_t {
        const int o = (int)((tok * W + wd) * 4);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rbm, in ? o : kOOB, 0, 0);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
            rbm, in && wd + 1 < W ? o + 4 : kOOB, 0, 0);
        return lo | ((uint64_t)hi << 32);
    };
    uint64_t uword = 0u;
    if constexpr (MODE == kWord) {
        uint64_t v[(BM + 63) / 64];
#pragma unroll
        for (int q = 0; q < (BM + 63) / 64; ++q) {
            const int64_t tok = m0 + 64 * q + lane;
            v[q] = token_words(tok, 64 * q + lane < BM && tok < B);
        }
#pragma unroll
        for (int q = 0; q < (BM + 63) / 64; ++q) uword |= v[q];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1)
            uword |= (uint64_t)__shfl_xor((unsigned long long)uword, m, kWave);
        // a word is written by the tile that has its first slot
        const int first = wsh == 0 ? 0 : 1;
        if (t >= first && t < 2 && wd + t < W && 32 * t < wsh + kS)
            words[(int64_t)tm * W + wd + t] = (uint32_t)(uword >> (32 * t));
    }
    // no token has a slot of the tile: h = 0, and nothing else is read (5 tokens with 10 slots
    // each of 100000, d = 1024: GEMM1 43 us without this)
    if constexpr (MODE == kWord) {
        const uint64_t mine = kS == 64 ? uword : (uword >> wsh) & ((1ull << kS) - 1ull);
        if (mine == 0u) {  // uniform: every wave has the OR over all the tile's tokens
            const V16 zero = {{0u, 0u, 0u, 0u}};
            for (int e = t; e < BM * (kS / 8); e += kThr) {
                const int64_t tok = m0 + e / (kS / 8), u = u0 + 8 * (e % (kS / 8));
                if (tok < B && u < Up) {
                    st16(Hhi + tok * Up + u, zero);
                    if (Hlo) st16(Hlo + tok * Up + u, zero);
                }
            }
            return;
        }
    }
    // kUnion: the tile's slots, -1 past the union, in a table for the row offsets; thread t
    // keeps slot t for the epilogue
    int32_t* const stab = reinterpret_cast<int32_t*>(w1);
    int32_t my_slot = -1;
    if constexpr (MODE == kUnion) {
        static_assert(kS <= kThr, "slots");
        if (nb > 0) {
            // thread t finds union position u0 + t: the last word that starts at or before it,
            // then the set bit of that rank
            __syncthreads();
            if (t < kS) {
                const int u = (int)u0 + t;
                int wd = 0;
#pragma unroll
                for (int s = kScanWords / 2; s >= 1; s >>= 1)
                    if (wpos[wd + s] <= u) wd += s;
                if (u < nU) my_slot = wd * 32 + nth_set_bit(wtab[wd], u - wpos[wd]);
            }
        } else if (t < kS && u0 + t < nU) {
            const int32_t sl = ulist[u0 + t];
            if ((unsigned)sl < (unsigned)L) my_slot = sl;
        }
        if (t < kS) stab[t] = my_slot;
        __syncthreads();
        if (nb > 0 && tm == 0 && t < kS && u0 + t < nU) ulist[u0 + t] = my_slot;
    }
    // slot of row pair p of the tile, -1: none
    auto tile_slot = [&](int p) -> int32_t {
        const int u = (int)u0 + p;
        if constexpr (MODE == kUnion) return p < kS ? stab[p] : -1;
        if constexpr (MODE == kWord) return ((uword >> (wsh + p)) & 1u) && u < nU ? u : -1;
        return u < nU ? u : -1;
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
        const int32_t sl = tile_slot(slot_of(r / 16, (r % 16) / 4, r & 1));
        woff[j] = sl >= 0 ? (int)(((int64_t)sl * 2 + ((r >> 1) & 1)) * d * 2) + cb : kOOB;
    }
    // the mask's window: kWin bitmap words from the first slot's on, unless the tile's slots
    // span more
    int win0 = 0;
    bool in_win = false;
    if constexpr (MODE == kUnion) {
        const int last = (int)(nU - u0 < kS ? nU - u0 : kS) - 1;
        win0 = __builtin_amdgcn_readfirstlane(stab[0] >> 5);
        in_win = __builtin_amdgcn_readfirstlane(stab[last] >> 5) - win0 < kWin;
        __syncthreads();  // the tables are done with: their stages may be loaded
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
            load_lds16<kWPol>(rg, s + (j * NW + w) * 1024, ok ? woff[j] : kOOB, k * 128);
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
    // kWord is bound by HBM and h keeps 16 bits and more: K is summed in runs (45 half-precision
    // tokens, d = 5120: 7.4e-7 from the 64-bit result in one run, 2.8e-7 in runs)
    const int run = MODE == kWord ? run_steps(nk) : 0;
    int left = run;
    f32x4_t tot[FW][FT];
    if constexpr (MODE == kWord) {
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int j = 0; j < FT; ++j) tot[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
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
    char* const xs[8] = {x0, x1, x2, x3, x4, x5, x6, x7};
    char* const ws[8] = {w0, w1, w2, w3, w4, w5, w6, w7};
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
            __builtin_amdgcn_sched_group_barrier(0x008, NM < NR ? 1 : NM / NR, 0);
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
        if constexpr (MODE == kWord) {
            if (--left == 0) {
                flush_sums(tot, acc);
                left = run;
            }
        }
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
    if constexpr (MODE == kWord) {
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int j = 0; j < FT; ++j) acc[i][j] += tot[i][j];
    }

    // The stages are done with (nothing is in flight to them either): their memory takes the
    // epilogue's tables.
    wait_vm_lds<0>();
    wg_barrier();
    uint64_t tword[FT];  // kWord: the tokens' words
    if constexpr (MODE == kWord) {
#pragma unroll
        for (int j = 0; j < FT; ++j) {
            const int64_t tok = m0 + 16 * (wt * FT + j) + nn;
            tword[j] = token_words(tok, tok < B);
        }
    }
    int32_t* const sslot = reinterpret_cast<int32_t*>(w0);       // the tile's slots
    uint32_t* const swin = reinterpret_cast<uint32_t*>(x0);      // the mask's window
    double* const ssum = reinterpret_cast<double*>(x0);          // kScore: sums per wave row
    static_assert(MODE != kUnion || BM * kWinP * 4 <= RX * 1024, "mask window");
    static_assert(MODE != kScore || WT * kS * 8 <= RX * 1024, "sums");
    if (MODE == kUnion && t < kS) sslot[t] = my_slot;
    if ((MODE == kAct || MODE == kScore) && t < kS) sslot[t] = tile_slot(t);
    if constexpr (MODE == kUnion) {
        if (in_win) {
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
    if constexpr (MODE != kWord) __syncthreads();

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
    auto finish = [&](auto win) {
        constexpr int kLast = FW & 1 ? FW - 1 : FW;
#pragma unroll
        for (int i = 0; i < FW; i += 2) {
            const int np = i == kLast ? 1 : 2;  // tiles of this pair: 2 np consecutive slots
            const int64_t u = u0 + slot_of(ww * FW + i, g, 0);
            const int p0 = slot_of(ww * FW + i, g, 0);
            int32_t sl[4];
#pragma unroll
            for (int e = 0; e < 2 * np; ++e) {
                const int p = slot_of(ww * FW + i, g, 0) + e;
                sl[e] = MODE == kWord ? p : sslot[p];
            }
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
                        if constexpr (MODE == kWord)
                            word = (uint32_t)(tword[j] >> wsh >> (p0 + e)) << (sl[e] & 31);
                        else if constexpr (decltype(win)::value)
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
                        if (Hlo) {  // with the hi + lo pair only
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
// LIST: the union list and its length; otherwise K = slot over W bitmap words, with the token
// tile's union words (words[tm * W]): a row that no token of the tile has is not loaded.
// ONCE: each down row is read by one token tile.
template <typename ET, bool LIST, int PL, int BM, int BN, int WT, int WW, int NH, int ND,
          bool ONCE = false>
__global__ __launch_bounds__(64 * WT * WW) void gemm2_pipe(
    const uint16_t* __restrict__ Hhi, const uint16_t* __restrict__ Hlo, int64_t Up, int64_t B,
    const uint16_t* __restrict__ dc, int64_t d, int64_t L, const int32_t* __restrict__ ulist,
    const int* __restrict__ ucount, const uint32_t* __restrict__ words, int64_t W,
    float* __restrict__ y, float* __restrict__ part, int KS, int ntm, int ntn) {
    constexpr int NW = WT * WW;
    constexpr int FT = BM / (16 * WT), FW = BN / (16 * WW);
    // 1 KB pieces of a stage (of H one a wave at least; those past its rows stay zero) and how
    // many of them a wave loads
    constexpr int RHP = PL * BM / 8, RH = RHP < NW ? NW : RHP, RD = BN / 8;
    constexpr int LH = RH / NW, LD = RD / NW;
    constexpr bool kSplit = ND > NH;
    constexpr int kPer = kSplit ? NH * ND : NH;  // steps after which the stages come round
    constexpr int kRow = 2 * BN;                 // bytes of a down row segment
    constexpr int kRpp = 1024 / kRow;            // down rows per piece
    static_assert((BN == 128 || BN == 256) && RH % NW == 0 && RD % NW == 0, "tile");
    static_assert(NH >= 2 && NH <= 8 && (ND == NH || (NH == 2 && ND == 3)), "stages");
    typedef typename Mfma<ET>::vec8 vec8;
    __shared__ __align__(1024) char h0[RH * 1024];
    __shared__ __align__(1024) char h1[RH * 1024];
    __shared__ __align__(1024) char h2[NH > 2 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h3[NH > 3 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h4[NH > 4 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h5[NH > 5 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h6[NH > 6 ? RH * 1024 : 16];
    __shared__ __align__(1024) char h7[NH > 7 ? RH * 1024 : 16];
    __shared__ __align__(1024) char d0[RD * 1024];
    __shared__ __align__(1024) char d1[RD * 1024];
    __shared__ __align__(1024) char d2[ND > 2 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d3[ND > 3 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d4[ND > 4 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d5[ND > 5 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d6[ND > 6 ? RD * 1024 : 16];
    __shared__ __align__(1024) char d7[ND > 7 ? RD * 1024 : 16];

    int tm, sc;
    if (!xcd_tile((int)blockIdx.x, ntm, ntn * KS, tm, sc)) return;  // uniform
    const int ks = __builtin_amdgcn_readfirstlane((int)((unsigned)sc / (unsigned)ntn));
    const int ct = sc - ks * ntn;
    const int nU = LIST ? *ucount : (int)(W * 32);
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

    // the tile's rows of H
    const int64_t hbytes = (B - m0 < BM ? B - m0 : BM) * Up * 2;
    // (16-token tiles have fewer pieces a plane than there are waves: a wave keeps to one plane)
    constexpr int HP = BM / 8;
    static_assert(HP % NW == 0 || RH == NW, "H pieces");
    const int hw = HP < NW ? w % HP : w;
    const uint16_t* const hfirst = PL == 2 && HP < NW && w >= HP ? Hlo : Hhi;
    const __amdgpu_buffer_rsrc_t rh = make_rsrc(hfirst + m0 * Up, hbytes);
    const __amdgpu_buffer_rsrc_t rl = make_rsrc((PL == 2 ? Hlo : Hhi) + m0 * Up, hbytes);
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(dc, L * d * 2);
    const __amdgpu_buffer_rsrc_t ru = LIST ? make_rsrc(ulist, (int64_t)(ke > 0 ? ke : 0) * 4)
                                           : make_rsrc(words + tm * W, W * 4);
    // H pieces as in GEMM1: row 8 p + lane / 8, chunk c at position c ^ (row % 8)
    // (a token past the batch has an offset past the buffer: reads as zeros)
    const int hc = (lane & 7) ^ (lane >> 3);
    const int hoff = RHP < NW && w >= RHP
                         ? kOOB
                         : (int)(((8 * hw + (lane >> 3)) * Up + kb) * 2) + hc * 16;
    const int hstep = (int)(8 * NW * Up * 2);  // from a wave's piece to its next
    // Down pieces: kRpp rows of BN columns. The 32-byte unit u (16 columns) of row r is kept at
    // unit u ^ f(r), f(r) = r % 4 + 4 (r / 8) mod the units of a row: the 8 (16) rows that a
    // transposing read takes at once then lie in different banks.
    constexpr int kF = kRow / 32 - 1;  // 7 or 15
    // From a wave's piece to its next the row grows by kDR, which adds to the upper bits of f
    // only: swz(j) in the byte offset.
    constexpr int kDR = NW * kRpp;
    static_assert(kDR % 8 == 0, "row swizzle");
    auto swz = [](int j) { return (((j * kDR) >> 3) & (kF >> 2)) * 128; };
    const int drow = w * kRpp + lane / (64 / kRpp);
    const int dcol =
        16 * ((lane % (64 / kRpp)) ^ ((((drow & 3) | ((drow >> 3) << 2)) & kF) << 1));
    const int dlim = (int)((d - n0) * 2);  // bytes of a row from the tile's first column on
    // LIST: the slots of a step's down rows are read a step ahead of the rows' loads (a position
    // out of the descriptor's range reads as 0, not used).
    auto load_ids = [&](int k, int32_t(&ids)[LD]) {
#pragma unroll
        for (int j = 0; j < LD; ++j)
            ids[j] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(
                ru, (kb + k * kBK + drow + j * kDR) * 4, 0, 0);
    };
    int32_t nid[LD];  // of the step whose rows are loaded next
    int doff[LD];     // the rows' offsets, from dso on
    int dso = 0;
    auto row_offsets = [&](int k, const int32_t(&ids)[LD]) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int pos = kb + k * kBK + drow + j * kDR;
            const int col = dcol ^ swz(j);
            // (no short circuits: each would be a branch; d % 8 == 0)
            bool ok = (pos < ke) & (col < dlim);
            ok &= (unsigned)ids[j] < (unsigned)L;
            const int o = ids[j] * (int)(d * 2) + (int)(n0 * 2) + col;
            doff[j] = ok ? o : kOOB;
        }
    };
    // Otherwise: the union words of kSeg steps lie in registers, those of step seg + l in lane l,
    // and um has the non-empty ones among them. The pipeline runs over those only, and anew for
    // the next kSeg (chunks are seldom that long: 4096 slots).
    constexpr int kSeg = 64;
    uint32_t uw0 = 0u, uw1 = 0u;
    uint64_t um = 0u;
    int seg = 0;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(words + (LIST ? 0 : tm * W), LIST ? 0 : W * 4);
    auto load_words = [&](int nk) -> int {  // the number of non-empty steps
        const int o = seg + lane < nk ? ((kb >> 5) + 2 * (seg + lane)) * 4 : kOOB;
        uw0 = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rw, o, 0, 0);
        uw1 = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rw, o + 4, 0, 0);
        um = __ballot((uw0 | uw1) != 0u);
        return __popcll(um);
    };
    auto next_step = [&]() -> int {  // in the segment; -1: none is left
        const int p = um ? __builtin_ctzll(um) : -1;
        um &= um - 1u;
        return p;
    };
    int roff[LD];  // offsets of a step's rows from its first
    if constexpr (!LIST) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int col = dcol ^ swz(j);
            roff[j] = col < dlim ? (drow + j * kDR) * (int)(d * 2) + (int)(n0 * 2) + col : kOOB;
        }
    }
    auto word_offsets = [&](int p) {
        const uint32_t lo = p < 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)uw0, p & 63);
        const uint32_t hi = p < 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)uw1, p & 63);
        dso = p < 0 ? 0 : (kb + (seg + p) * kBK) * (int)(d * 2);
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const int row = drow + j * kDR;
            doff[j] = ((row & 32 ? hi : lo) >> (row & 31)) & 1u ? roff[j] : kOOB;
        }
    };
    // loads of step k into stage s (H past the chunk reads as zeros, so that what its rows hold
    // there does not matter)
    // (k < 0: no step)
    auto load_h = [&](int k, char* s) {
        const bool ok = LIST ? 8 * hc < ke - kb - k * kBK
                             : (k >= 0) & (8 * hc < ke - kb - (seg + k) * kBK);
        const int so = LIST ? k * 128 : k < 0 ? 0 : (seg + k) * 128;
#pragma unroll
        for (int j = 0; j < LH; ++j)
            load_lds16(HP >= NW && j * NW >= HP ? rl : rh, s + (j * NW + w) * 1024,
                       ok ? hoff + (HP >= NW ? j % (HP / (HP < NW ? HP : NW)) : 0) * hstep : kOOB,
                       so);
    };
    auto load_d = [&](char* s) {  // at row_offsets() or word_offsets()
#pragma unroll
        for (int j = 0; j < LD; ++j)
            load_lds16<ONCE ? kNonTemporal : 0>(rd, s + (j * NW + w) * 1024, doff[j],
                                               LIST ? 0 : dso);
    };

    f32x4_t acc[FW][FT];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < FT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // hi + lo: K in runs, as in GEMM1's kWord (the 128 x 256 tile has no registers for it and sums
    // its chunk, the shortest that the workspace allows, in one)
    constexpr bool kRuns = PL == 2 && FT * FW < 16;
    const int run = kRuns ? run_steps(2 * ((ke - kb + kBK - 1) / kBK)) / 2 + 1 : 0;
    int left = run;
    f32x4_t tot[FW][FT];
    if constexpr (kRuns) {
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int j = 0; j < FT; ++j) tot[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
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
                // (one sum of offsets: the compiler follows few pointer steps from a stage's
                // array to its reads, and has a read that it loses wait for every load)
                fh[h][q][j] = Mfma<ET>::vec(ld16(sh + (q * BM * 128 + to + j * 2048 + c)));
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
    char* const hs[8] = {h0, h1, h2, h3, h4, h5, h6, h7};
    char* const ds[8] = {d0, d1, d2, d3, d4, d5, d6, d7};
    // A K step, as in GEMM1. The offsets of the next down loads are formed from their slots just
    // before the barrier; the slots after those are then asked for, a step ahead of their use.
    int hnext = -1;  // with kSplit: the step whose H loads follow (its down loads go first)
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
            __builtin_amdgcn_sched_group_barrier(0x008, NM < NR ? 1 : NM / NR, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the next step's loads have landed: at least these many were issued after them
        wait_vm_lds<kSplit ? LD : (NH - 2) * (LH + LD)>();
        int pn = -1;
        if constexpr (LIST) {
            row_offsets(k + ND, nid);
        } else {
            pn = next_step();
            word_offsets(pn);
        }
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LIST) {
            load_ids(k + ND + 1, nid);
            __builtin_amdgcn_sched_barrier(0);
            load_h(k + NH, hs[q % NH]);
        } else {
            load_h(kSplit ? hnext : pn, hs[q % NH]);
            hnext = pn;
        }
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
        if constexpr (kRuns) {
            if (--left == 0) {
                flush_sums(tot, acc);
                left = run;
            }
        }
    };
    if (kb < ke) {
        const int nk = (ke - kb + kBK - 1) / kBK;
        int n = nk;  // steps to run
        do {
            if constexpr (LIST) {
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
                    __builtin_amdgcn_sched_barrier(0);  // the counted waits rely on this order
                }
                if constexpr (kSplit) row_offsets(ND - 1, pid[ND - 1]);  // for step 0
            } else {
                n = load_words(nk);
                if (n == 0) continue;  // uniform: every wave reads the same words
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < NH; ++q) {
                    const int p = next_step();
                    word_offsets(p);
                    load_h(p, hs[q]);
                    load_d(ds[q]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (kSplit) {
                    hnext = next_step();
                    word_offsets(hnext);
                }
            }
            wait_vm_lds<(NH - 1) * (LH + LD)>();
            wg_barrier();
            frags(h0, d0, 0);
            int k = 0;
            for (; k + kPer <= n; k += kPer) {
#pragma unroll
                for (int q = 0; q < kPer; ++q) step(k + q, q);
            }
#pragma unroll
            for (int q = 0; q < kPer - 1; ++q)
                if (k + q < n) step(k + q, q);
            wait_vm_lds<0>();  // nothing may land in LDS once the work-group is gone
            if constexpr (!LIST) wg_barrier();  // every wave has read the segment's last stages
        } while (!LIST && (seg += kSeg) < nk);
        if constexpr (kRuns) flush_sums(tot, acc);
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
                *reinterpret_cast<f32x4_t*>(p) = kRuns ? tot[i][j] : acc[i][j];
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
    // eight sums side by side, then added up: the rounding errors of an eighth of the chain
    f32x4_t s[8];
    s[0] = *reinterpret_cast<const f32x4_t*>(y + e);
#pragma unroll
    for (int r = 1; r < 8; ++r) s[r] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    int q = 0;
    for (; q + 8 <= P; q += 8) {
        f32x4_t v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = p[(q + r) * (kChunk / 4)];
#pragma unroll
        for (int r = 0; r < 8; ++r) s[r] += v[r];
    }
#pragma unroll
    for (int r = 0; r < 7; ++r)
        if (q + r < P) s[r + 1] += p[(q + r) * (kChunk / 4)];
    *reinterpret_cast<f32x4_t*>(y + e) =
        ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// The same with a wave per (token, 16 columns): lane l adds float4 l % 4 of partials l / 4,
// l / 4 + 16, ..., the lanes meet in a fixed order.
__global__ __launch_bounds__(256) void add_many_partials(const float* __restrict__ part, int P,
                                                         int64_t pairs, int64_t nch, int64_t d,
                                                         float* __restrict__ y) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t pair = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (pair >= pairs) return;
    const int64_t b = pair / nch;
    const int64_t c = (pair - b * nch) * kChunk + 4 * lane;
    const bool mine = lane < kChunk / 4 && c < d;  // d % 8 == 0: the float4 is all in range
    float* const py = y + b * d + c;
    const f32x4_t* p = reinterpret_cast<const f32x4_t*>(part + pair * P * kChunk);
    const int n4 = P * (kChunk / 4);
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
    if (mine) s = *reinterpret_cast<const f32x4_t*>(py);
    for (int i = lane; i < n4; i += 4 * kWave) {
        f32x4_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = i + q * kWave < n4 ? p[i + q * kWave] : f32x4_t{0.f, 0.f, 0.f, 0.f};
        s += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int m = kChunk / 4; m < kWave; m <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += __shfl_xor(s[e], m, kWave);
    if (mine) *reinterpret_cast<f32x4_t*>(py) = s;
}

// Up to this many (token, 16 columns) pairs, and from 4 partials, a wave a pair: with few sums a
// thread's chain of loads is the launch's time (whole call, 6000 slots, thread / wave a sum: 5
// tokens, d = 256, 63 partials 23.2 / 13.4 us, 16 tokens, d = 4096, 7 partials 31.6 / 30.5; 33
// tokens, d = 4096, 15 partials 45.0 / 43.3). With more, the waves' extra instructions are
// (100 tokens, d = 5120, 11 partials 72.7 / 75.3 us, 300 tokens, d = 1024 45.5 / 46.9).
constexpr int64_t kManyPairs = 10240;
constexpr int kManyPartials = 4;
// y += the P partials of B x d sums
inline hipError_t launch_add_partials(const float* part, int P, int64_t B, int64_t d, float* y,
                                      hipStream_t s) {
    const int64_t nch = part_chunks(d), pairs = B * nch;
    if (P >= kManyPartials && pairs <= kManyPairs) {
        hipLaunchKernelGGL(add_many_partials, dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, s,
                           part, P, pairs, nch, d, y);
    } else if (P > 0) {
        const int64_t n4 = B * d / 4;
        hipLaunchKernelGGL(add_partials, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, part,
                           P, n4, d, y);
    }
    return hipGetLastError();
}

}  // namespace

}  // namespace si
