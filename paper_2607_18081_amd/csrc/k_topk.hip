// Per-token top-k over the loaded neurons (dynamic-neuron selection, Selective Computation
// section): for each score row, the k slots with the largest key, returned in ascending order.
//
// Order: key = |s| (ABS) or s (RAW); larger key first; equal keys -> lower index first;
// -0 == +0; NaN after every number. Each float key is mapped to a uint32 whose unsigned order
// is that order (NaN -> 0); counts are taken as unsigned integers directly. One work-group per
// row:
//   1. radix select from the top: a histogram of the candidates by their next digit gives the
//      digit of the k-th largest key T and how many keys equal to T must still be taken;
//   2. selection in index order: an element is selected iff key > T, or key == T and fewer
//      than that many equal keys precede it; block-wide prefix counts give each selected element
//      its output position, so the output is ascending without a sort.
// Rows of up to 32768 keys (topk_rows_reg): thread t holds the C contiguous keys t*C .. in
// registers, read once. The digits cover the range between the least and the largest candidate,
// the search stops once the whole bin of T is taken (the lower bits cannot change the choice;
// the selection then needs no scan of equal keys), and a bin of at most 16 candidates is ranked
// by one wave. The choice can also be written as a bitmap per row, or joined with a given set.
// Longer rows (topk_rows) are read again in each of 4 passes of 8 bits.
#include "common.h"
#include "launch.h"

namespace si {

namespace {

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / kWave;

// Integer-only mapping, so no floating-point mode can change how -0 or NaN are treated.
// mode 0: |v|, 1: v, 2: the 32 bits as an unsigned integer (counts).
__device__ __forceinline__ uint32_t order_key(float v, int mode) {
    uint32_t u = __float_as_uint(v);
    if (mode == 2) return u;
    if (mode == 0) u &= 0x7fffffffu;                 // |v|
    const uint32_t mag = u & 0x7fffffffu;
    if (mag > 0x7f800000u) return 0u;                // NaN: below every number
    if (mag == 0u) u = 0u;                           // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Lane 63: the largest of the wave's values (DPP row shifts, then two row broadcasts).
__device__ __forceinline__ uint32_t wave_umax_last(uint32_t v) {
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));  // row_shr:4
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));  // row_shr:8
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // bcast:15
    step((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // bcast:31
    return v;
}

// Exclusive prefix count of `flag` over the block in thread order; returns the prefix and
// writes the block total to *total. Uses wave ballots and a scan of the 16 wave counts.
__device__ __forceinline__ int block_prefix(bool flag, int* wave_cnt, int* total) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const unsigned long long m = __ballot(flag);
    const unsigned long long below = lane == 0 ? 0ull : (m & ((~0ull) >> (64 - lane)));
    const int in_wave = __popcll(below);
    if (lane == 0) wave_cnt[w] = __popcll(m);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kTopkWaves; ++q) {
        const int c = wave_cnt[q];
        before += q < w ? c : 0;
        all += c;
    }
    __syncthreads();
    *total = all;
    return before + in_wave;
}

__global__ __launch_bounds__(kTopkThreads) void topk_rows(const float* __restrict__ scores,
                                                         int64_t L, int64_t ld, int64_t k,
                                                         int mode, int32_t* __restrict__ out) {
    const int64_t b = blockIdx.x;
    const float* row = scores + b * ld;
    int32_t* orow = out + b * k;
    __shared__ int hist[256];
    __shared__ int wave_cnt[kTopkWaves];
    __shared__ uint32_t s_prefix;
    __shared__ int64_t s_take;

    uint32_t prefix = 0u, pmask = 0u;
    int64_t take = k;  // how many still to take among candidates matching the prefix
#pragma unroll 1
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int i = threadIdx.x; i < 256; i += kTopkThreads) hist[i] = 0;
        __syncthreads();
        for (int64_t i = threadIdx.x; i < L; i += kTopkThreads) {
            const uint32_t key = order_key(row[i], mode);
            if ((key & pmask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t above = 0;
            int dsel = 0;
            for (int dg = 255; dg >= 0; --dg) {
                const int64_t c = hist[dg];
                if (above + c >= take) {
                    dsel = dg;
                    break;
                }
                above += c;
            }
            s_prefix = prefix | ((uint32_t)dsel << shift);
            s_take = take - above;
        }
        __syncthreads();
        prefix = s_prefix;
        take = s_take;
        pmask |= 255u << shift;
        __syncthreads();
    }
    const uint32_t T = prefix;

    int64_t run_eq = 0, run_sel = 0;
    for (int64_t base = 0; base < L; base += kTopkThreads) {
        const int64_t i = base + threadIdx.x;
        const uint32_t key = i < L ? order_key(row[i], mode) : 0u;
        const bool gt = i < L && key > T;
        const bool eq = i < L && key == T;
        int eq_total;
        const int eq_rank = block_prefix(eq, wave_cnt, &eq_total);
        const bool sel = gt || (eq && run_eq + eq_rank < take);
        int sel_total;
        const int pos = block_prefix(sel, wave_cnt, &sel_total);
        if (sel && run_sel + pos < k) orow[run_sel + pos] = (int32_t)i;
        run_eq += eq_total;
        run_sel += sel_total;
    }
}

// Exclusive prefix sum of v over the block (NW waves) in thread order; *total = block sum. Two
// barriers.
template <int NW>
__device__ __forceinline__ int block_excl_scan(int v, int* wave_tot, int* total) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int incl = wave_incl_scan(v);
    if (lane == kWave - 1) wave_tot[w] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        const int c = wave_tot[q];
        before += q < w ? c : 0;
        all += c;
    }
    __syncthreads();
    *total = all;
    return before + incl - v;
}

// What a register-resident launch writes (exactly one of idx, bmp, ulist is set):
struct TopkOut {
    int32_t* idx;  // [B][k] the chosen indices, ascending
    uint32_t* bmp;  // [B][bW] a bitmap per row: bit j of word w set iff slot 32 w + j is chosen
    int64_t bW;
    // one row: the set join_ids[0 .. n_join) (ids outside [0, L) ignored) joined with the k
    // chosen among the other keys, ascending, at most ucap of them -> ulist, their number ->
    // *ucount
    const int32_t* join_ids;
    int64_t n_join;
    int32_t* ulist;
    int64_t ucap;
    int* ucount;
};

constexpr int kMaxRegKeys = 32 * kTopkThreads;  // the register-resident kernel's longest row

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// NT threads a row, at least WPS waves a SIMD: two 1024-thread work-groups share a CU with 8
// only, and the compiler must be told (left alone it takes 106 scalar registers for C = 8: 7
// waves).
constexpr int kDigit = 11, kBins = 1 << kDigit;  // bits and bins of a pass
// Candidates that one wave ranks, a lane each: its loop over them is a chain that another pass
// beats from about 20 on (128 rows of 2048 keys by value 7.3 / 6.0 / 5.8 us with 64 / 32 / 16)
constexpr int kFew = 16;
template <int C, int NT, int WPS>
__global__ __launch_bounds__(NT, WPS) void topk_rows_reg(const float* __restrict__ scores,
                                                         int64_t L, int64_t ld, int64_t k,
                                                         int mode, TopkOut o) {
    static_assert(32 % C == 0, "a thread's keys lie in one bitmap word");
    constexpr int NW = NT / kWave;
    constexpr int kOwn = kBins / NT;  // bins a thread reads
    const int64_t b = blockIdx.x;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = t >> 6;
    __shared__ int hist[kBins];
    __shared__ int wave_tot[NW];
    __shared__ uint32_t s_min[NW], s_max[NW];
    __shared__ int s_digit, s_take, s_n;
    __shared__ uint32_t s_key;
    __shared__ uint32_t few[kFew];
    __shared__ int n_few;
    __shared__ uint32_t jbits[kMaxRegKeys / 32];
    if (o.ulist) {  // the joined set as a bitmap
        for (int q = t; q < kMaxRegKeys / 32; q += NT) jbits[q] = 0u;
        __syncthreads();
        for (int64_t i = t; i < o.n_join; i += NT) {
            const int32_t v = o.join_ids[i];
            if (v >= 0 && v < L) atomicOr(&jbits[v >> 5], 1u << (v & 31));
        }
        __syncthreads();
    }
    const float* row = scores + b * ld;
    // keys t*C .. t*C + C - 1 (the first nvalid of them lie in the row)
    uint32_t key[C];
    const int64_t rest = L - (int64_t)t * C;
    const int nvalid = rest <= 0 ? 0 : (rest < C ? (int)rest : C);
    if (C % 4 == 0 && nvalid == C) {
        // rows may begin at any float: 16-byte loads of 4-byte alignment (scalar loads of the
        // lanes' runs of C keys took 3.4 us of a 7706-key row, these 1.2)
        const f32x4_a4* r4 = reinterpret_cast<const f32x4_a4*>(row + (int64_t)t * C);
#pragma unroll
        for (int q = 0; q < C / 4; ++q) {
            const f32x4_a4 v = r4[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) key[4 * q + e] = order_key(v[e], mode);
        }
    } else {
#pragma unroll
        for (int j = 0; j < C; ++j)
            key[j] = j < nvalid ? order_key(row[(int64_t)t * C + j], mode) : 0u;
    }
    // candidates: the keys in the row, less (join mode) the slots of the joined set
    const uint32_t vmask = nvalid >= 32 ? ~0u : (1u << nvalid) - 1u;  // keys in the row
    uint32_t cand = k > 0 ? vmask : 0u;
    const uint32_t jw = (o.ulist && nvalid > 0) ? jbits[(t * C) / 32] >> ((t * C) & 31) : 0u;
    cand &= ~jw;
    // least and largest candidate: the first digits cover just that range
    uint32_t kmin = ~0u, kmax = 0u;
#pragma unroll
    for (int j = 0; j < C; ++j)
        if ((cand >> j) & 1u) {
            kmin = key[j] < kmin ? key[j] : kmin;
            kmax = key[j] > kmax ? key[j] : kmax;
        }
    // (largest of ~kmin and of kmax over the wave: in lane 63)
    const uint32_t wmin = ~wave_umax_last(~kmin), wmax = wave_umax_last(kmax);
    if (lane == kWave - 1) {
        s_min[w] = wmin;
        s_max[w] = wmax;
    }
    for (int q = t; q < kBins; q += NT) hist[q] = 0;
    if (t == 0) n_few = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        kmin = s_min[q] < kmin ? s_min[q] : kmin;
        kmax = s_max[q] > kmax ? s_max[q] : kmax;
    }
    // The k-th largest key T lies in [base, base + span]; a pass splits that into 2^11
    // bins of 2^shift keys. (No candidates at all: nothing is counted, and the first pass ends it.)
    const uint32_t range = kmax - kmin;
    const int width = range ? 32 - __clz((int)range) : 0;
    int shift = width > kDigit ? width - kDigit : 0;
    uint32_t base = kmin, span = ~0u;
    int take = (int)k;   // how many still to take among the candidates in the range
    bool done = k == 0;  // all of them are taken
    while (!done) {
        // 1. count the candidates by bin; a run of equal digits in a thread's keys is added at
        //    once (few distinct digits would serialise the atomics on one bin)
        int cur = -1, cnt = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            if (((cand >> j) & 1u) && key[j] - base <= span) {
                const int dg = (int)((key[j] - base) >> shift);
                if (dg != cur) {
                    if (cnt) atomicAdd(&hist[cur], cnt);
                    cur = dg;
                    cnt = 0;
                }
                ++cnt;
            }
        }
        if (cnt) atomicAdd(&hist[cur], cnt);
        __syncthreads();
        // 2. the bins read (and cleared for the next pass): thread t owns kOwn bins, the largest
        //    digits in the lowest threads, and a block-wide scan counts the keys above
        int c[kOwn], sum = 0;
#pragma unroll
        for (int e = 0; e < kOwn; ++e) {
            const int bin = kBins - 1 - kOwn * t - e;
            c[e] = hist[bin];
            hist[bin] = 0;
            sum += c[e];
        }
        int all;
        int above = block_excl_scan<NW>(sum, wave_tot, &all);
        if (all < take) {  // k above the number of candidates: every candidate is taken
            base = 0u;
            done = true;
            break;
        }
        // 3. exactly one bin holds the key of the wanted rank
#pragma unroll
        for (int e = 0; e < kOwn; ++e) {
            if (above < take && above + c[e] >= take) {
                s_digit = kBins - 1 - kOwn * t - e;
                s_take = take - above;
                s_n = c[e];
            }
            above += c[e];
        }
        __syncthreads();
        base += (uint32_t)s_digit << shift;
        span = (1u << shift) - 1u;
        take = s_take;
        const int n = s_n;  // candidates in the bin
        done = take == n;
        if (done || shift == 0) break;
        shift = shift > kDigit ? shift - kDigit : 0;
        if (n > kFew) continue;
        // 4. few candidates: they are gathered, one a lane, and one wave ranks them by comparing
        //    each with all (all waves at it take 1 us longer)
#pragma unroll
        for (int j = 0; j < C; ++j)
            if (((cand >> j) & 1u) && key[j] - base <= span) few[atomicAdd(&n_few, 1)] = key[j];
        __syncthreads();
        if (w == 0) {
            const uint32_t mine = lane < n ? few[lane] : 0u;
            int gt = 0, ge = 0;
            for (int i = 0; i < n; ++i) {
                const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
                gt += other > mine ? 1 : 0;
                ge += other >= mine ? 1 : 0;
            }
            // a lane that holds the k-th key
            const unsigned long long hit = __ballot(lane < n && gt < take && take <= ge);
            if (lane == __ffsll((long long)hit) - 1) {
                s_key = mine;
                s_take = take - gt;
                s_n = ge - gt;
            }
        }
        __syncthreads();
        base = s_key;
        take = s_take;
        done = take == s_n;
        break;
    }
    const uint32_t T = base;
    uint32_t sel = 0u;  // bit j: key t*C + j is chosen
    if (done) {  // every candidate from T on is taken
#pragma unroll
        for (int j = 0; j < C; ++j) sel |= (((cand >> j) & 1u) && key[j] >= T) ? 1u << j : 0u;
    } else {  // those above T, and the first `take` candidates equal to T in index order
        int n_eq = 0;
#pragma unroll
        for (int j = 0; j < C; ++j) n_eq += (((cand >> j) & 1u) && key[j] == T) ? 1 : 0;
        int eq_all;
        int eq_before = block_excl_scan<NW>(n_eq, wave_tot, &eq_all);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const bool ok = (cand >> j) & 1u;
            const bool eq = ok && key[j] == T;
            sel |= (ok && (key[j] > T || (eq && eq_before < take))) ? 1u << j : 0u;
            eq_before += eq ? 1 : 0;
        }
    }
    if (o.bmp) {
        // the 32 / C threads of one word (consecutive lanes) OR their bits together
        uint32_t m = C == 32 ? sel : sel << ((t * C) & 31);
#pragma unroll
        for (int q = 1; q < 32 / C; q <<= 1) m |= (uint32_t)__shfl_xor((int)m, q, kWave);
        const int64_t wd = ((int64_t)t * C) / 32;
        if (((t * C) & 31) == 0 && wd < o.bW) o.bmp[b * o.bW + wd] = m;
        return;
    }
    int64_t cap = k;
    int32_t* orow = o.ulist;
    if (!o.ulist) {
        orow = o.idx + b * k;
    } else {
        sel |= jw & vmask;  // join the bits of o.join (none of them a candidate)
        cap = o.ucap;
    }
    int sel_all;
    int pos = block_excl_scan<NW>(__popc(sel), wave_tot, &sel_all);
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const bool on = (sel >> j) & 1u;
        if (on && pos < cap) orow[pos] = (int32_t)((int64_t)t * C + j);
        pos += on ? 1 : 0;
    }
    if (o.ulist && t == 0) *o.ucount = sel_all < cap ? sel_all : (int)cap;
}

}  // namespace

namespace {

// One register-resident launch, one work-group per row; false when a row has more than 32768
// keys. What a row costs beside its keys goes by the work-group's threads (scans over the waves,
// barriers, bins), so rows of few keys take 512 of them, and so do rows of up to 4096 keys where a
// CU has more than one; with fewer rows than CUs a row of more than 2048 is quicker with 1024 (256
// rows of 3000 keys by |value| 6.9 / 6.3 us with 512 / 1024 threads, of 2047 5.6 / 5.7; 300 rows
// of 3000 7.8 / 10.5, of 64 4.0 / 5.3). Rows of 4097 to 8192 keys on shared CUs need 8 waves a
// SIMD (300 rows of 4500 keys 14.8 / 12.6 us, of 7706 17.0 / 14.8), which costs 0.7 us where a CU
// has one.
bool launch_reg(const float* scores, int64_t B, int64_t L, int64_t ld, int64_t k, int mode,
                const TopkOut& o, hipStream_t s) {
    const bool shared_cu = B > current_cu_count();
#define SI_TOPK(C, NT, WPS)                                                                      \
    hipLaunchKernelGGL((topk_rows_reg<C, NT, WPS>), dim3((unsigned)B), dim3(NT), 0, s, scores, L, \
                       ld, k, mode, o)
    if (L <= 512)
        SI_TOPK(1, 512, 1);
    else if (L <= 1024)
        SI_TOPK(2, 512, 1);
    else if (L <= 2048)
        SI_TOPK(4, 512, 1);
    else if (L <= 4096 && shared_cu)
        SI_TOPK(8, 512, 1);
    else if (L <= 4096)
        SI_TOPK(4, 1024, 1);
    else if (L <= 8192 && shared_cu)
        SI_TOPK(8, 1024, 8);
    else if (L <= 8192)
        SI_TOPK(8, 1024, 1);
    else if (L <= 16384)
        SI_TOPK(16, 1024, 1);
    else if (L <= kMaxRegKeys)
        SI_TOPK(32, 1024, 1);
    else
        return false;
#undef SI_TOPK
    return true;
}

}  // namespace

hipError_t launch_topk_strided(const float* scores, int64_t B, int64_t L, int64_t ld, int64_t k,
                               int mode, int32_t* out, hipStream_t s) {
    if (B == 0 || k == 0) return hipSuccess;
    TopkOut o{};
    o.idx = out;
    if (!launch_reg(scores, B, L, ld, k, mode, o, s))
        hipLaunchKernelGGL(topk_rows, dim3((unsigned)B), dim3(kTopkThreads), 0, s, scores, L, ld,
                           k, mode, out);
    return hipGetLastError();
}

hipError_t launch_topk_bitmap(const float* scores, int64_t B, int64_t L, int64_t ld, int64_t k,
                              int mode, uint32_t* bits, int64_t W, hipStream_t s) {
    if (B == 0) return hipSuccess;
    TopkOut o{};
    o.bmp = bits;
    o.bW = W;
    // every word of a row is written by the kernel: W must be exactly the row's word count
    if (W != (L + 31) / 32 || !launch_reg(scores, B, L, ld, k, mode, o, s))
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_topk_join(const float* scores, int64_t L, int64_t k, int mode,
                            const int32_t* join_ids, int64_t n_join, int32_t* list, int64_t cap,
                            int* count, hipStream_t s) {
    TopkOut o{};
    o.join_ids = join_ids;
    o.n_join = n_join;
    o.ulist = list;
    o.ucap = cap;
    o.ucount = count;
    if (!launch_reg(scores, 1, L, L, k, mode, o, s)) return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_topk(const float* scores, int64_t B, int64_t L, int64_t k, int mode,
                       int32_t* out, hipStream_t s) {
    return launch_topk_strided(scores, B, L, L, k, mode, out, s);
}

}  // namespace si
