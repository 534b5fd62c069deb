// Token selection at the end of the prefill (Section 3.1.2, Algorithm 1 line 3): per unit keep the recent
// window and, of the other prompt tokens, the n_hh with the largest cumulative attention score; write the
// kept positions in ascending order.
//
// Two ways.  One workgroup per unit (select_kernel, after score_key_kernel where that cannot add the heads itself), and, for
// long prompts of few units, several (the sel_ kernels further down).
//   score_key_kernel   (only when a unit has several query heads) streams the rep fp32 score rows of a
//                      unit once, adds them in head order in fp32 and stores an order-preserving 32-bit
//                      key per token.  Grid over (unit, 4096-token chunk): the whole chip streams.
//   select_kernel      one workgroup of 16 waves per unit.  A radix select (digits of 11, 11 and 10 bits of the
//                      key from the top; LDS histogram, scan from the top bin down; the first digit is counted
//                      while the keys are read from memory) finds the key T of the weakest kept heavy hitter
//                      and how many tokens equal to T are kept; then one ordered compaction
//                      pass writes position i if key_i > T, or key_i == T and fewer than that many equal
//                      keys precede it, to slot (#larger before i) + min(#equal before i, kept equals).
//                      Equal scores therefore go to the earlier position and the output is ascending
//                      without a sort.  When the prompt fits, the keys are read from memory once and held
//                      in LDS (up to 32768 tokens = 128 KB) for the other passes.
#include "common.h"

#include <atomic>
#include <type_traits>

namespace minikv {

constexpr int kSelThreads = 1024;      // 16 waves: one workgroup per unit
constexpr int kSelBins = 2048;         // 11-bit digits
constexpr int kSelLoads = 8;           // keys per thread in flight in a histogram pass
constexpr int kSelSparse = 56;         // of a wave's 64 lanes with 8 keys each in such a step: matches in up to this
                                       // many lanes count as few
constexpr int kSelRangeLoads = 16;     // ... and in the first pass, which streams them from memory
constexpr int kSelFixedWords = kSelBins + 2 * 16 + 16 + 16;   // hist, compaction totals (two buffers), scan totals, result
constexpr int kSelMaxCached = 32768;   // most keys held in LDS

// Order-preserving map from finite floats to unsigned integers; the two zeros map to one key.
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// REP > 0: query heads per unit known at compile time, so that all REP x 4 loads of a step are in flight
// together; REP == 0: any number of heads, one load at a time.
template <int REP>
__global__ __launch_bounds__(256) void score_key_kernel(const float *__restrict__ A, uint32_t *__restrict__ keys,
                                                        int rep_rt, long L, int nchunk)
{
    const int rep = REP ? REP : rep_rt;
    const long unit = blockIdx.x / nchunk;
    const long base = (long)(blockIdx.x % nchunk) * 4096;
    const float *rows = A + unit * rep * L;
    for (int e0 = 0; e0 < 16; e0 += 4) {
        float s[4];
        if (REP) {
            float x[4][REP ? REP : 1];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const long i = min(base + (e0 + e) * 256 + (long)threadIdx.x, L - 1);   // clamped: no branch at the loads
#pragma unroll
                for (int h = 0; h < REP; ++h) x[e][h] = rows[h * L + i];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s[e] = x[e][0];
#pragma unroll
                for (int h = 1; h < REP; ++h) s[e] = s[e] + x[e][h];                   // head order, one rounding per add
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const long i = min(base + (e0 + e) * 256 + (long)threadIdx.x, L - 1);
                s[e] = rows[i];
                for (int h = 1; h < rep; ++h) s[e] = s[e] + rows[h * L + i];
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const long i = base + (e0 + e) * 256 + threadIdx.x;
            if (i < L) keys[unit * L + i] = score_key(s[e]);
        }
    }
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves only (no LDS traffic):
// shifts by 1, 2, 3 inside each row of 16 lanes, then by 4 and 8 on the lanes that have such a neighbour, then
// lane 15 of a row into the next row and lane 31 into the upper half.  A lane a move does not reach adds 0.
__device__ __forceinline__ int wave_scan_incl(int v)
{
    int s = v;
    s += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);     // row_shr:1
    s += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);     // row_shr:2
    s += __builtin_amdgcn_update_dpp(0, v, 0x113, 0xf, 0xf, true);     // row_shr:3
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xe, true);     // row_shr:4, lanes 4..15 of a row
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xc, true);     // row_shr:8, lanes 8..15 of a row
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xa, 0xf, false);    // row_bcast:15 into rows 1 and 3
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xc, 0xf, false);    // row_bcast:31 into rows 2 and 3
    return s;
}

// One more count for digit d from every lane with match set.  The lanes that share the first matching lane's
// digit are counted with one ballot and added once (constant or heavily tied scores would otherwise queue
// on one LDS address); the others add one each.
__device__ __forceinline__ void hist_add(int *hist, bool match, int d, int lane)
{
    const unsigned long long m = __ballot(match);
    if (m == 0) return;
    const int first = __ffsll((long long)m) - 1;
    const int d0 = __shfl(d, first, 64);
    const unsigned long long same = __ballot(match && d == d0);
    if (lane == first)
        atomicAdd(&hist[d0], (int)__popcll(same));
    else if (match && d != d0)
        atomicAdd(&hist[d], 1);
}

// FROM_FLOAT: the scores are read from A (REP rows per unit, added in head order in binary32 while they are read;
// with REP > 1 only when the keys then stay in LDS), else the keys score_key_kernel left in `keys`.
template <bool FROM_FLOAT, int REP = 1>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float *__restrict__ A,
                                                             const uint32_t *__restrict__ keys, long L,
                                                             const int *__restrict__ n_hh,
                                                             const int *__restrict__ n_rw,
                                                             int *__restrict__ idx, long idx_stride,
                                                             int *__restrict__ n_tok, int cached)
{
    extern __shared__ __align__(16) uint32_t smem[];
    int *hist = (int *)smem;                         // [kSelBins]
    int *sub_tot = hist + kSelBins;                  // [2][16]
    int *scan_tot = sub_tot + 2 * 16;                // [16]
    int *digit_found = scan_tot + 16;                // [3][4] digit, kept count below it, keys in the digit's bin
    uint32_t *ck = smem + kSelFixedWords;            // [L] when cached

    const long u = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(wave);             // the same number, known to be wave-uniform
    const long rw = n_rw[u], hh = n_hh[u];
    if (rw < 0 || hh < 0 || rw > L || hh > L - rw || hh + rw > idx_stride) {
        if (tid == 0) n_tok[u] = 0;
        return;
    }
    const int N = (int)(L - rw), k = (int)hh;
    int *row = idx + u * idx_stride;
    for (int j = tid; j < (int)rw; j += kSelThreads) row[k + j] = N + j;          // the recent window
    if (tid == 0) n_tok[u] = k + (int)rw;
    if (k == 0) return;
    if (k == N) {
        for (int j = tid; j < N; j += kSelThreads) row[j] = j;
        return;
    }
    const float *arow = A + u * REP * L;
    const uint32_t *krow = keys + u * L;
    // raw 32 bits of token i, and the key they stand for
    auto gload = [&](int i) -> uint32_t { return FROM_FLOAT ? __float_as_uint(arow[i]) : krow[i]; };
    auto gkey = [&](uint32_t raw) -> uint32_t { return FROM_FLOAT ? score_key(__uint_as_float(raw)) : raw; };
    // keys of tokens start .. start+3 (start a multiple of 4); tokens at or beyond N give unspecified values
    const int npad = (N + 3) & ~3;
    auto load4 = [&](int start, uint32_t *out) {
        if (cached) {
            const uint4 q = *(const uint4 *)&ck[min(start, npad - 4)];
            out[0] = q.x, out[1] = q.y, out[2] = q.z, out[3] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) out[j] = gload(min(start + j, N - 1));
#pragma unroll
            for (int j = 0; j < 4; ++j) out[j] = gkey(out[j]);
        }
    };

    // ---- radix select on the key, 11 + 11 + 10 bits from the top.  Bits hi and above of T are known (`prefix`);
    // `rem` = how many tokens sharing them are still to be kept.  The FIRST digit is counted while the keys are
    // read from memory (and go to LDS when they fit): that pass waits for memory, the LDS counting rides along.
    uint32_t prefix = 0;
    int rem = k, in_bin = 0;                             // (in_bin: after the last digit, the keys equal to T)
    int hi = 32;
    // bins from the top down, two per thread; the thread whose pair crosses `rem` owns the digit.  Every thread clears its
    // bins for the next digit as it reads them, and every digit has a result of its own: two barriers, not five (a barrier
    // of 16 waves is 0.1-0.2 us, and a short call does little else).
    auto settle_digit = [&](int lo) {
        const int c0 = hist[kSelBins - 1 - 2 * tid], c1 = hist[kSelBins - 2 - 2 * tid];
        hist[kSelBins - 1 - 2 * tid] = 0, hist[kSelBins - 2 - 2 * tid] = 0;
        int *found = digit_found + (lo >= 21 ? 0 : lo ? 4 : 8);
        int incl = wave_scan_incl(c0 + c1);
        if (lane == 63) scan_tot[wave] = incl;
        __syncthreads();
        {
            const int t = lane < 16 ? scan_tot[lane] : 0;              // totals of the 16 waves, one read
            const int ti = wave_scan_incl(t);
            incl += __builtin_amdgcn_readlane(ti, wv) - __builtin_amdgcn_readlane(t, wv);   // waves before mine
        }
        const int excl = incl - c0 - c1;
        if (excl < rem && rem <= incl) {
            const bool upper = excl + c0 >= rem;
            found[0] = kSelBins - 1 - 2 * tid - (upper ? 0 : 1);
            found[1] = rem - (upper ? excl : excl + c0);
            found[2] = upper ? c0 : c1;
        }
        __syncthreads();
        prefix |= (uint32_t)found[0] << lo;
        rem = found[1];
        in_bin = found[2];
        hi = lo;
    };
    for (int b = tid; b < kSelBins; b += kSelThreads) hist[b] = 0;
    __syncthreads();
    constexpr int NT = kSelRangeLoads / REP;             // tokens per thread and step: kSelRangeLoads loads in flight
    for (int base = 0; base < N; base += kSelThreads * NT) {
        uint32_t kk[NT];
        // every load of the step is issued before the first is used: indices clamped, no branches
        if (REP == 1) {
#pragma unroll
            for (int e = 0; e < NT; ++e) kk[e] = gload(min(base + e * kSelThreads + tid, N - 1));
#pragma unroll
            for (int e = 0; e < NT; ++e) kk[e] = gkey(kk[e]);
        } else {
            float x[NT][REP];
#pragma unroll
            for (int e = 0; e < NT; ++e)
#pragma unroll
                for (int h = 0; h < REP; ++h) x[e][h] = arow[h * L + min(base + e * kSelThreads + tid, N - 1)];
#pragma unroll
            for (int e = 0; e < NT; ++e) {
                float sum = x[e][0];
#pragma unroll
                for (int h = 1; h < REP; ++h) sum = sum + x[e][h];                          // head order, one rounding per add
                kk[e] = score_key(sum);
            }
        }
#pragma unroll
        for (int e = 0; e < NT; ++e) {
            const int i = base + e * kSelThreads + tid;
            if (cached && i < N) ck[i] = kk[e];
            hist_add(hist, i < N, (int)(kk[e] >> 21), lane);
        }
    }
    __syncthreads();
    settle_digit(21);
    // Further digits are needed only while the bin of the cut holds more keys than are kept from it.  Once ALL of
    // them are kept (typically after the second digit: 32768 keys over four million bins leave the weakest kept
    // key alone in its bin), T = the bin's lowest key does the same job, "kept" being key >= T.  (Only with the
    // keys in LDS: the compaction that re-reads them from memory keeps the exact T.)
    while (hi > 0 && !(cached && in_bin == rem)) {
        const int lo = max(hi - 11, 0);
        const uint32_t dm = (1u << (hi - lo)) - 1u;
        for (int base = 0; base < N; base += kSelThreads * kSelLoads) {
            // slot e of this thread holds token tok(e): from LDS two runs of 4 consecutive tokens (128-bit
            // reads), from memory consecutive lanes take consecutive tokens (coalesced); any order will do here
            uint32_t kk[kSelLoads];
            auto tok = [&](int e) {
                return cached ? base + ((e >> 2) * kSelThreads + tid) * 4 + (e & 3) : base + e * kSelThreads + tid;
            };
            if (cached) {
#pragma unroll
                for (int g = 0; g < kSelLoads / 4; ++g) load4(tok(4 * g), &kk[4 * g]);
            } else {
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e) kk[e] = gload(min(tok(e), N - 1));
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e) kk[e] = gkey(kk[e]);
            }
            bool match[kSelLoads];
            unsigned long long lanes = 0;              // lanes that hold a token still sharing the prefix
            const uint32_t span = hi < 32 ? 1u << hi : 0u;           // (hi < 32 here: the first digit is settled)
            if (base + kSelThreads * kSelLoads <= N) { // (uniform) all but the last step: every slot is a token
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e) {
                    match[e] = (kk[e] ^ prefix) < span;
                    lanes |= __ballot(match[e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e) {
                    match[e] = tok(e) < N && (kk[e] ^ prefix) < span;
                    lanes |= __ballot(match[e]);
                }
            }
            if (lanes == 0) continue;                  // after the first digit few tokens still share the prefix
            if (__popcll(lanes) <= kSelSparse) {
                // ... and those few spread over the bins: one plain LDS add each costs a fraction of the
                // ballots and shuffles of hist_add (5.4 -> 1.5 us for the second digit of 32768 keys)
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e)
                    if (match[e]) atomicAdd(&hist[(kk[e] >> lo) & dm], 1);
            } else {
                // many: ties or a narrow range of scores, which would queue on few LDS addresses
#pragma unroll
                for (int e = 0; e < kSelLoads; ++e) hist_add(hist, match[e], (int)((kk[e] >> lo) & dm), lane);
            }
        }
        __syncthreads();
        settle_digit(lo);
    }

    // ---- ordered compaction
    const uint32_t T = prefix;
    if (cached) {
        // Keys in LDS (at most kSelMaxCached of them, so at most 8 steps of 4096 tokens): every thread counts its 4
        // consecutive tokens of every step first -- one wave scan per step, no barrier --, the 8 x 16 wave totals
        // (in token order: step, then wave) are exchanged ONCE, and then every thread knows the slots of its
        // tokens.  (One barrier per step, as in the loop below, made this phase 7 of the kernel's 26 us.)
        constexpr int NS = kSelMaxCached / (kSelThreads * 4);
        uint32_t *tots = (uint32_t *)hist;             // [NS][16] packed counts: larger | equal << 16 (each < 65536)
        uint32_t before[NS];                           // counts of the lanes before this one in its wave, per step
        const int nsteps = (N + kSelThreads * 4 - 1) / (kSelThreads * 4);
        // When every key of T's bin is kept (the usual case: no tie across the cut), "kept" is just key >= T and
        // the bookkeeping of the equal ones falls away (3.7 instead of 5.9 us on 32768 tokens).
        const bool all_equal_kept = in_bin == rem;     // (uniform)
        // (whole steps, all but the last, compare without asking whether the token is a candidate)
        auto count = [&](int start, auto whole) -> uint32_t {
            uint32_t key[4], tot = 0;
            load4(start, key);
            if (all_equal_kept) {
#pragma unroll
                for (int j = 0; j < 4; ++j) tot += (uint32_t)((whole || start + j < N) && key[j] >= T);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t g = (whole || start + j < N) && key[j] > T, e = (whole || start + j < N) && key[j] == T;
                    tot += g | e << 16;
                }
            }
            return tot;
        };
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            before[st] = 0;
            if (st < nsteps) {                         // (uniform)
                const int start = st * kSelThreads * 4 + tid * 4;
                const uint32_t tot = (st + 1) * kSelThreads * 4 <= N ? count(start, std::true_type()) : count(start, std::false_type());
                const uint32_t incl = (uint32_t)wave_scan_incl((int)tot);
                before[st] = incl - tot;
                if (lane == 63) tots[st * 16 + wave] = incl;
            }
        }
        __syncthreads();
        // prefix over the (step, wave) totals: lane l holds entries 2l and 2l + 1
        const uint2 tv = lane < nsteps * 8 ? *(const uint2 *)&tots[2 * lane] : uint2{0u, 0u};
        const uint32_t pair_incl = (uint32_t)wave_scan_incl((int)(tv.x + tv.y));
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            if (st >= nsteps) break;
            const int e = st * 16 + wv;                // this wave's entry of the step (uniform)
            const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)pair_incl, e >> 1);   // through entry e | 1
            const uint32_t x1 = (uint32_t)__builtin_amdgcn_readlane((int)tv.y, e >> 1), x0 = (uint32_t)__builtin_amdgcn_readlane((int)tv.x, e >> 1);
            uint32_t excl = upto - x1 - ((e & 1) ? 0u : x0) + before[st];   // everything before this thread's 4 tokens
            const int start = st * kSelThreads * 4 + tid * 4;
            uint32_t key[4];
            load4(start, key);
            if (all_equal_kept) {
                // (excl < k always holds for a kept token; the test keeps a write in its row)
                if ((st + 1) * kSelThreads * 4 <= N) { // (uniform)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool g = key[j] >= T;
                        if (g && (int)excl < k) row[excl] = start + j;
                        excl += (uint32_t)g;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool g = start + j < N && key[j] >= T;
                        if (g && (int)excl < k) row[excl] = start + j;
                        excl += (uint32_t)g;
                    }
                }
                continue;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool g = start + j < N && key[j] > T, eq = start + j < N && key[j] == T;
                const int g_before = (int)(excl & 0xFFFFu), e_before = (int)(excl >> 16);
                // a larger key goes behind the larger ones and the kept equal ones before it; an equal one is kept
                // while fewer than rem came before it, and then sits at that same place
                const int slot = g_before + min(e_before, rem);
                if ((g || (eq && e_before < rem)) && slot < k) row[slot] = start + j;   // (slot < k always holds; the test keeps a write in its row)
                excl += (uint32_t)g | (uint32_t)eq << 16;
            }
        }
        return;
    }
    int gt_run = 0, eq_run = 0, buf = 0;
    for (int base = 0; base < N; base += kSelThreads * 4, buf ^= 1) {
        // 4 consecutive tokens per thread: their flags are summed in the thread, one scan per wave, and the 16
        // wave totals (in token order) are read and scanned by every wave after the barrier
        const int start = base + tid * 4;
        uint32_t key[4];
        load4(start, key);
        int f[4], tot = 0;                             // packed counts: larger | equal << 16
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[j] = start + j < N ? (int)(key[j] > T) | ((int)(key[j] == T) << 16) : 0;
            tot += f[j];
        }
        const int incl = wave_scan_incl(tot);
        if (lane == 63) sub_tot[buf * 16 + wave] = incl;
        __syncthreads();
        const int tv = lane < 16 ? sub_tot[buf * 16 + lane] : 0;
        const int ti = wave_scan_incl(tv);
        const int run = __builtin_amdgcn_readlane(ti, 15);
        int excl = __builtin_amdgcn_readlane(ti, wv) - __builtin_amdgcn_readlane(tv, wv) + incl - tot;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int g_before = gt_run + (excl & 0xFFFF), e_before = eq_run + (excl >> 16);
            int slot = -1;
            if (f[j] & 1)
                slot = g_before + min(e_before, rem);
            else if (f[j] && e_before < rem)
                slot = g_before + e_before;
            if (slot >= 0 && slot < k) row[slot] = start + j;   // slot < k always holds; the test keeps a write in its row
            excl += f[j];
        }
        gt_run += run & 0xFFFF;
        eq_run += run >> 16;
    }
}

// ------------------------------------------------------------------------------------------------------
// The same selection with SEVERAL workgroups per unit (prompts of up to kChMaxChunks * 4096 tokens): two launches over
// (unit, 4096-token chunk), 16 waves each, no atomics in memory, no waiting between workgroups.
//   sel_sort_kernel       streams the score rows once.  Per chunk: the candidates' keys in descending order of their top 11
//                         bits (a counting sort in LDS; inside a bin any order), and for every bin how many of them lie in
//                         it or above ("cumulative counts"); with several heads also the summed-score keys in token order.
//   sel_unit_hist_kernel  (only where adding a unit's cumulative counts in every workgroup would cost more than a launch)
//                         adds them up once.
//   sel_pick_kernel       every workgroup adds up its unit's cumulative counts -- the bin b1 of the weakest kept heavy hitter
//                         is where the sum falls below the budget, no scan --, fetches the unit's keys inside that bin, one
//                         contiguous piece per chunk, settles the remaining 21 bits on them in LDS, counts what precedes its
//                         chunks, and compacts those in order to the slots that follow.  (A bin of more keys than LDS holds --
//                         ties, but also a quarter of an octave that simply is the fullest -- is read again in each of the three
//                         passes: 16 units x 8 heads x 200000 'attention' scores 43 us with 40 % kept and 10586 keys in the bin,
//                         48 with 70 % and 14351.)
// A launch whose workgroups do a few dependent steps costs 4 to 9 us however small the input, so what counts is their number
// and the round trips inside.  An earlier form (histograms, a unit sum, a candidate list, the rest: four launches of 4
// waves per chunk) took 24.8 us on 8 units x 4 heads x 131072 where this takes 16.8 (the same scores every call; 27.0 and 19.3
// with two sets in turn), and 54 on 48 where this takes 47 (58.6 while the second launch had a workgroup for every four chunks,
// of which a compute unit held one at a time).
// Workspace, in 32-bit words: keys [units][Lp] (several heads only; Lp = L rounded up to 4), sorted keys
// [units][nchunk][4096], cumulative counts [units][nchunk][1024] (two 16-bit counts per word), sums of those
// [units][2048], four spare words per chunk.
constexpr int kCh = 4096;              // tokens per chunk
constexpr int kChThreads = 1024;       // 16 waves, four tokens each thread
constexpr int kChMaxChunks = 1024;     // most chunks of one unit
constexpr int kChList = 12288;         // keys of the cut's bin that sel_pick_kernel holds in LDS (more are read again in every pass)

struct SelWs {
    uint32_t *keys, *sorted, *cum;
    int *ucum;
    long Lp;
    int nchunk, units;
};

// Workgroup b of a launch over (unit, part), `parts` parts per unit: the hardware deals consecutive workgroups
// round-robin to the eight dies, each with an L2 of its own, so all parts of a unit are given numbers that are
// equal modulo 8 -- what one kernel writes for a unit is then still in the L2 of the die whose workgroups read
// it in the next (only speed depends on this).  Grids are sized by sel_grid_units(); false = no such unit.
__device__ __forceinline__ bool sel_map(unsigned b, int parts, int units, long &unit, int &part)
{
    if (units < 8) {                                       // fewer units than dies: spread every unit over all of them
        unit = b / (unsigned)parts;
        part = (int)(b % (unsigned)parts);
        return true;
    }
    const unsigned per = 8u * (unsigned)parts, g = b / per, r = b % per;
    unit = (long)g * 8 + (r & 7u);
    part = (int)(r >> 3);
    return unit < units;
}

static long sel_grid_units(long units) { return units < 8 ? units : (units + 7) / 8 * 8; }

__host__ __device__ inline long sel_ws_words(long units, int rep, long L)
{
    const long nchunk = (L + kCh - 1) / kCh, Lp = (L + 3) & ~3L;
    return units * ((rep > 1 ? Lp : 0) + nchunk * (kCh + kSelBins / 2 + 4) + kSelBins);
}

static SelWs sel_ws_carve(void *workspace, long units, int rep, long L)
{
    SelWs w;
    w.nchunk = (int)((L + kCh - 1) / kCh);
    w.units = (int)units;
    w.Lp = (L + 3) & ~3L;
    w.keys = (uint32_t *)workspace;
    w.sorted = w.keys + (rep > 1 ? units * w.Lp : 0);
    w.cum = w.sorted + units * (long)w.nchunk * kCh;
    w.ucum = (int *)(w.cum + units * (long)w.nchunk * (kSelBins / 2));
    return w;
}

// Budgets of a unit: false when they are out of range.  N = candidates (tokens before the recent window).
__device__ __forceinline__ bool sel_budgets(long r, long h, long L, long idx_stride, int &N, int &k, int &rw)
{
    if (r < 0 || h < 0 || r > L || h > L - r || h + r > idx_stride) return false;
    N = (int)(L - r), k = (int)h, rw = (int)r;
    return true;
}

// Inclusive prefix sum over the 1024 threads of a workgroup (tot[16] in LDS; one barrier); also the grand total.
__device__ __forceinline__ int block_scan_incl(int v, int *tot, int lane, int wv, int &total)
{
    int incl = wave_scan_incl(v);
    if (lane == 63) tot[wv] = incl;
    __syncthreads();
    const int t = lane < 16 ? tot[lane] : 0, ti = wave_scan_incl(t);
    incl += __builtin_amdgcn_readlane(ti, wv) - __builtin_amdgcn_readlane(t, wv);      // waves before this one
    total = __builtin_amdgcn_readlane(ti, 15);
    return incl;
}

// hist_add that also returns this lane's place among the keys of its digit (in the order they arrive).
__device__ __forceinline__ int hist_place(int *hist, bool match, int d, int lane)
{
    const unsigned long long m = __ballot(match);
    if (m == 0) return 0;
    const int first = __ffsll((long long)m) - 1;
    const int d0 = __shfl(d, first, 64);
    const unsigned long long same = __ballot(match && d == d0);
    int at = 0;
    if (lane == first)
        at = atomicAdd(&hist[d0], (int)__popcll(same));
    else if (match && d != d0)
        at = atomicAdd(&hist[d], 1);
    const int base = __builtin_amdgcn_readlane(at, first);
    return match && d == d0 ? base + (int)__popcll(same & ((1ull << lane) - 1ull)) : at;
}

template <int REP>
__global__ __launch_bounds__(kChThreads) void sel_sort_kernel(const float *__restrict__ A, SelWs w, int rep_rt, long L,
                                                              const int *__restrict__ n_hh,
                                                              const int *__restrict__ n_rw, long idx_stride)
{
    __shared__ int hist[kSelBins], tot[16];
    __shared__ uint32_t sorted[kCh];
    const int rep = REP ? REP : rep_rt;
    long unit;
    int chunk;
    if (!sel_map(blockIdx.x, w.nchunk, w.units, unit, chunk)) return;
    const long base = (long)chunk * kCh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long r_ = n_rw[unit], h_ = n_hh[unit];
    const float *rows = A + unit * rep * L;
    float x[4][REP ? REP : 1], s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const long i = min(base + e * kChThreads + (long)tid, L - 1);       // clamped: no branch at the loads
#pragma unroll
        for (int h = 0; h < (REP ? REP : 1); ++h) x[e][h] = rows[h * L + i];
    }
    hist[tid] = 0, hist[tid + kChThreads] = 0;
    int N = 0, k = 0, rw;                                  // the loads are on their way: now look at the budgets
    const bool live = sel_budgets(r_, h_, L, idx_stride, N, k, rw) && k != 0 && k != N && base < N;
    if (!live) return;                                     // nothing is selected by score here / no candidate in this chunk
    __syncthreads();
    int place[4];
    uint32_t key[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const long i = base + e * kChThreads + tid;
        s[e] = x[e][0];
        if (REP) {
#pragma unroll
            for (int h = 1; h < REP; ++h) s[e] = s[e] + x[e][h];                    // head order, one rounding per add
        } else {
            for (int h = 1; h < rep; ++h) s[e] = s[e] + rows[h * L + min(i, L - 1)];
        }
        key[e] = score_key(s[e]);
        if (REP != 1 && i < N) w.keys[unit * w.Lp + i] = key[e];
        place[e] = hist_place(hist, i < N, (int)(key[e] >> 21), lane);
    }
    __syncthreads();
    const int c0 = hist[2 * tid], c1 = hist[2 * tid + 1];
    int total;
    const int incl = block_scan_incl(c0 + c1, tot, lane, wv, total);
    const int ge1 = total - incl + c1, ge0 = ge1 + c0;     // keys in bin 2 tid + 1, 2 tid or above (at most 4096)
    w.cum[(unit * w.nchunk + chunk) * (long)(kSelBins / 2) + tid] = (uint32_t)ge0 | (uint32_t)ge1 << 16;
    hist[2 * tid] = ge1, hist[2 * tid + 1] = ge1 - c1;     // where the bin's keys start
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (base + e * kChThreads + tid < N) sorted[hist[key[e] >> 21] + place[e]] = key[e];
    __syncthreads();
    uint32_t *dst = w.sorted + (unit * w.nchunk + chunk) * (long)kCh;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = e * kChThreads + tid;
        if (i < total) dst[i] = sorted[i];
    }
}

// grid (units, 8): workgroup j of a unit adds bins 256j .. 256j+255 of the chunks that hold candidates
__global__ __launch_bounds__(256) void sel_unit_hist_kernel(SelWs w, long L, const int *__restrict__ n_hh,
                                                            const int *__restrict__ n_rw, long idx_stride)
{
    long unit;
    int part;
    if (!sel_map(blockIdx.x, 8, w.units, unit, part)) return;
    const int bin = part * 256 + threadIdx.x;
    int N, k, rw;
    if (!sel_budgets(n_rw[unit], n_hh[unit], L, idx_stride, N, k, rw) || k == 0 || k == N) return;
    const int nc = (N + kCh - 1) / kCh;
    const uint16_t *hp = reinterpret_cast<const uint16_t *>(w.cum + unit * w.nchunk * (long)(kSelBins / 2)) + bin;
    int sum = 0;
    for (int q0 = 0; q0 < nc; q0 += 8) {
        int v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = hp[(long)min(q0 + j, nc - 1) * kSelBins];
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += q0 + j < nc ? v[j] : 0;
    }
    w.ucum[unit * kSelBins + bin] = sum;
}

// DIRECT: the unit's cumulative counts are added up here, else sel_unit_hist_kernel has done it.  A workgroup compacts `per`
// consecutive chunks ("chunk" is the first; ONE: one, known at compile time).
template <bool FROM_FLOAT, bool DIRECT, bool ONE>
__global__ __launch_bounds__(kChThreads, ONE ? 4 : 8) void sel_pick_kernel(const float *__restrict__ A, SelWs w, long L,
                                                              const int *__restrict__ n_hh,
                                                              const int *__restrict__ n_rw,
                                                              int *__restrict__ idx, long idx_stride,
                                                              int *__restrict__ n_tok, int per_rt)
{
    __shared__ int hist[kSelBins];                         // (first: piece ends and starts of the chunks)
    __shared__ uint32_t list[kChList];
    __shared__ int tot[16], tot2[16], found[2], acc[4];
    long unit;
    int chunk;
    const int per = ONE ? 1 : per_rt;
    if (!sel_map(blockIdx.x, (w.nchunk + per - 1) / per, w.units, unit, chunk)) return;
    chunk *= per;
    const int base = chunk * kCh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long r_ = n_rw[unit], h_ = n_hh[unit];
    // a chunk's keys for the compaction: tokens base + 4096 r + 4 tid .. + 3 (the first chunk's are requested now, used last)
    uint32_t key[4];
    auto request = [&](int r) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const long i = min((long)base + r * kCh + 4 * tid + j, L - 1);
            key[j] = FROM_FLOAT ? __float_as_uint(A[unit * L + i]) : w.keys[unit * w.Lp + i];
        }
    };
    request(0);
    const uint32_t *crow = w.cum + unit * w.nchunk * (long)(kSelBins / 2);
    int N, k, rw;
    if (!sel_budgets(r_, h_, L, idx_stride, N, k, rw)) {
        if (chunk == 0 && tid == 0) n_tok[unit] = 0;
        return;
    }
    int *row = idx + unit * idx_stride;
    const int end = (int)min((long)base + (long)per * kCh, L);
    for (int i = max(base, N) + tid; i < end; i += kChThreads) row[k + (i - N)] = i;       // the recent window
    if (chunk == 0 && tid == 0) n_tok[unit] = k + rw;
    if (k == 0 || base >= N) return;
    if (k == N) {
        for (int i = base + tid; i < min(end, N); i += kChThreads) row[i] = i;
        return;
    }
    const int nc = (N + kCh - 1) / kCh;
    // ---- keys of the unit in bin 2 tid / 2 tid + 1 or above; b1 = the last bin where at least k are
    int ge0 = 0, ge1 = 0;
    if (DIRECT) {
        for (int q0 = 0; q0 < nc; q0 += 32) {              // (32 loads in flight: one round trip up to 131072 tokens)
            uint32_t v[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) v[j] = crow[(long)min(q0 + j, nc - 1) * (kSelBins / 2) + tid];
#pragma unroll
            for (int j = 0; j < 32; ++j)
                if (q0 + j < nc) ge0 += (int)(v[j] & 0xFFFFu), ge1 += (int)(v[j] >> 16);
        }
    } else {
        const int2 v = reinterpret_cast<const int2 *>(w.ucum + unit * kSelBins)[tid];
        ge0 = v.x, ge1 = v.y;
    }
    if (lane == 0) tot[wv] = ge0;
    if (tid < 4) acc[tid] = 0;
    __syncthreads();
    {
        const int below = __shfl_down(ge0, 1, 64);         // of the bin after this thread's two
        const int next = lane < 63 ? below : wv < 15 ? tot[(wv + 1) & 15] : 0;
        if (ge0 >= k && ge1 < k) found[0] = 2 * tid;
        if (ge1 >= k && next < k) found[0] = 2 * tid + 1;
    }
    __syncthreads();
    const uint32_t b1 = (uint32_t)found[0];
    // ---- chunk q = tid: where its keys of bin b1 start in its sorted list (= how many lie above), and how many there are
    int gt = 0, cnt = 0;
    if (tid < nc) {
        const uint16_t *cq = reinterpret_cast<const uint16_t *>(crow + (long)tid * (kSelBins / 2)) + b1;
        gt = b1 + 1 < (uint32_t)kSelBins ? cq[1] : 0;
        cnt = cq[0] - gt;
    }
    int M, above_all;
    const int cnt_end = block_scan_incl(cnt, tot2, lane, wv, M);
    const int gt_end = block_scan_incl(gt, tot, lane, wv, above_all);
    int *piece_at = hist, *piece_end = hist + kChMaxChunks;          // start in the chunk's list; end among the unit's bin keys
    piece_at[tid] = gt, piece_end[tid] = cnt_end;
    if (tid == chunk) acc[2] = gt_end - gt, acc[3] = cnt_end - cnt;  // keys above the bin / in it, in the chunks before this one
    __syncthreads();
    const int above_before = acc[2], m_before = acc[3];
    const uint32_t *sorted = w.sorted + unit * w.nchunk * (long)kCh;
    // f(key, index): the unit's bin keys, from their pieces in memory (wave v takes chunks v, v + 16, ...)
    auto from_pieces = [&](auto f) {
        for (int q = wv; q < nc; q += 16) {
            const int e = piece_end[q], b = q ? piece_end[q - 1] : 0;
            const uint32_t *src = sorted + (long)q * kCh + piece_at[q] - b;
            for (int i = b + lane; i < e; i += 64) f(src[i], i);
        }
    };
    const bool listed = M <= kChList;                      // (uniform)
    int rem = k - above_all;
    uint32_t T = 0;
    int g = 0, eq = 0;
    if (listed) {
        // as from_pieces, but 256 keys of each of two pieces are requested before the first is stored
        for (int q0 = wv; q0 < nc; q0 += 32) {
            int at[2], b[2], e[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int q = min(q0 + 16 * p, nc - 1);
                e[p] = q0 + 16 * p < nc ? piece_end[q] : 0, b[p] = q ? piece_end[q - 1] : 0;
                at[p] = q * kCh + piece_at[q] - b[p];
            }
            uint32_t x[2][4];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) x[p][j] = sorted[at[p] + max(min(b[p] + 64 * j + lane, e[p] - 1), b[p])];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (b[p] + 64 * j + lane < e[p]) list[b[p] + 64 * j + lane] = x[p][j];
                for (int i = b[p] + 256 + lane; i < e[p]; i += 64) list[i] = sorted[at[p] + i];
            }
        }
        __syncthreads();
        // the 21 bits below the bin's: 11, then 10
#pragma unroll 1
        for (int level = 0; level < 2; ++level) {
            const int lo = level ? 0 : 10;
            const uint32_t dm = level ? 0x3FFu : 0x7FFu;
            hist[tid] = 0, hist[tid + kChThreads] = 0;
            __syncthreads();
            for (int i = tid; i < M; i += kChThreads) {
                const uint32_t x = list[i];
                if (level == 0 || ((x >> 10) & 0x7FFu) == (T >> 10)) atomicAdd(&hist[(x >> lo) & dm], 1);
            }
            __syncthreads();
            const int c0 = hist[2 * tid], c1 = hist[2 * tid + 1];
            int total;
            const int incl = block_scan_incl(c0 + c1, level ? tot2 : tot, lane, wv, total);
            const int run = total - incl;                  // count in the bins above this thread's
            if (run < rem && rem <= run + c1) found[0] = 2 * tid + 1, found[1] = rem - run;
            if (run + c1 < rem && rem <= run + c1 + c0) found[0] = 2 * tid, found[1] = rem - run - c1;
            __syncthreads();
            T |= (uint32_t)found[0] << lo;
            rem = found[1];
        }
        for (int i = tid; i < m_before; i += kChThreads) {
            const uint32_t x = list[i] & 0x1FFFFFu;
            g += (int)(x > T), eq += (int)(x == T);
        }
    } else {
        // ties or a narrow range of scores: most keys share the bin, and many of them a digit.  The counts cannot use the
        // bytes that describe the pieces: they take the list's.
        int *count = (int *)list;
#pragma unroll 1
        for (int level = 0; level < 2; ++level) {
            const int lo = level ? 0 : 10;
            const uint32_t dm = level ? 0x3FFu : 0x7FFu;
            count[tid] = 0, count[tid + kChThreads] = 0;
            __syncthreads();
            from_pieces([&](uint32_t x, int) {
                hist_add(count, level == 0 || ((x >> 10) & 0x7FFu) == (T >> 10), (int)((x >> lo) & dm), lane);
            });
            __syncthreads();
            const int c0 = count[2 * tid], c1 = count[2 * tid + 1];
            int total;
            const int incl = block_scan_incl(c0 + c1, level ? tot2 : tot, lane, wv, total);
            const int run = total - incl;
            if (run < rem && rem <= run + c1) found[0] = 2 * tid + 1, found[1] = rem - run;
            if (run + c1 < rem && rem <= run + c1 + c0) found[0] = 2 * tid, found[1] = rem - run - c1;
            __syncthreads();
            T |= (uint32_t)found[0] << lo;
            rem = found[1];
        }
        from_pieces([&](uint32_t x, int i) {
            g += (int)(i < m_before && (x & 0x1FFFFFu) > T), eq += (int)(i < m_before && (x & 0x1FFFFFu) == T);
        });
    }
    const uint32_t Tfull = (b1 << 21) | T;                 // key of the weakest kept heavy hitter; `rem` of its equals are kept
    // larger / equal keys among the bin keys of the chunks before this one
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        g += __shfl_xor(g, d, 64);
        eq += __shfl_xor(eq, d, 64);
    }
    if (lane == 0 && (g | eq)) {
        atomicAdd(&acc[0], g);
        atomicAdd(&acc[1], eq);
    }
    __syncthreads();
    int gt_run = above_before + acc[0], eq_run = acc[1];
    // ---- ordered compaction of the chunks: 4 consecutive tokens per thread
    for (int r = 0; r < per && base + r * kCh < N; ++r) {  // (uniform)
        const int start = base + r * kCh + 4 * tid;
        int f[4], sum = 0;                                 // packed counts: larger | equal << 16
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = FROM_FLOAT ? score_key(__uint_as_float(key[j])) : key[j];
            f[j] = start + j < N ? (int)(x > Tfull) | ((int)(x == Tfull) << 16) : 0;
            sum += f[j];
        }
        if (!ONE && r + 1 < per) request(r + 1);
        int total;
        int excl = block_scan_incl(sum, r & 1 ? tot2 : tot, lane, wv, total) - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int g_before = gt_run + (excl & 0xFFFF), e_before = eq_run + (excl >> 16);
            int slot = -1;
            if (f[j] & 1)
                slot = g_before + min(e_before, rem);
            else if (f[j] && e_before < rem)
                slot = g_before + e_before;
            if (slot >= 0 && slot < k) row[slot] = start + j;   // slot < k always holds; the test keeps a write in its row
            excl += f[j];
        }
        gt_run += total & 0xFFFF;
        eq_run += total >> 16;
    }
}

static std::atomic<int> g_select_path{0};

bool set_select_path(int path)
{
    if (path < 0 || path > 2) return false;
    g_select_path.store(path);
    return true;
}

// Several workgroups per unit pay two dependent launches and read the keys twice; they win when
// one workgroup per unit would leave most of the chip idle.
static bool select_chunked(int32_t units, int32_t rep, int64_t L)
{
    const long nchunk = (L + kCh - 1) / kCh;
    if (L <= 0 || nchunk > kChMaxChunks || ((long)units + 7) * nchunk > 0x7FFFFFFFL) return false;
    const int path = g_select_path.load();
    if (path) return path == 2;
    // Prompts whose keys one workgroup cannot hold in LDS, up to 128 units (one workgroup against several: 128 units x 32769
    // 30.4 -> 29.9 us with one head, 42 -> 35 with four; 160 units 30.5 -> 35.9 and 46 -> 42, 160 x 65536 56.4 -> 56.8), and of
    // those it can hold the long ones while every workgroup of the second launch has a compute unit: the units are dealt to the
    // dies by eights (1 and 8 heads, 32 units x 24577 16.1 -> 15.0, 17.3 -> 16.8, 36 units 16.1 -> 19.6, 17.6 -> 23.3; 32 x
    // 32768 18.7 -> 15.6, 21.4 -> 19.1).  Sums of a number of heads that select_kernel does not add itself take it a launch
    // more: there the last die may share some (3 heads, 36 x 24577 24.1 -> 21.7).
    if (nchunk > 8) return units <= 128;
    const bool adds = rep == 1 || rep == 2 || rep == 4 || rep == 8;
    return nchunk > 6 && (adds ? sel_grid_units(units) : units) * nchunk <= kComputeUnits;
}

size_t select_workspace_bytes(int32_t units, int32_t rep, int64_t L)
{
    if (units <= 0 || rep < 1 || L <= 0) return 0;
    if ((L + kCh - 1) / kCh > kChMaxChunks)                 // one workgroup per unit: only the summed-score keys
        return rep > 1 ? (size_t)units * (size_t)L * sizeof(uint32_t) : 0;
    return (size_t)sel_ws_words(units, rep, L) * sizeof(uint32_t);
}

template <bool FROM_FLOAT, bool ONE>
static void launch_pick(const float *A, const SelWs &w, int per, int32_t units, int64_t L, const int32_t *n_hh, const int32_t *n_rw,
                        int32_t *idx, int64_t idx_stride, int32_t *n_tok, hipStream_t st)
{
    const long units8 = sel_grid_units(units), parts = (w.nchunk + per - 1) / per;
    const dim3 grid((unsigned)(units8 * parts));
    // Every workgroup reads 4 KB of counts per chunk of its unit from its die's L2: units / 8 * parts * nchunk * 4 KB per die
    // at 2 KB a cycle.  Up to 3 us of that are less than the launch that adds them once costs.
    if (w.nchunk <= 64 && units * parts * w.nchunk <= 24576) {
        hipLaunchKernelGGL((sel_pick_kernel<FROM_FLOAT, true, ONE>), grid, dim3(kChThreads), 0, st, A, w, (long)L, n_hh, n_rw, idx,
                           (long)idx_stride, n_tok, per);
    } else {
        hipLaunchKernelGGL(sel_unit_hist_kernel, dim3((unsigned)(units8 * 8)), dim3(256), 0, st, w, (long)L, n_hh, n_rw,
                           (long)idx_stride);
        hipLaunchKernelGGL((sel_pick_kernel<FROM_FLOAT, false, ONE>), grid, dim3(kChThreads), 0, st, A, w, (long)L, n_hh, n_rw, idx,
                           (long)idx_stride, n_tok, per);
    }
}

int launch_select(int32_t units, int32_t rep, int64_t L, const float *A, const int32_t *n_hh,
                  const int32_t *n_rw, int32_t *idx, int64_t idx_stride, int32_t *n_tok, void *workspace,
                  hipStream_t st)
{
    if (units == 0) return MINIKV_OK;
    if (select_chunked(units, rep, L)) {
        const SelWs w = sel_ws_carve(workspace, units, rep, L);
        const dim3 grid((unsigned)(sel_grid_units(units) * w.nchunk));
        auto k1 = rep == 1   ? sel_sort_kernel<1>
                  : rep == 2 ? sel_sort_kernel<2>
                  : rep == 4 ? sel_sort_kernel<4>
                  : rep == 8 ? sel_sort_kernel<8>
                             : sel_sort_kernel<0>;
        hipLaunchKernelGGL(k1, grid, dim3(kChThreads), 0, st, A, w, rep, (long)L, n_hh, n_rw, (long)idx_stride);
        // One workgroup per compute unit, each with as many chunks as that leaves it: a second one repeats the work on the cut
        // (4 heads: 32 units x 32769 21.5 -> 19.2 us for the call, 16 x 131072 28.7 -> 25.0, 8 x 200000 30.9 -> 25.1).
        const int most = (int)max(kComputeUnits / sel_grid_units(units), 1L), per = (w.nchunk + most - 1) / most;
        const auto pick = rep == 1 ? (per == 1 ? launch_pick<true, true> : launch_pick<true, false>)
                                   : per == 1 ? launch_pick<false, true> : launch_pick<false, false>;
        pick(A, w, per, units, L, n_hh, n_rw, idx, idx_stride, n_tok, st);
        return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
    }
    // keys stay in LDS when the whole prompt fits beside the fixed part
    int dev = 0, max_lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return MINIKV_ELAUNCH;
    long cap = ((long)max_lds - kSelFixedWords * 4) / 4;
    if (cap > kSelMaxCached) cap = kSelMaxCached;
    int cached = L > 0 && L <= cap;
    size_t lds = (size_t)kSelFixedWords * 4 + (cached ? (size_t)((L + 3) / 4 * 4) * 4 : 0);
    // with 2, 4 or 8 heads per unit and the keys held in LDS, the select kernel adds the heads' rows itself while
    // it reads them; otherwise (other head counts, or prompts whose keys are read again in every pass) the
    // streaming kernel leaves the summed-score keys in the workspace first
    const bool fused = cached && (rep == 2 || rep == 4 || rep == 8);
    auto kern = rep == 1            ? select_kernel<true, 1>
                : !fused            ? select_kernel<false, 1>
                : rep == 2          ? select_kernel<true, 2>
                : rep == 4          ? select_kernel<true, 4>
                                    : select_kernel<true, 8>;
    if (cached && lds > 48 * 1024 &&
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        cached = 0;                                    // read the keys from memory in every pass instead
        lds = (size_t)kSelFixedWords * 4;
        if (rep > 1) kern = select_kernel<false, 1>;
    }
    uint32_t *keys = (uint32_t *)workspace;
    if (rep > 1 && L > 0 && kern == select_kernel<false, 1>) {
        const int nchunk = (int)((L + 4095) / 4096);
        auto k1 = rep == 2 ? score_key_kernel<2> : rep == 4 ? score_key_kernel<4> : rep == 8 ? score_key_kernel<8>
                                                                                            : score_key_kernel<0>;
        hipLaunchKernelGGL(k1, dim3((unsigned)((long)units * nchunk)), dim3(256), 0, st, A, keys, rep, (long)L,
                           nchunk);
        if (hipGetLastError() != hipSuccess) return MINIKV_ELAUNCH;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)units), dim3(kSelThreads), lds, st, A, keys, (long)L, n_hh, n_rw,
                       idx, (long)idx_stride, n_tok, cached);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

}  // namespace minikv
