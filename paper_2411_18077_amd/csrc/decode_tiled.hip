// Decode attention over the packed 2-bit cache: the one-launch kernel of minikv_decode_attn (gfx950, wave64).
//
// Computes Algorithm 1 lines 17-19 of the MiniKV paper (scores of the dequantized keys and the fp16
// residual keys, one softmax, weighted dequantized + residual values; eq. (1) scale passed in) with the
// dequantization folded into both products (Section 3.3, "fused unpacking and multiplication"):
//
//   score_t = sum_c (q_c * Ks[g,c]) * code_tc  +  sum_c q_c * Kz[g,c]          g = t / G
//   out_c   = sum_t (p_t * Vs[t,gc]) * code_tc +  sum_t p_t * Vz[t,gc]         gc = c / G
//
// so the inner products run over the raw 2-bit codes and the scales move onto the small operands.
//
// Work split: one workgroup of eight waves (four at G = 16) per compute unit.  A flat, weighted list of work items
// (items of 64 fp16 residual tokens, passes of 128 quantized tokens) over all (batch, KV head) units is cut
// into equal ranges, one per wave; see "Work distribution" below.  Every wave keeps one online-softmax
// state per unit it touches, the waves of a workgroup merge theirs in local memory, and the last workgroup to finish a
// unit merges the unit's partial results, all inside one launch.
//
// One pass of 128 quantized tokens, lane l of the wave:
//   K phase: the lane owns tokens 2l and 2l+1; four 128-bit loads bring their 2 x 8 code words.  Codes
//     are NOT converted: (word & (0x00030003 << 2j)) is used directly as two fp16 SUBNORMALS
//     code * 4^j * 2^-24 (j <= 4 keeps the field inside the mantissa; fields 5..7 come from the word
//     shifted right by 6), the 4^-j sits on the other operand and the 2^24 on the result.  The products
//     go to v_mfma_f32_4x4x4f16: 16 blocks = 64 tokens per instruction, lane = token, the 4 result
//     registers = 4 query heads, k = 4 channels.  The other operand, q_c * Ks[g,c] for (head, 4 channels),
//     is an exact fp16 pair (hi, lo) computed in registers by the lanes of the token's K group and handed
//     to the whole group by the instruction's block broadcast (cbsz / abid), so it never touches LDS;
//     the K scale / zero rows are stored so that each lane's channel quads are contiguous.
//   softmax: per-head wave maximum (DPP), lazy rescale of the accumulators, p = exp2(score - m).
//   V phase: the lane owns channels l and l+64.  ps[gc][h][t] = p * Vs * 2^4 * 4^-j(t) goes through LDS as
//     fp16 (written by the token lanes, read once by the lanes that supply it, again broadcast by the
//     instruction); the V words (16 tokens of one channel, even tokens in the low half-word) are masked
//     like the K words and multiplied 4 tokens x 4 heads at a time.  The zero-point term is accumulated
//     per lane in fp32 and reduced once per unit and wave.
//
// Input domain: every finite fp16 input.  The fp16 operands of the matrix instructions hold |q * Ks| < 65504
// and V scales < 4096 with the default scalings; a wave whose sums show an overflow repeats its share of the
// unit with range-normalised operands (see "Operand ranges" in the kernel).
#include <atomic>
#include <type_traits>

#include "decode_wave.h"

namespace minikv {

// ------------------------------------------------------------------------------------------------
// Work distribution.  Every unit (batch, KV head, set of 4 query heads) has ceil(R/64) residual items and
// ceil(T/128) quantized passes; its span of the weight line holds the even residual items, the passes,
// then the odd residual items (so that the usual two items fall to two different waves).  The units'
// spans (2^wr_log per residual item, 2^wq_log per pass) are laid end to end and the line is cut into NW equal
// ranges, one per wave; a wave owns the items that START inside its range, so ragged lengths are balanced
// by construction.  A workgroup has the ranges of its waves side by side.  What its waves do for one unit ends in one
// split-K partial (running max, sum, un-normalised output), merged in local memory; where several workgroups share a unit,
// the partial that arrives last (device-scope ticket counter) merges the unit's partials, and the fp16 output is written: one
// kernel launch does the whole call.  (Drawing passes from a per-unit counter instead was tried: a vector
// atomic per pass, even one whose result is needed a full pass later, slowed the pass loop by 40 %.)
//
// What bounds a call whose waves have a few items each is the chain behind the last pass: a partial per WAVE, merged through
// memory in two levels of up to sixteen, cost 4 to 8 us of round trips, and a range had to hold a whole residual item (3.5
// passes), so that 700 items ran on 128 waves one after the other.  With a partial per workgroup a unit has at most sixteen or
// so, one level merges them, and a range can be shorter than an item (only a workgroup's range must hold one).  Fused steps, us:
// 8 heads x 7168 tokens 18.9 -> 12.2 (G = 64), 32 x 5120 20.2 -> 13.0, 32/8 heads x 16 x 13088 39.4 -> 37.2; attention 1024 units x
// 4896 96.7 -> 93.1, ragged 128k 42.5 -> 40.7 (41.0 -> 40.3 on another box, inside its noise); 1.15 times in the geometric mean
// over 233 shapes from 8 to 1024 units.  Behind (0.93-0.97) where a call does not wait for the chain: 512 units and more of at most
// four passes each and no residual token, or of one pass and the new token only (1024 units x 512, one head, G = 32 18.4 -> 19.9);
// with residual tokens the same units gain 1.05 to 1.5 times.
struct UnitItems { int nq, nr, T, R, rn; };   // rn: residual row the fused step appends (-1: none)
constexpr int kSkew16 = 10;             // share (in sixteenths) of a wave pair's range given to its first wave

// Residual tokens a unit attends to: its stored ones, plus -- in the fused step -- the token this launch appends
// (when the buffer has room for it, as kv_append_residual would).
// A 32-bit word that no kernel of this launch writes, read through the constant address space: a wave-uniform
// address then gets a scalar load, which does not queue behind the wave's outstanding vector loads.  (Without
// this the fused step's stores of 32-bit words make the compiler read the lengths with vector loads.)
__device__ inline int load_const_i32(const int32_t *p)
{
    typedef const __attribute__((address_space(4))) int32_t *const_ptr;
    return *(const_ptr)(uintptr_t)p;
}
// (bit kAppBit of the result says that a token is appended, so that one register carries both facts)
constexpr int kAppBit = 20;
__device__ inline int res_len(bool APPEND, const DecArgs &a, int r)
{
    const int rc = clampi(r, 0, a.Rcap);
    return APPEND && r >= 0 && r < a.Rcap ? (rc + 1) | (1 << kAppBit) : rc;
}
__device__ inline UnitItems make_items(bool APPEND, int T, int Rtag)
{
    const int R = APPEND ? Rtag & ((1 << kAppBit) - 1) : Rtag;
    return UnitItems{(T + kPass - 1) / kPass, (R + 63) / 64, T, R, APPEND && (Rtag >> kAppBit) ? R - 1 : -1};
}
__device__ inline UnitItems unit_items(bool APPEND, const DecArgs &a, int up)
{
    const int u = up >> a.hs_shift;
    return make_items(APPEND, clampi(load_const_i32(a.q_len + u), 0, a.Tcap), res_len(APPEND, a, load_const_i32(a.r_len + u)));
}
// P weight units are cut into NW = 2^nw_log ranges.  Waves 2p and 2p+1 share the pair range
// [p*2P >> nw_log, (p+1)*2P >> nw_log); the first of them takes skew16/16 of it (8 = equal halves).
__device__ inline int range_start(int w, int P, int nw_log, int skew16)
{
    const int s0 = (int)(((long)(w >> 1) * P) >> (nw_log - 1));
    if (!(w & 1)) return s0;
    const int s1 = (int)(((long)((w >> 1) + 1) * P) >> (nw_log - 1));
    return s0 + (int)(((long)(s1 - s0) * skew16) >> 4);
}
// wave that owns position i: binary32 estimate, then exact correction against the range bounds
__device__ inline int wave_of(int i, int P, int nw_log, float inv_p, int skew16)
{
    int w = (int)((float)i * inv_p);                       // inv_p = NW / P
    w = min(max(w, 0), (1 << nw_log) - 1);
    while (range_start(w, P, nw_log, skew16) > i) w--;
    while (range_start(w + 1, P, nw_log, skew16) <= i) w++;
    return w;
}

// wave-wide inclusive prefix sum of an int (lane 63 ends up with the total)
__device__ inline int wave_scan_i32(int v)
{
    asm volatile("s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n s_nop 1\n"
                 "v_add_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n"
                 : "+v"(v));
    return v;
}
__device__ inline int wave_sum_i32(int v) { return __builtin_amdgcn_readlane(wave_scan_i32(v), 63); }

// Two waves per SIMD, except for G = 16, whose per-lane share of the K scale / zero rows and of q*Ks does not
// fit 256 registers: one wave per SIMD with the full register file runs 1.6x faster there than two that
// spill (the pass loop is bound by instruction issue, which one wave nearly saturates).
//
// PAIRED (units with at most two query heads, i.e. multi-head attention): the four rows of the K-phase
// A operand are (head 0 hi, head 0 lo, head 1 hi, head 1 lo) instead of four heads, so one matrix
// instruction does the work of the hi and the lo one, and the two result rows of a head are added afterwards.
//
// FUSED: the instance that serves the fused decode step (the plain call compiles none of it).  Inside it the
// step's code still hangs on the run-time flag a.append and not on the template parameter: measured on the
// 16 x 32768 workload, the instance built with the flag as a constant ran 3 us (7 %) slower, with or without a
// token to append -- the compiler then arranges the unit set-up and the residual item differently.
//
// UNIT: a workgroup of kGroupWaves waves IS one unit; they divide its items, and their partials meet in local memory.
// What a small launch spends its time on is round trips -- lengths to work line, partial to ticket, ticket to merge --,
// and this form has one of them, the unit's own two lengths: see unit_per_workgroup() for where it is taken.  It has no loop
// over units (the compiler is told: while it allowed for a second one, half of the instances kept 20 to 80 scalar registers in
// vector ones), its residual items stand in one place, behind the passes, on waves that have a pass less.  us, before -> now: fused
// step, 8 heads x 1024 10.7 -> 8.0, 32/8 heads x 512, two residual items 11.5 -> 7.6, 240 units x 1024 13.6 -> 10.8, attention, G = 16 x
// 2048, 256 units 16.4 -> 15.7, with two residual items 19.2 -> 17.7.  Requesting a wave's first tiles together with the lengths, a
// round trip less, was tried on up to 64 units and lost: the tiles' registers were then written on two paths, and every instance
// paid for it, also where the branch was not taken (8 heads x 1024 8.0 -> 8.7, 216 units x 896 5.7 -> 6.1, 1.05 times in the
// geometric mean over 880 shapes; only 64 units x 12 passes, four heads, gained, 10.2 -> 9.7).
//
// STREAM: the code words are loaded with the streaming hint, where a call reads each of them once (one set of heads); without
// the hint they push each other through the caches, and the read rate is what suffers: see launch_stream() for where and how much.
template <int G> constexpr int kGroupWaves = G == 16 ? 4 : 8;     // (two per SIMD, one at G = 16)
template <int G, bool LO, bool PAIRED, bool FUSED, bool UNIT, bool STREAM>
__global__ __launch_bounds__(64 * kGroupWaves<G>, G == 16 ? 1 : 2) void decode_stream_kernel(DecArgs a)
{
    constexpr int kWaves = kGroupWaves<G>, kWavesLog = ilog2(kWaves);
    constexpr int kPrH = 72, kPrHalfs = UNIT ? kNH * kD : kNH * kPrH;        // weights of a residual item [kNH][64 + 8], in front of its rows
    constexpr int kLdsHalfs = kPrHalfs + 64 * kKRowH;      // local memory of one wave
    static_assert(kLdsHalfs >= (kD / G) * kPsG && kLdsHalfs * 2 >= kNH * kPartialStride * 4, "weights of a pass; a partial");
    const int wq_log = UNIT ? 0 : a.wq_log, wr_log = UNIT ? 0 : a.wr_log, kWQ = 1 << wq_log, kWR = 1 << wr_log;
    const bool APPEND = FUSED && a.append;
    static_assert(!PAIRED || LO, "the paired rows are the hi and lo parts");
    constexpr int NHQ = PAIRED ? 2 : kNH;                  // heads the quantized passes work on
    // K side: a K group spans G/2 token-lanes = BGK blocks of 4 lanes.  Block j of a group supplies the
    // A operand (4 heads x 4 channels of q*Ks) of k-steps j, j+BGK, ...; the matrix instruction
    // broadcasts it to the other blocks of the group (cbsz = log2 BGK, abid = j).
    constexpr int BGK = G / 8, CBK = ilog2(BGK), NKR = 32 / BGK;
    // V side: the lanes' channels lane, lane+64 share a channel group in runs of BGV blocks.
    constexpr int BGV = G / 4 < 16 ? G / 4 : 16, CBV = ilog2(BGV), NVR = 32 / BGV;
    constexpr int NCG = kD / G;
    constexpr int NKW = NKR * 2;                           // words of one lane's slice of a K meta row
    typedef KData<NKW> KD;
    typedef VData<NCG> VD;
    // The tiles that a wave's last pass requests are used by nobody.  Its own ones again are still cached, but not with the
    // streaming hint; they then came from memory a second time (190.1 MB read per call on the 16 x 32768 workload, 177.6
    // without the hint).  So every wave of the work line requests the same tile there, the first unit's first: 176.1 MB (171.6 since a
    // workgroup has one partial), 1024
    // units x 4896 98.2 -> 96.5 us, 512 x 4864 53.8 -> 51.9, 128 x 13088, two heads, 35.6 -> 34.7, four 36.6 -> 36.1.
    constexpr bool kOneTile = !UNIT || (STREAM && !(FUSED && !PAIRED && G == 32));   // (that instance has no register left)

    __shared__ __attribute__((aligned(16))) _Float16 lds_all[kWaves * kLdsHalfs];
    // A wave's partials of the unit its range begins with and of the one it ends with are entries 2 * pos and 2 * pos + 1
    // (pos: the wave's place in the workgroup's range): which unit, its first and last workgroup, the row appended to it
    struct Entry { int up, wf, wl, rn; };
    Entry *entries = nullptr;
    float *first_part = nullptr;
    if constexpr (!UNIT) {
        __shared__ __attribute__((aligned(16))) float lds_first[kWaves * kNH * kPartialStride];
        __shared__ __attribute__((aligned(16))) Entry lds_entries[2 * kWaves];
        first_part = lds_first, entries = lds_entries;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (the older wave of a SIMD first: waves i and i + 4 are neighbours in the range)
    const int pos = !UNIT && kWaves == 8 ? (wave < 4 ? 2 * wave : 2 * wave - 7) : wave;
    _Float16 *lds = lds_all + wave * kLdsHalfs;
    _Float16 *ps = lds;                                    // [NCG][kNH][kPsH] halfs (quantized passes)

    const int lane = threadIdx.x & 63;
    const int NU = a.units * a.hsets;

    // ---------------- the work list: total weight P, this wave's range, the unit that holds its start.
    // Lane l looks at units l, l+64, ...; up to 256 units the lengths stay in registers between the two
    // steps (sum, then locate), beyond that the second step reads them again.  Units without any token
    // get their zeros here.
    auto zero_fill = [&](int uu) {
        const int u = uu >> a.hs_shift, hs = uu & (a.hsets - 1);
        const int bi = (int)fast_div((uint32_t)u, a.hkv_magic, a.hkv_shift);
        const int bq0 = bi * a.Hq + (u - bi * a.Hkv) * a.rep + hs * kNH;
        const int nh = min(kNH, a.rep - hs * kNH);
        for (int i = lane; i < nh * kD; i += 64) a.out[(size_t)bq0 * kD + i] = 0;   // the whole wave
        if (APPEND && lane == 0 && hs == 0) a.r_len_out[u] = a.r_len[u];          // (nothing was appended: see res_len)
    };
    // lengths of units base + 64k + lane, k = 0..3: all eight loads go out before any is waited for
    auto lengths4 = [&](int base, int (&T)[4], int (&R)[4]) {
        int t[4], r[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int u = min(base + 64 * k + lane, NU - 1) >> a.hs_shift;
            t[k] = a.q_len[u];
            r[k] = a.r_len[u];
        }
        asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const bool in = base + 64 * k + lane < NU;
            T[k] = in ? clampi(t[k], 0, a.Tcap) : 0;
            R[k] = in ? res_len(APPEND, a, r[k]) : 0;
        }
    };
    auto weight_of = [&](int T, int R) -> int {
        if (APPEND) R &= (1 << kAppBit) - 1;
        return (((T + kPass - 1) / kPass) << wq_log) + (((R + 63) >> 6) << wr_log);
    };
    const bool small = NU <= 256;
    int Tl[4], Rl[4], wl4[4], incl4[4];
    int P = 0;
    bool empties = false;                                  // some unit of this wave's share holds no token
    // Fused step: workgroup b files the new rows of units b, b + grid size, ... in the residual buffer (32 lanes,
    // 16 bytes each: the key row, then the value row).  Nothing in this launch reads those rows from the buffer
    // -- the residual items take them from the caller's arrays -- so the copy needs no ordering against the
    // rest; the first unit's rows are requested here and stored after the lengths below have arrived, so that
    // the wave waits once for both.  (Inside the residual item the copy cost the whole launch 4 us: whatever
    // form it took there, the item's local-memory reads and its loads lost their overlap.)
    uint4 new_piece = {0u, 0u, 0u, 0u};
    int new_row = -1;
    const int file_unit = UNIT ? (int)blockIdx.x >> a.hs_shift : (int)blockIdx.x;
    const bool files_new = UNIT ? APPEND && wave == 0 && ((int)blockIdx.x & (a.hsets - 1)) == 0 && lane < 32
                                : APPEND && wave == 0 && (int)blockIdx.x < a.units && lane < 32;
    auto new_src = [&](int u) { return reinterpret_cast<const uint4 *>((lane < 16 ? a.k_new : a.v_new) + (size_t)u * kD) + (lane & 15); };
    auto new_dst = [&](int u, int r) { return reinterpret_cast<uint4 *>(const_cast<uint16_t *>(lane < 16 ? a.Rk : a.Rv) + ((size_t)u * a.Rcap + r) * kD) + (lane & 15); };
    if (files_new) {
        new_row = a.r_len[file_unit];
        new_piece = *new_src(file_unit);
    }
    // (UNIT: only this unit's two lengths are read; the work line below does not exist.  It is guarded statement by
    // statement, not enclosed, so that the line instances are compiled from unchanged code: other arrangements of the same
    // statements ran up to 3 % slower there.)
    int unit_T = 0, unit_R = 0;
    if constexpr (UNIT) {
        unit_T = clampi(load_const_i32(a.q_len + file_unit), 0, a.Tcap);
        unit_R = res_len(APPEND, a, load_const_i32(a.r_len + file_unit));
        if (files_new && new_row >= 0 && new_row < a.Rcap) *new_dst(file_unit, new_row) = new_piece;
        if (weight_of(unit_T, unit_R) == 0) {              // (uniform in the workgroup)
            if (wave == 0) zero_fill(blockIdx.x);
            return;
        }
    }
    for (int base = 0; !UNIT && base < NU; base += 256) {
        lengths4(base, Tl, Rl);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int uu = base + 64 * k + lane;
            wl4[k] = weight_of(Tl[k], Rl[k]);
            empties |= uu < NU && wl4[k] == 0 && uu % (int)gridDim.x == (int)blockIdx.x;
            incl4[k] = wave_scan_i32(wl4[k]);
            P += __builtin_amdgcn_readlane(incl4[k], 63);
        }
    }
    if (!UNIT && files_new) {
        if (new_row >= 0 && new_row < a.Rcap) *new_dst(blockIdx.x, new_row) = new_piece;
        for (int u = blockIdx.x + gridDim.x; u < a.units; u += gridDim.x) {     // (more units than workgroups)
            const int r = a.r_len[u];
            if (r >= 0 && r < a.Rcap) *new_dst(u, r) = *new_src(u);
        }
    }
    if (!UNIT && wave == 0 && __ballot(empties)) {                               // rare: look again, one unit at a time
        for (int uu = blockIdx.x; uu < NU; uu += gridDim.x) {
            const UnitItems it = unit_items(APPEND, a, uu);
            if (it.nq + it.nr == 0) zero_fill(uu);
        }
    }
    // The weight line is cut into NW ranges, those of a workgroup together at least one residual item long (so that every
    // workgroup between the first and the last of a unit owns an item of it).  NW is a power of two so that the cuts need no
    // division.
    if (!UNIT && P == 0) return;
    const int nw_cap = max(1, min((int)gridDim.x, P >> wr_log));
    const int nw_log = 31 - __builtin_clz(nw_cap) + kWavesLog, NW = 1 << nw_log;
    if (!UNIT && (int)blockIdx.x >= NW >> kWavesLog) return;
    if (!UNIT && lane < 2) entries[2 * pos + lane].up = -1;
    // This workgroup's place on the line: its number, or, workgroups being dealt to the eight dies in turn, a numbering that
    // gives every die a contiguous eighth of the line (see by_die in launch_stream).
    const int groups_log = nw_log - kWavesLog;
    const int group = groups_log < 3 || !a.by_die ? (int)blockIdx.x : (((int)blockIdx.x & 7) << (groups_log - 3)) + ((int)blockIdx.x >> 3);
    const int w = group * kWaves + pos;
    // Waves i and i + 4 of a workgroup share a SIMD, which serves the older one first, so that one gets through its passes
    // measurably faster: it takes skew16 sixteenths of the pair's range.
    const int skew16 = kWaves == 8 && ((((2L * P) >> nw_log) * min(kSkew16, 16 - kSkew16)) >> 4) >= kWR ? kSkew16 : 8;
    const int start = UNIT ? 0 : range_start(w, P, nw_log, skew16), end = UNIT ? 1 : range_start(w + 1, P, nw_log, skew16);
    // (NW / P as a wave-uniform value in a scalar register)
    const float inv_p = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, (float)NW / (float)P)));

    // ---------------- the unit whose weight span holds position `start`
    int up = UNIT ? (int)blockIdx.x : -1;
    int ib = 0;                                            // position of the unit's first item
    int T_first = unit_T, R_first = unit_R;                // its lengths
    if (!UNIT) {
        int running = 0;
        for (int base = 0; base < NU && up < 0; base += 256) {
            if (!small) {
                lengths4(base, Tl, Rl);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    wl4[k] = weight_of(Tl[k], Rl[k]);
                    incl4[k] = wave_scan_i32(wl4[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int excl = running + incl4[k] - wl4[k];
                const bool hit = up < 0 && wl4[k] > 0 && start >= excl && start < excl + wl4[k];
                const unsigned long long mask = __ballot(hit);
                if (mask) {
                    const int src = __ffsll((long long)mask) - 1;
                    up = base + 64 * k + src;
                    ib = running + __builtin_amdgcn_readlane(incl4[k] - wl4[k], src);
                    T_first = __builtin_amdgcn_readlane(Tl[k], src);
                    R_first = __builtin_amdgcn_readlane(Rl[k], src);
                }
                running += __builtin_amdgcn_readlane(incl4[k], 63);
            }
        }
    }
    const int up_first = up;

    const int blk4 = lane >> 2, row = lane & 3;            // block of 4 lanes; row = query head this lane
                                                           // supplies as A operand
    const int gl = blk4 / BGK;                             // K group (of the pass) of this lane's tokens
    const int bbk = blk4 % BGK;                            // this lane's bin of k-steps: bbk, bbk+BGK, ...
    const int bbv = blk4 % BGV;                            // same on the V side (k-steps of 4 tokens)
    const int cg0 = lane / G;                              // channel groups of channels lane, lane+64
    const int cg1 = (lane + 64) / G;
    // Tokens 2*lane, 2*lane+1 are field j = lane & 7 of their V word.  The weights of this lane carry the
    // constant factor 2^lg = 16 * 4^-shift so that the masked V field needs no shift; the lane's running
    // sums l and oz carry the same factor and are unscaled once per unit.
    const float kscale = a.c1 * 16777216.0f;               // undo the 2^-24 of the subnormal code fields

    // A wave owns the items whose start position lies in [start, end).
    for (; up < NU && ib < end; up++) {
        // (the lengths of the first unit are already known)
        const UnitItems it = up == up_first ? make_items(APPEND, T_first, R_first) : unit_items(APPEND, a, up);
        const int wt = (it.nr << wr_log) + (it.nq << wq_log);
        if (!UNIT && wt == 0) continue;
        const int ib_next = ib + wt;
        // this wave's items of the unit (the offsets are clamped to the unit's span first, so 32-bit
        // arithmetic suffices): front residual items f0..f1-1, passes j0..j1-1, back residual items b0..b1-1
        const int nf = (it.nr + 1) >> 1, nb = it.nr >> 1;
        const int span = wt + kWR;
        const int ds = min(span, max(0, start - ib)), de = min(span, max(0, end - ib));
        const int dq = nf << wr_log, db = dq + (it.nq << wq_log);
        // UNIT: a wave at the end of the row for each residual item (half of the waves at most), which therefore has no part in
        // the first round of passes; the later rounds go to all.
        const int with_res = UNIT ? min(it.nr, kWaves / 2) : 0, np = kWaves - with_res;
        const int f0 = min(nf, (ds + kWR - 1) >> wr_log), f1 = min(nf, (de + kWR - 1) >> wr_log);
        const int j0 = UNIT ? (wave < np ? wave : np + wave) : min(it.nq, (max(0, ds - dq) + kWQ - 1) >> wq_log);
        const int j1 = UNIT ? it.nq : min(it.nq, (max(0, de - dq) + kWQ - 1) >> wq_log);
        const int b0 = min(nb, (max(0, ds - db) + kWR - 1) >> wr_log), b1 = min(nb, (max(0, de - db) + kWR - 1) >> wr_log);
        if (!UNIT && f0 >= f1 && j0 >= j1 && b0 >= b1) { ib = ib_next; continue; }
        const int u = up >> a.hs_shift, hs = up & (a.hsets - 1);
        const int bi = (int)fast_div((uint32_t)u, a.hkv_magic, a.hkv_shift);
        const int bq0 = bi * a.Hq + (u - bi * a.Hkv) * a.rep + hs * kNH;
        const int nheads = min(kNH, a.rep - hs * kNH);
        const int t_end = it.T;
        const bool ends_here = ib_next >= end;             // (the wave's last unit)
        const uint32_t *Kc = a.Kc + (size_t)u * kc_words(a.Tcap);
        const uint32_t *Vc = a.Vc + (size_t)u * vc_words(a.Tcap);
        const uint16_t *Ks = a.Ks + (size_t)u * (a.Tcap / G) * kD;
        const uint16_t *Kz = a.Kz + (size_t)u * (a.Tcap / G) * kD;
        const uint16_t *Vs = a.Vs + (size_t)u * a.Tcap * NCG;
        const uint16_t *Vz = a.Vz + (size_t)u * a.Tcap * NCG;

        int lane_u = lane;
        asm volatile("" : "+v"(lane_u));                   // (opaque copy: per-lane load offsets are set up per unit)
        const int bbk_u = (lane_u >> 2) % BGK;
        // Loaders of one pass's tiles, in the pieces the phases consume them in (each piece is requested again,
        // for the wave's next pass, as soon as its registers have been read for the last time: every piece is
        // then in flight for about a whole pass, which is what keeps enough bytes outstanding per wave).
        auto load_k_meta = [&](KD &d, int tp) {
            const bool gvalid = tp + gl * G < t_end;
            const size_t go = ((size_t)(tp / G) + (gvalid ? gl : 0)) * kD + bbk_u * (NKR * 4);
            d.ks = load_words<NKW>(Ks + go);
            d.kz = load_words<NKW>(Kz + go);
        };
        auto words = [](const u4 *p) -> u4 {
            if constexpr (STREAM) return __builtin_nontemporal_load(p);
            return *p;
        };
        auto load_k_codes = [&](KD &d, int tp, int half, bool last = false) {   // half 0: words 0..3 of both tokens, 1: words 4..7
            const u4 *ktile = reinterpret_cast<const u4 *>(kOneTile && last ? a.Kc : Kc + (size_t)(tp >> 7) * 1024);
            d.kw[half] = words(ktile + half * 64 + lane_u);
            d.kw[2 + half] = words(ktile + (2 + half) * 64 + lane_u);
        };
        auto load_v_meta = [&](VD &d, int tp) {
            // past the end the (clamped) load still happens (the weights of those tokens are zero), so that the
            // number of loads in flight is the same on every path
            const bool valid = tp + 2 * lane_u < t_end;
            const size_t vo = (size_t)(valid ? tp + 2 * lane_u : tp) * NCG;
            d.vs = load_words<NCG>(Vs + vo);
            d.vz = load_words<NCG>(Vz + vo);
        };
        auto load_v_codes = [&](VD &d, int tp, int tl, bool last = false) {     // tl: 64-token tile of the pass
            const u4 *vtile = reinterpret_cast<const u4 *>(kOneTile && last ? a.Vc : Vc + (size_t)(tp >> 6) * (4 * kD));
            d.vw[0][tl] = words(vtile + tl * kD + lane_u);
            d.vw[1][tl] = words(vtile + tl * kD + lane_u + 64);
        };
        auto load_k = [&](int tp) -> KD {
            KD d;
            load_k_codes(d, tp, 0);
            load_k_codes(d, tp, 1);
            load_k_meta(d, tp);
            return d;
        };
        auto load_v = [&](int tp) -> VD {
            VD d;
            load_v_codes(d, tp, 0);
            load_v_codes(d, tp, 1);
            load_v_meta(d, tp);
            return d;
        };

        // Operand ranges.  The A operands of both products are fp16: q*Ks*4^-j on the K side and p*Vs*2^lg on
        // the V side (p <= 1, 2^lg <= 2^hd).  The first attempt uses the scalings that keep the most precision
        // (q as it is, hd = 4); they hold as long as |q*Ks| < 65504 and Vs < 4096.  Beyond that an operand
        // overflows to infinity, which ends up in the wave's sums: an infinite q*Ks meets a code 0 in its group
        // (every group with a non-zero scale has one), the product is NaN, so is that token's weight, and the sum
        // of weights keeps it; an infinite p*Vs makes the output sums infinite or NaN.  The sums are checked once
        // per unit, and if one is not finite the wave does its items of the unit again with q scaled per head to
        // below 1 and hd = -1: then |A| <= max Ks, max Vs / 2 <= 43669 whatever the inputs (the largest fp16
        // scale is (65504 + 65504) / 3).  No cost for data inside the range; outside it the result keeps fewer
        // bits of the small weights.
        float m[kNH], lsum[kNH];                           // running max; sum of weights (wave-uniform at the end)
        float oa[kNH], ob[kNH];                            // un-normalised output of channels lane, lane+64
#pragma nounroll
        for (int attempt = 0; attempt < 2; attempt++) {
        const bool safe = attempt != 0;
        if (safe && lane == 0) atomicAdd(a.redo, 1);       // (diagnostics: how often the second attempt is taken)
        const float hd = safe ? -1.0f : 4.0f;
        const float lg = hd - (float)fld_shift(lane & 7);
        const float vun = safe ? 33554432.0f : 1048576.0f; // 2^24 (subnormal fields) / 2^hd (ps headroom)
        const float inv_vun = 1.0f / vun;
        // This lane's query values for the quantized passes (head `row`, the channels of its k-steps).
        h2 qraw[NKR][2];
        auto load_q = [&]() {
#pragma unroll
            for (int i = 0; i < NKR; i++) {
                const int c = 4 * (bbk_u + BGK * i);
                uint2 bits = {0u, 0u};
                const int hq = PAIRED ? (lane_u & 3) >> 1 : (lane_u & 3);   // the head whose A rows this lane supplies
                if (hq < nheads && j0 < j1) bits = *reinterpret_cast<const uint2 *>(a.q + (size_t)(bq0 + hq) * kD + c);
                qraw[i][0] = as_h2(bits.x);
                qraw[i][1] = as_h2(bits.y);
            }
        };
        // The tiles of the first pass are requested before anything else is waited for; without residual items
        // in front the query values go first (they are needed first, and a wait for them then does not wait
        // for the tiles), with residual items they are fetched afterwards (fewer registers live in between).
        const bool front = !UNIT && f0 < f1;               // (UNIT: all residual items after the passes)
        KD kd = {};
        VD vd = {};
        if (!front) load_q();
        if (j0 < j1) {
            kd = load_k(j0 * kPass);
            vd = load_v(j0 * kPass);
        }
        // the wave's online-softmax state for this unit
        float l_lane[kNH];
        f4 O0 = {0.f, 0.f, 0.f, 0.f}, O1 = {0.f, 0.f, 0.f, 0.f};   // channel lane / lane+64, 4 heads each
        float oz[kNH][NCG];
#pragma unroll
        for (int h = 0; h < kNH; h++) {
            m[h] = -1e30f; l_lane[h] = 0.f;
#pragma unroll
            for (int g = 0; g < NCG; g++) oz[h][g] = 0.f;
        }

        // =============================== residual items (64 fp16 tokens each): Algorithm 1's R_K t_Q^T and
        // A_unquant R_V, on the same 4x4x4 matrix instruction as the quantized passes (the vector ALU is
        // several times slower here because the wave shares its SIMD with one that saturates the matrix
        // pipe).  The 64 key rows, then the 64 value rows, are fetched with fully coalesced loads (4 rows
        // per instruction, 16 lanes x 16 B per row) and staged in LDS.  Scores: lane = token, its key row
        // read back as the B operand, q as the A operand broadcast to all 16 blocks.  Values: lane =
        // channels lane, lane+64, the B operand gathered token by token from the staged rows, the weights
        // p (fp16, through LDS) as the broadcast A operand.  The result is folded into the wave's state.
        auto residual_items = [&](int first, int end_item, int step) {
#pragma unroll 1
        for (int ri = first; ri < end_item; ri += step) {
            const int R = it.R;
            _Float16 *pr = lds;                            // [kNH][kPrH] halfs: weights of the item's tokens
            _Float16 *rows = lds + kPrHalfs;               // [64][kKRowH] halfs: key rows, then value rows
            const uint16_t *Rk = a.Rk + (size_t)u * a.Rcap * kD, *Rv = a.Rv + (size_t)u * a.Rcap * kD;
            int lane_r = lane;                             // (opaque copy: keeps the address terms below out of
            asm volatile("" : "+v"(lane_r));               //  the registers that live across the pass loop)
            const int rsub = lane_r >> 4, piece = lane_r & 15;  // row within a group of 4, 16-byte piece of the row
            const int t0 = ri * 64;
            const bool valid = t0 + lane < R;

            // (fused step: the unit's last residual row is the token this launch appends; it is read from the
            // caller's new rows, never from the residual buffer, where another wave files it at some point of
            // this launch)
            const int r_new = it.rn;                       // (a full or invalid buffer takes no token)
            const uint16_t *kn = APPEND ? a.k_new + (size_t)u * kD : nullptr, *vn = APPEND ? a.v_new + (size_t)u * kD : nullptr;
            // (an empty buffer: its row 0, which stands in for the rows past the end, may hold anything, NaN included, and is being
            // written by the wave that files the new token; the new token's row stands in for them)
            if (APPEND && r_new == 0) Rk = kn, Rv = vn;
            // (the rows are loaded as in the plain call; the item that holds the new row then loads it once more, from the
            // caller's array.  UNIT: 16 bytes a lane, put over the row the buffer gave once the rows are in local memory, 12 to 45
            // registers less.  The work line, whose tiles are in flight meanwhile, has none for it: into the registers of the
            // four-row step the row belongs to, one wave-uniform branch per step instead of a select per row.)
            const bool has_new = APPEND && r_new >= t0 && r_new < t0 + 64;     // (uniform)
            const int new_step = (r_new - t0) >> 2, new_sub = (r_new - t0) & 3;
            uint4 fresh = {0u, 0u, 0u, 0u};
            auto request_new = [&](Words<64> &g, const uint16_t *row) __attribute__((always_inline)) {
                if (!has_new) return;
                if (UNIT) {
                    fresh = reinterpret_cast<const uint4 *>(row)[piece];
                    return;
                }
#pragma unroll
                for (int i = 0; i < 16; i++)
                    if (i == new_step && rsub == new_sub) {
                        const uint4 x = reinterpret_cast<const uint4 *>(row)[piece];
                        g.v[4 * i] = x.x; g.v[4 * i + 1] = x.y; g.v[4 * i + 2] = x.z; g.v[4 * i + 3] = x.w;
                    }
            };
            auto put_new = [&]() {
                if (UNIT && has_new && lane_r < 16) *reinterpret_cast<uint4 *>(rows + (r_new - t0) * kKRowH + piece * 8) = fresh;
            };
            Words<64> g;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const int rr = t0 + 4 * i + rsub;
                const uint16_t *src = Rk + (size_t)(rr < R ? rr : 0) * kD;
                const uint4 x = reinterpret_cast<const uint4 *>(src)[piece];
                g.v[4 * i] = x.x; g.v[4 * i + 1] = x.y; g.v[4 * i + 2] = x.z; g.v[4 * i + 3] = x.w;
            }
            request_new(g, kn);
            // A operands of the scores: block b supplies k-steps b and b+16 (channels 4b.., 64+4b..) of head `row`
            h4 qa[2];
#pragma unroll
            for (int i = 0; i < 2; i++) {
                uint2 bits = {0u, 0u};
                if ((lane_r & 3) < nheads) bits = *reinterpret_cast<const uint2 *>(a.q + (size_t)(bq0 + (lane_r & 3)) * kD + 4 * ((lane_r >> 2) + 16 * i));
                const h2 lo = as_h2(bits.x), hi = as_h2(bits.y);
                qa[i] = h4{lo[0], lo[1], hi[0], hi[1]};
            }
#pragma unroll
            for (int i = 0; i < 16; i++)
                *reinterpret_cast<uint4 *>(rows + (4 * i + rsub) * kKRowH + piece * 8) =
                    uint4{g.v[4 * i], g.v[4 * i + 1], g.v[4 * i + 2], g.v[4 * i + 3]};
            put_new();
            // the value rows are requested now and travel while the scores are computed
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const int rr = t0 + 4 * i + rsub;
                const uint16_t *src = Rv + (size_t)(rr < R ? rr : 0) * kD;
                const uint4 x = reinterpret_cast<const uint4 *>(src)[piece];
                g.v[4 * i] = x.x; g.v[4 * i + 1] = x.y; g.v[4 * i + 2] = x.z; g.v[4 * i + 3] = x.w;
            }
            request_new(g, vn);
            __builtin_amdgcn_wave_barrier();

            f4 sc = {0.f, 0.f, 0.f, 0.f};                  // scores of token t0 + lane for the 4 heads
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const u4 kk = *reinterpret_cast<const u4 *>(rows + lane * kKRowH + i * 8);   // channels 8i..8i+7
                const h2 k0 = as_h2(kk[0]), k1 = as_h2(kk[1]), k2 = as_h2(kk[2]), k3 = as_h2(kk[3]);
                mfma_bc<4>(sc, qa[(2 * i) / 16], h4{k0[0], k0[1], k1[0], k1[1]}, (2 * i) % 16);
                mfma_bc<4>(sc, qa[(2 * i + 1) / 16], h4{k2[0], k2[1], k3[0], k3[1]}, (2 * i + 1) % 16);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 16; i++)
                *reinterpret_cast<uint4 *>(rows + (4 * i + rsub) * kKRowH + piece * 8) =
                    uint4{g.v[4 * i], g.v[4 * i + 1], g.v[4 * i + 2], g.v[4 * i + 3]};
            put_new();

            // softmax update against the wave's state
            float s[kNH], mn[kNH];
            bool grow = false;
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                s[h] = valid ? sc[h] * a.c1 : -INFINITY;
                mn[h] = s[h];
            }
            wave_max64x4(mn);
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                mn[h] = fmaxf(m[h], mn[h]);
                grow |= mn[h] > m[h];
            }
            if (grow) {                                    // wave-uniform
#pragma unroll
                for (int h = 0; h < kNH; h++) {
                    const float so = fast_exp2(m[h] - mn[h]);
                    l_lane[h] *= so;
                    O0[h] *= so;
                    O1[h] *= so;
#pragma unroll
                    for (int gq = 0; gq < NCG; gq++) oz[h][gq] *= so;
                    m[h] = mn[h];
                }
            }
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                const float p = fast_exp2(s[h] - m[h]);    // 0 past the end
                l_lane[h] += p * fast_exp2(lg);            // the lane sums carry the factor 2^lg
                pr[h * kPrH + lane] = (_Float16)p;
            }
            __builtin_amdgcn_wave_barrier();

            // values: 16 k-steps of 4 tokens; block b supplies the weights of k-step b
            const h4 pa = *reinterpret_cast<const h4 *>(pr + row * kPrH + 4 * blk4);
            f4 R0 = {0.f, 0.f, 0.f, 0.f}, R1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 16; ks++) {
                const _Float16 *v = rows + (4 * ks) * kKRowH + lane;
                const h4 b0 = {v[0], v[kKRowH], v[2 * kKRowH], v[3 * kKRowH]};
                const h4 b1 = {v[64], v[kKRowH + 64], v[2 * kKRowH + 64], v[3 * kKRowH + 64]};
                mfma_bc<4>(R0, pa, b0, ks);
                mfma_bc<4>(R1, pa, b1, ks);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                O0[h] += R0[h] * inv_vun;                  // the state's outputs carry the factor 1/vun
                O1[h] += R1[h] * inv_vun;
            }
        }
        };
        if (front) {
            residual_items(2 * f0, 2 * f1, 2);             // (even items sit before the passes, odd ones after)
            load_q();
        }
        {
        // =============================== quantized passes
            // the query values pre-scaled by the 4^-j of the code field (channel pair (c, c+1), c even, is field
            // (c % 16) / 2 of its K word)
            h2 qscl[NKR][2];
            // qf: the power of two this lane's head is scaled by (1 on the first attempt; on the second
            // 2^(14 - E) with E the biased exponent of the head's largest |q|, so that |q| * qf < 1)
            float qf = 1.0f;
            if (safe) {
                typedef unsigned short us2 __attribute__((ext_vector_type(2)));
                us2 mx2 = {0, 0};
#pragma unroll
                for (int i = 0; i < NKR; i++)
#pragma unroll
                    for (int ep = 0; ep < 2; ep++)
                        mx2 = __builtin_elementwise_max(mx2, __builtin_bit_cast(us2, as_u32(qraw[i][ep]) & 0x7fff7fffu));
                int mx = max((int)mx2[0], (int)mx2[1]);
                for (int d = 4; d < 64; d <<= 1) mx = max(mx, __shfl_xor(mx, d));   // lanes with the same `row`
                qf = fast_exp2(14.0f - (float)min(mx >> 10, 30));
            }
            float ksc[kNH];                                // kscale / qf of head h (wave-uniform)
#pragma unroll
            for (int h = 0; h < NHQ; h++) {
                const float f = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, qf), PAIRED ? 2 * h : h));
                ksc[h] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, kscale / f)));
            }
#pragma unroll
            for (int i = 0; i < NKR; i++) {
                const int c = 4 * (bbk + BGK * i);
#pragma unroll
                for (int ep = 0; ep < 2; ep++)
                    qscl[i][ep] = qraw[i][ep] * (_Float16)(fld_scale(((c + 2 * ep) & 15) >> 1) * qf);
            }

            float s0[kNH], s1[kNH];                        // scores of the lane's two tokens (NHQ heads)

            // ---------------- K phase: scores of tokens 2*lane, 2*lane+1 for the 4 heads
            auto k_phase = [&](KD &d, int tp, int t2, bool last) {        // t2: the pass whose tiles are requested meanwhile
                const bool valid = tp + 2 * lane < t_end;  // both tokens of the lane (t_end % 16 == 0)
                // A operands of this lane's k-steps (exact hi + lo split of q * Ks), qz = sum_c q_c Kz[g,c]
                h4 a_hi[NKR], a_lo[NKR];
                float qz = 0.f;
#pragma unroll
                for (int i = 0; i < NKR; i++) {
                    h2 hi[2], lo[2];
#pragma unroll
                    for (int ep = 0; ep < 2; ep++) {
                        const h2 ks2 = as_h2(d.ks.v[2 * i + ep]), kz2 = as_h2(d.kz.v[2 * i + ep]);
                        hi[ep] = qscl[i][ep] * ks2;
                        if constexpr (LO) lo[ep] = __builtin_elementwise_fma(qscl[i][ep], ks2, -hi[ep]);
                        qz = __builtin_amdgcn_fdot2(qraw[i][ep], kz2, qz, false);
                    }
                    if constexpr (PAIRED) {                 // odd rows carry the lo part
                        const h2 u0 = (row & 1) ? lo[0] : hi[0], u1 = (row & 1) ? lo[1] : hi[1];
                        a_hi[i] = h4{u0[0], u0[1], u1[0], u1[1]};
                    } else {
                        a_hi[i] = h4{hi[0][0], hi[0][1], hi[1][0], hi[1][1]};
                        if constexpr (LO) a_lo[i] = h4{lo[0][0], lo[0][1], lo[1][0], lo[1][1]};
                    }
                }
                __builtin_amdgcn_sched_barrier(0);         // (all A operands first: the rows are then free)
                load_k_meta(d, t2);                        // the scale / zero rows have been consumed
                __builtin_amdgcn_sched_barrier(0);
                // sum the partial qz of the BGK blocks of the group (same row, lanes 4 apart)
                if constexpr (BGK == 2) qz += __shfl_xor(qz, 4);
                if constexpr (BGK >= 4) { qz = dpp_ror_add<4>(qz); qz = dpp_ror_add<8>(qz); }
                if constexpr (BGK >= 8) qz += __shfl_xor(qz, 16);
                if constexpr (BGK >= 16) qz += __shfl_xor(qz, 32);

                f4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int wd = 0; wd < 8; wd++) {
                    const uint32_t w0 = d.kw[wd >> 2][wd & 3], w1 = d.kw[2 + (wd >> 2)][wd & 3];
                    const uint32_t w0s = w0 >> 6, w1s = w1 >> 6;
#pragma unroll
                    for (int sq = 0; sq < 4; sq++) {
                        const int s = 4 * wd + sq;         // k-step: channels 4s..4s+3
                        const h2 x00 = field(w0, w0s, 2 * sq), x01 = field(w0, w0s, 2 * sq + 1);
                        const h2 x10 = field(w1, w1s, 2 * sq), x11 = field(w1, w1s, 2 * sq + 1);
                        const h4 b0 = {x00[0], x00[1], x01[0], x01[1]};
                        const h4 b1 = {x10[0], x10[1], x11[0], x11[1]};
                        mfma_k<CBK>(acc0, acc1, a_hi[s / BGK], b0, b1, s % BGK);
                        if constexpr (LO && !PAIRED) mfma_k<CBK>(acc0, acc1, a_lo[s / BGK], b0, b1, s % BGK);
                    }
                    if (wd == 3) {                         // words 0..3 are done
                        __builtin_amdgcn_sched_barrier(0);
                        load_k_codes(d, t2, 0, last);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                load_k_codes(d, t2, 1, last);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (PAIRED) {
                    const float zz[2] = {quad_bcast<0>(qz) * a.c1, quad_bcast<2>(qz) * a.c1};
#pragma unroll
                    for (int h = 0; h < 2; h++) {
                        s0[h] = valid ? (acc0[2 * h] + acc0[2 * h + 1]) * ksc[h] + zz[h] : -INFINITY;
                        s1[h] = valid ? (acc1[2 * h] + acc1[2 * h + 1]) * ksc[h] + zz[h] : -INFINITY;
                    }
                } else {
                    const float zz[kNH] = {quad_bcast<0>(qz) * a.c1, quad_bcast<1>(qz) * a.c1,
                                           quad_bcast<2>(qz) * a.c1, quad_bcast<3>(qz) * a.c1};
#pragma unroll
                    for (int h = 0; h < kNH; h++) {
                        s0[h] = valid ? acc0[h] * ksc[h] + zz[h] : -INFINITY;
                        s1[h] = valid ? acc1[h] * ksc[h] + zz[h] : -INFINITY;
                    }
                }
            };

            // ---------------- softmax update, ps table, V products
            auto v_phase = [&](VD &d, int tp, int t2, bool last) {
                const bool valid = tp + 2 * lane < t_end;
                float mn[kNH];
                bool grow = false;
#pragma unroll
                for (int h = 0; h < NHQ; h++) mn[h] = fmaxf(s0[h], s1[h]);
                if constexpr (PAIRED) wave_max64x2(mn); else wave_max64x4(mn);
#pragma unroll
                for (int h = 0; h < NHQ; h++) {
                    mn[h] = fmaxf(m[h], mn[h]);
                    grow |= mn[h] > m[h];
                }
                if (grow) {                                // wave-uniform
#pragma unroll
                    for (int h = 0; h < NHQ; h++) {
                        const float sc = fast_exp2(m[h] - mn[h]);
                        l_lane[h] *= sc;
                        O0[h] *= sc;
                        O1[h] *= sc;
#pragma unroll
                        for (int g = 0; g < NCG; g++) oz[h][g] *= sc;
                        m[h] = mn[h];
                    }
                }
                {
                    // (vs, vz) words hold [token 2l: NCG halfs][token 2l+1: NCG halfs]; pair them per group
                    h2 vsp[NCG], vzp[NCG];
#pragma unroll
                    for (int g = 0; g < NCG; g++) {
                        const int i0 = g, i1 = NCG + g;    // half index of (token 0, g) and (token 1, g)
                        const uint32_t sel = ((i0 & 1) ? 0x00000302u : 0x00000100u) | ((i1 & 1) ? 0x07060000u : 0x05040000u);
                        const uint32_t sv = __builtin_amdgcn_perm(d.vs.v[i1 >> 1], d.vs.v[i0 >> 1], sel);
                        const uint32_t zv = __builtin_amdgcn_perm(d.vz.v[i1 >> 1], d.vz.v[i0 >> 1], sel);
                        vsp[g] = as_h2(valid ? sv : 0u);
                        vzp[g] = as_h2(valid ? zv : 0u);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    load_v_meta(d, t2);                    // the scales and zero-points have been consumed
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int h = 0; h < NHQ; h++) {
                        const float mo = m[h] - lg;
                        const float p0 = fast_exp2(s0[h] - mo), p1 = fast_exp2(s1[h] - mo);   // masked: 0
                        l_lane[h] += p0 + p1;
                        const h2 ph = {(_Float16)p0, (_Float16)p1};
#pragma unroll
                        for (int g = 0; g < NCG; g++) {
                            *reinterpret_cast<h2 *>(ps + g * kPsG + h * kPsH + 2 * lane) = ph * vsp[g];
                            oz[h][g] = __builtin_amdgcn_fdot2(ph, vzp[g], oz[h][g], false);
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();

                // A operands of this lane's V k-steps (4 tokens each): ps[channel group][head row][tokens]
                h4 a0[NVR], a1[NVR];
#pragma unroll
                for (int i = 0; i < NVR; i++) {
                    const int tok = 4 * (bbv + BGV * i);
                    a0[i] = *reinterpret_cast<const h4 *>(ps + cg0 * kPsG + row * kPsH + tok);
                    a1[i] = *reinterpret_cast<const h4 *>(ps + cg1 * kPsG + row * kPsH + tok);
                }
#pragma unroll
                for (int blk = 0; blk < 8; blk++) {
                    const uint32_t v0 = d.vw[0][blk >> 2][blk & 3], v1 = d.vw[1][blk >> 2][blk & 3];
                    const uint32_t v0s = v0 >> 6, v1s = v1 >> 6;
#pragma unroll
                    for (int kq = 0; kq < 4; kq++) {
                        const int ks = 4 * blk + kq;       // k-step: tokens 4ks..4ks+3 of the pass
                        const h2 x00 = field(v0, v0s, 2 * kq), x01 = field(v0, v0s, 2 * kq + 1);
                        const h2 x10 = field(v1, v1s, 2 * kq), x11 = field(v1, v1s, 2 * kq + 1);
                        const h4 b0 = {x00[0], x00[1], x01[0], x01[1]};
                        const h4 b1 = {x10[0], x10[1], x11[0], x11[1]};
                        mfma_v<CBV>(O0, O1, a0[ks / BGV], a1[ks / BGV], b0, b1, ks % BGV);
                    }
                    if (blk == 3) {                        // the first 64-token tile is done
                        __builtin_amdgcn_sched_barrier(0);
                        load_v_codes(d, t2, 0, last);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                load_v_codes(d, t2, 1, last);
                __builtin_amdgcn_wave_barrier();
            };

            // Every piece of a pass's tiles is requested for the next pass right after its last use and is
            // issued on every path (the last pass requests tiles again, nobody uses them: see kOneTile), so the
            // number in flight is always the same.
            for (int jj = j0, next; jj < j1; jj = next) {
                next = UNIT ? jj + (jj < np ? np : kWaves) : jj + 1;
                const int tp = jj * kPass;
                const bool last = next >= j1;
                const int t2 = (last ? jj : next) * kPass;
                k_phase(kd, tp, t2, last);
                v_phase(vd, tp, t2, last);
            }
        }
        if (UNIT) residual_items(kWaves - 1 - wave, wave >= np ? it.nr : 0, kWaves / 2);
        else residual_items(2 * b0 + 1, 2 * b1 + 1, 2);

        {
            // finish: undo operand scalings, add the zero-point term
            const float unlg = fast_exp2(-lg);
#pragma unroll
            for (int h = 0; h < kNH; h++) lsum[h] = l_lane[h] * unlg;
            wave_sum64x4(lsum);
#pragma unroll
            for (int g = 0; g < NCG; g++) {
                float zs[kNH];
#pragma unroll
                for (int h = 0; h < kNH; h++) zs[h] = oz[h][g] * unlg;
                wave_sum64x4(zs);
#pragma unroll
                for (int h = 0; h < kNH; h++) oz[h][g] = zs[h];    // now the wave total (uniform)
            }
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                float z0 = 0.f, z1 = 0.f;
#pragma unroll
                for (int g = 0; g < NCG; g++) {
                    z0 = (g == cg0) ? oz[h][g] : z0;
                    z1 = (g == cg1) ? oz[h][g] : z1;
                }
                oa[h] = O0[h] * vun + z0;
                ob[h] = O1[h] * vun + z1;
            }
        }
        {
            // any overflowed operand has left an infinity or a NaN in one of the sums (of the heads in use:
            // with paired rows the accumulators of rows 2 and 3 hold nothing meaningful)
            float chk = 0.f;
#pragma unroll
            for (int h = 0; h < NHQ; h++) chk += (O0[h] + O1[h]) + l_lane[h];
            if (__ballot(!(chk - chk == 0.f)) == 0) break;
        }
        }   // attempt

        // =============================== publish this wave's partial of the unit
        int lane_p = lane;
        asm volatile("" : "+v"(lane_p));                   // (opaque copy: address terms computed here, not hoisted)
        // the waves that own items of this unit: from the owner of the first item to the owner of the last
        const int wf = UNIT ? 0 : wave_of(ib, P, nw_log, inv_p, skew16);
        const int wl = UNIT ? 0 : wave_of(ib_next - (nb ? kWR : it.nq ? kWQ : kWR), P, nw_log, inv_p, skew16);
        // (fused step: the unit's residual length after the append, for the next call -- into an array of its own,
        // because every wave of THIS launch still reads the old lengths when it starts; written by the wave that
        // writes the unit's output)
        auto write_next_len = [&]() {
            if (APPEND && lane == 0) a.r_len_out[u] = it.rn >= 0 ? it.rn + 1 : a.r_len[u];
        };
        if constexpr (UNIT) {
            // every wave's state goes to its own part of the local memory; then a thread per (head, channel) merges them
            // in wave order (a wave without items left m = -1e30, weight 0)
            constexpr int NWV = kWaves;
            float *mine = reinterpret_cast<float *>(lds);
            asm volatile("" ::: "memory");                 // (the same bytes held weights and rows, as other types)
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                mine[h * kPartialStride + 4 + lane] = oa[h];
                mine[h * kPartialStride + 4 + lane + 64] = ob[h];
                if (lane == 0) mine[h * kPartialStride] = m[h], mine[h * kPartialStride + 1] = lsum[h];
            }
            __syncthreads();
            if (wave == 0) write_next_len();
            for (int i = wave * 64 + lane_p; i < nheads * kD; i += 64 * NWV) {
                const int h = i / kD, c = i % kD;
                const float *part = reinterpret_cast<const float *>(lds_all) + h * kPartialStride;
                constexpr size_t step = kLdsHalfs / 2;
                float M = part[0];
#pragma unroll
                for (int k = 1; k < NWV; k++) M = fmaxf(M, part[k * step]);
                float L = 0.f, O = 0.f;
#pragma unroll
                for (int k = 0; k < NWV; k++) {
                    const float e = fast_exp2(part[k * step] - M);
                    L = __builtin_fmaf(part[k * step + 1], e, L);
                    O = __builtin_fmaf(part[k * step + 4 + c], e, O);
                }
                a.out[(size_t)(bq0 + h) * kD + c] = __half_as_ushort(__float2half_rn(L > 0.f ? O / L : 0.f));
            }
        } else if (wf != wl) {
            // (the last one into the memory the wave worked in, the first one must outlive the wave's next unit)
            float *part = ends_here ? reinterpret_cast<float *>(lds) : first_part + wave * (kNH * kPartialStride);
            asm volatile("" ::: "memory");                 // (the same bytes held weights and rows, as other types)
#pragma unroll
            for (int h = 0; h < NHQ; h++) {
                part[h * kPartialStride + 4 + lane_p] = oa[h];
                part[h * kPartialStride + 4 + lane_p + 64] = ob[h];
                if (lane == 0) part[h * kPartialStride] = m[h], part[h * kPartialStride + 1] = lsum[h];
            }
            if (lane == 0) entries[2 * pos + ends_here] = Entry{up, wf >> kWavesLog, wl >> kWavesLog, it.rn};
        } else {
            // the only partial of its unit: normalise and write the result directly
            write_next_len();
#pragma unroll
            for (int h = 0; h < kNH; h++) {
                if (h < nheads) {
                    const float inv = lsum[h] > 0.f ? 1.0f / lsum[h] : 0.f;
                    a.out[(size_t)(bq0 + h) * kD + lane_p] = __half_as_ushort(__float2half_rn(oa[h] * inv));
                    a.out[(size_t)(bq0 + h) * kD + lane_p + 64] = __half_as_ushort(__float2half_rn(ob[h] * inv));
                }
            }
        }
        if constexpr (UNIT) break;
        ib = ib_next;
    }
    if constexpr (!UNIT) {
        // =============================== the workgroup's partials: a wave per unit merges the entries of the unit in local
        // memory, and, if other workgroups have items of the unit as well, publishes the result and takes a ticket
        // (the arguments once more from memory: held over the passes they would not fit the scalar registers)
        auto b = (const __attribute__((address_space(4))) DecArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(b));
        // split-K partial of (slot, head): [0] running max (base-2 domain), [1] sum of weights, [4..131] output
        auto slot_of = [&](int slot, int h) -> float * { return b->ws + ((size_t)slot * kNH + h) * kPartialStride; };
        __syncthreads();
        constexpr int NE = 2 * kWaves, NJ = NHQ / 2;       // (NJ: pairs of heads in use)
        constexpr int kSlotB = kNH * kPartialStride * 4, kHeadB = kPartialStride * 4, kSc1 = 16;  // (cache policy: device scope)
        typedef unsigned int u4v __attribute__((ext_vector_type(4)));
        const int half_p = lane >> 5, c4 = lane & 31;      // a lane holds channels 4 c4 .. 4 c4 + 3 of heads half_p and 2 + half_p
        const unsigned lane_off = (unsigned)(half_p * kHeadB + 16 + c4 * 16);
        const Entry mine = entries[min(lane, NE - 1)];
        const int up_e = lane < NE ? mine.up : -1;
        auto part_of = [&](int e) -> const float * {
            const int p = e >> 1, wv = kWaves == 8 ? (p >> 1) + (p & 1) * 4 : p;
            return e & 1 ? reinterpret_cast<const float *>(lds_all + wv * kLdsHalfs) : first_part + wv * (kNH * kPartialStride);
        };
        unsigned long long left = __ballot(up_e >= 0);
        for (int seg = 0; left != 0; seg++) {
            const int head = __ffsll((long long)left) - 1, up = __builtin_amdgcn_readlane(up_e, head);
            unsigned long long same = __ballot(up_e == up);
            left &= ~same;
            if ((seg & (kWaves - 1)) != wave) continue;
            const int gf = __builtin_amdgcn_readlane(mine.wf, head), gl = __builtin_amdgcn_readlane(mine.wl, head);
            const int rn = __builtin_amdgcn_readlane(mine.rn, head);
            const int u = up >> b->hs_shift, hs = up & (b->hsets - 1);
            const int bi = (int)fast_div((uint32_t)u, b->hkv_magic, b->hkv_shift);
            const int bq0 = bi * b->Hq + (u - bi * b->Hkv) * b->rep + hs * kNH;
            const int nheads = min(kNH, b->rep - hs * kNH);

            float M[kNH], L[kNH];
            f4 Oq[NJ];
#pragma unroll
            for (int h = 0; h < kNH; h++) { M[h] = -1e30f; L[h] = 0.f; }
#pragma unroll
            for (int j = 0; j < NJ; j++) Oq[j] = f4{0.f, 0.f, 0.f, 0.f};
            // adds `n` partials to (M, L, Oq): lane k holds (max, sum) of partial k, x their outputs
            auto fold = [&](float (&ms)[kNH], float (&ls)[kNH], auto &x, auto n) __attribute__((always_inline)) {
                float cm[kNH], wgt[kNH], lw[kNH], so2[2] = {0.f, 0.f};
#pragma unroll
                for (int h = 0; h < kNH; h++) cm[h] = ms[h];
                if constexpr (PAIRED) wave_max64x2(cm); else wave_max64x4(cm);
#pragma unroll
                for (int h = 0; h < NHQ; h++) {
                    const float Mn = fmaxf(M[h], cm[h]), so = fast_exp2(M[h] - Mn);
                    wgt[h] = fast_exp2(ms[h] - Mn);        // exactly 0 for ms = -1e30
                    lw[h] = ls[h] * wgt[h];
                    L[h] *= so;
                    if ((h & 1) == 0) so2[h >> 1] = so; else so2[h >> 1] = half_p ? so : so2[h >> 1];
                    M[h] = Mn;
                }
                if constexpr (PAIRED) lw[2] = lw[3] = 0.f;
                wave_sum64x4(lw);
#pragma unroll
                for (int h = 0; h < NHQ; h++) L[h] += lw[h];
#pragma unroll
                for (int j = 0; j < NJ; j++) Oq[j] *= so2[j];
#pragma unroll
                for (int k = 0; k < decltype(n)::value; k++)
#pragma unroll
                    for (int j = 0; j < NJ; j++) {
                        const float w0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wgt[2 * j]), k));
                        const float w1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wgt[2 * j + 1]), k));
                        Oq[j] += x[k][j] * (half_p ? w1 : w0);
                    }
            };
            {
                // (partial k of the unit: the k-th entry; past the last one the last again, with weight 0)
                float ms[kNH], ls[kNH];
                f4 x[kWaves][NJ];
                const int count = __builtin_popcountll(same);
                int place = 0;
#pragma unroll
                for (int k = 0; k < kWaves; k++) {
                    const int e = __ffsll((long long)same) - 1;
                    if (same & (same - 1)) same &= same - 1;
                    place = lane == k ? e : place;
                    const float *p = part_of(e);
#pragma unroll
                    for (int j = 0; j < NJ; j++) x[k][j] = *reinterpret_cast<const f4 *>(p + (2 * j + half_p) * kPartialStride + 4 + 4 * c4);
                }
                const float *p = part_of(lane < kWaves ? place : head);
#pragma unroll
                for (int h = 0; h < kNH; h++) {
                    const bool on = lane < count && h < nheads;
                    const float2 ml = *reinterpret_cast<const float2 *>(p + (h < NHQ ? h : 0) * kPartialStride);
                    ms[h] = on ? ml.x : -1e30f;
                    ls[h] = on ? ml.y : 0.f;
                }
                fold(ms, ls, x, std::integral_constant<int, kWaves>{});
            }
            auto write_out = [&]() {
                if (FUSED && b->append && lane == 0) b->r_len_out[u] = rn >= 0 ? rn + 1 : b->r_len[u];
#pragma unroll
                for (int j = 0; j < NJ; j++) {
                    const int h = 2 * j + half_p;
                    if (h >= nheads) continue;
                    const float Lh = half_p ? L[2 * j + 1] : L[2 * j], inv = Lh > 0.f ? 1.0f / Lh : 0.f;
                    const h2 r0 = {(_Float16)(Oq[j][0] * inv), (_Float16)(Oq[j][1] * inv)};
                    const h2 r1 = {(_Float16)(Oq[j][2] * inv), (_Float16)(Oq[j][3] * inv)};
                    *reinterpret_cast<uint2 *>(b->out + (size_t)(bq0 + h) * kD + 4 * c4) = uint2{as_u32(r0), as_u32(r1)};
                }
            };
            if (gf == gl) { write_out(); continue; }

            auto slots = [&](int first) {
                return __builtin_amdgcn_make_buffer_rsrc(slot_of(first, 0), 0, 0x7fffffff, 0x00020000);
            };
            // (device scope throughout: the workgroups of a unit run on different dies, see take_ticket)
            auto publish = [&](int slot) {
                const __amdgpu_buffer_rsrc_t rs = slots(slot);
#pragma unroll
                for (int j = 0; j < NJ; j++)
                    if (2 * j + half_p < nheads)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, Oq[j]), rs, lane_off, 2 * j * kHeadB, kSc1);
#pragma unroll
                for (int h = 0; h < NHQ; h++)
                    if (h < nheads && lane == 0) { float *pp = slot_of(slot, h); st_agent(pp, M[h]); st_agent(pp + 1, L[h]); }
            };
            auto take_ticket = [&](int *counter) -> int {  // after this wave's stores are acknowledged
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                int old = 0;
                if (lane == 0) old = atomicAdd(counter, 1);
                return __builtin_amdgcn_readfirstlane(old);
            };
            // merges `count` partials, `stride` slots apart from slot `first`, MB of them a round trip
            auto merge = [&](int first, int stride, int count, auto mb) __attribute__((always_inline)) {
                constexpr int MB = decltype(mb)::value;
                const char *const sbase = reinterpret_cast<const char *>(slot_of(first, 0));
                const __amdgpu_buffer_rsrc_t rs = slots(first);
                const unsigned step = (unsigned)stride * kSlotB;
#pragma unroll
                for (int h = 0; h < kNH; h++) { M[h] = -1e30f; L[h] = 0.f; }
#pragma unroll
                for (int j = 0; j < NJ; j++) Oq[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int base = 0; base < count; base += MB) {
                    const int cnt = min(MB, count - base);
                    const bool has = lane < cnt;
                    const char *const mine_p = sbase + (size_t)(base + (has ? lane : 0)) * step;
                    float ms[kNH], ls[kNH];
#pragma unroll
                    for (int h = 0; h < kNH; h++) {
                        const bool on = has && h < nheads;
                        const float2 ml = h < NHQ ? ld_agent2(reinterpret_cast<const float *>(mine_p + h * kHeadB)) : float2{0.f, 0.f};
                        ms[h] = on ? ml.x : -1e30f;        // partials that do not exist get weight 0
                        ls[h] = on ? ml.y : 0.f;
                    }
                    f4 x[MB][NJ];
#pragma unroll
                    for (int k = 0; k < MB; k++) {
                        const unsigned pk = (unsigned)(base + min(k, cnt - 1)) * step;   // uniform
#pragma unroll
                        for (int j = 0; j < NJ; j++)
                            x[k][j] = __builtin_bit_cast(f4, (u4v)__builtin_amdgcn_raw_buffer_load_b128(rs, lane_off, pk + (unsigned)(2 * j * kHeadB), kSc1));
                    }
                    fold(ms, ls, x, mb);
                }
            };
            // Up to kOneLevel workgroups merge at once; more in sets of 16, whose results take the place of the set's first slot
            constexpr int kOneLevel = 32;
            const int expected = gl - gf + 1, me = group - gf;
            const int per = expected <= kOneLevel ? kOneLevel : 16, sg = expected <= kOneLevel ? 0 : me >> 4;
            const int n1 = min(per, expected - per * sg), nsg = expected <= kOneLevel ? 1 : (expected + 15) >> 4;
            const int slot1 = gf + per * sg + 2 * up;
            int into = group + 2 * up, from = slot1, stride = 1, count = n1;
            int *counter = b->cnt1 + slot1;
#pragma unroll 1
            for (bool last = nsg == 1;; last = true) {
                publish(into);
                if (take_ticket(counter) != count - 1) break;
                if (count <= 4) merge(from, stride, count, std::integral_constant<int, 4>{});
                else if (count <= 8) merge(from, stride, count, std::integral_constant<int, 8>{});
                else merge(from, stride, count, std::integral_constant<int, 16>{});
                if (lane == 0) st_agent_i32(counter, 0);   // ready for the next call
                if (last) { write_out(); break; }
                into = slot1, from = gf + 2 * up, stride = 16, count = nsg, counter = b->cnt + up;
            }
        }
    }
}

template <int G, bool LO, bool PAIRED, bool APPEND, bool UNIT, bool STREAM>
static int launch_form(const DecArgs &a, long groups, hipStream_t st)
{
    hipLaunchKernelGGL((decode_stream_kernel<G, LO, PAIRED, APPEND, UNIT, STREAM>), dim3((unsigned)groups),
                       dim3(64 * kGroupWaves<G>), 0, st, a);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

// Whether a workgroup per unit serves the call, from the capacities (the lengths are on the device).  It needs a compute
// unit per unit, and few enough items that the eight waves of a unit (four at G = 16) are done before the work line, which
// spreads the items over the whole device and balances ragged lengths, has paid for its round trips.  More items where the line
// cannot give a unit two workgroups (beyond 128 units), where a pass is short (G = 128), where one wave has a SIMD for itself (G =
// 16) fewer.  Time of the line over that of the unit form, mean (least) of attention and fused steps, one and two heads / three
// to eight heads per KV head, all lengths alike -- ragged (5 .. 100 % of the capacity):
//   units       G    at the limit                                               behind it
//   8 .. 48     16   10 items 1.20 (1.14) / 1.06 (0.97) -- 1.19 (1.08) / 1.04 (0.94)  12 items 1.10 / 0.98 -- 1.10 / 0.99
//               32   14 items / 1.11 (1.07) -- / 1.11 (1.04)                    18 items 1.12 / 0.98 -- 1.15 / 0.98 (0.90)
//               64   18 items 1.21 (1.12) / 1.09 (1.05) -- 1.22 (1.14) / 1.09 (1.00)
//               128  20 items 1.17 (1.10) / 1.12 (1.03) -- 1.28 (1.19) / 1.20 (1.10)
//   49 .. 95    16   12 items 1.26 (1.22) / 1.32 (1.24) -- 1.46 (1.24) / 1.36 (1.18)
//               32   14 items / 1.27 (1.21) -- / 1.27 (1.20)                    18 items 1.16 / 1.08 (1.07) -- 1.20 / 1.08 (1.03)
//               64   18 items 1.25 (1.22) / 1.18 (1.16) -- 1.30 (1.21) / 1.17 (1.10)
//               128  20 items 1.26 (1.21) / 1.22 (1.19) -- 1.34 (1.26) / 1.25 (1.18)
//   96 .. 128   16   20 items 1.15 (1.10) / 1.06 (0.99) -- 1.14 (0.97) / 1.04 (0.89)
//               32   22 items 1.26 (1.19) / 1.11 (1.04) -- 1.11 (1.05) / 0.98 (0.92)  26 items 1.18 / 1.06 -- 1.09 / 0.96 (0.86)
//               64   26 items 1.21 (1.20) / 1.10 (1.04) -- 1.10 (0.99) / 1.00 (0.88)
//               128  30 items 1.23 (1.17) / 1.11 (0.98) -- 1.11 (0.96) / 1.02 (0.88)
//   136 .. 192  16   26 items 1.21 (1.13) / 1.13 (1.06) -- 1.12 (0.98) / 1.02 (0.89)      28 items 1.19 / 1.13 -- 1.08 / 1.00
//                    two sets of heads: 20 items 1.19 (1.09) -- 1.10 (0.94)      24 items 1.17 (1.14) -- 1.04 (0.91)
//   193 .. 224  16   35 items 1.18 (1.11) -- 1.00 (0.90), four heads and more;  225 .. 256  1.11 (1.08) -- 1.09 (1.00)
//   225 .. 256  32   52 items 1.13 (1.10) / 1.09 (0.99) -- 1.08 (1.03) / 1.03 (0.98)   56 items 1.13 / 1.09 -- 1.06 / 1.00 (0.96)
//               128  60 items 1.18 (1.18) / 1.16 (1.12) -- 1.08 (1.03) / 1.02 (0.96)   66 items 1.12 / 1.07 -- 1.05 / 0.99 (0.94)
// Beyond 128 units the longest unit's compute unit decides, and with three heads and more the line wins back on ragged lengths the
// sooner the fewer units there are, hence units / 5; sooner with two sets of heads, whose words the line reads once (by_die).
// Three to eight heads, all lengths alike -- ragged, G = 32 / 64:
//   136 .. 159 units x 34 items 1.13 (1.12) / 1.18 (1.17) -- 1.04 (0.92) / 1.07 (0.94)   x 38 1.09 (1.07) -- 0.98 (0.89), G = 32
//                    x 42 items 1.09 (1.07) / 1.13 (1.11) -- 0.95 (0.89) / 0.98 (0.90)
//   160 .. 192 units x 38 items 1.17 (1.12) / 1.22 (1.15) -- 1.04 (0.93) / 1.07 (0.95)   x 42 1.14 (1.08) -- 1.00 (0.91), G = 32
//   193 .. 224 units x 44 items 1.19 (1.15) / 1.24 (1.20) -- 1.03 (0.97) / 1.05 (0.97)   x 52 1.12 (1.10) -- 0.97 (0.91), G = 32
static bool unit_per_workgroup(const DecArgs &a, int G, bool paired)
{
    const long units = (long)a.units * a.hsets;
    const long items = ((long)a.Tcap + kPass - 1) / kPass + ((long)a.Rcap + 63) / 64;
    if (units > kComputeUnits) return false;
    if (G == 16) return items <= (units > 192 ? 35 : units > 128 && a.hsets == 1 ? 26 : units >= 96 ? 20 : units >= 32 ? 12 : paired ? 11 : 10);
    if (units > 128) {
        const long most = units <= 192 ? 42 : G == 128 ? 66 : 52;
        return items <= most && (paired || items <= units / 5 + (G == 128 ? 12 : G == 64 ? 8 : 4) + (a.hsets > 1 ? 0 : G == 128 ? 66 : 4));
    }
    if (units >= 96) return items <= (G == 128 ? 30 : G == 64 ? 26 : 24);
    return items <= (G == 128 ? 20 : G == 64 || paired ? 18 : 14);
}

static std::atomic<int> g_decode_weights{0};
bool set_decode_weights(int mode)
{
    if (mode < 0 || mode > 2) return false;
    g_decode_weights.store(mode);
    return true;
}

template <int G, bool LO, bool PAIRED, bool APPEND>
static int launch_stream(DecArgs a, hipStream_t st)
{
    const long cap_items = (long)a.units * a.hsets * ((a.Tcap + kPass - 1) / kPass + (a.Rcap + 63) / 64);
    const int mode = g_decode_weights.load();
    // Weight of a residual item against a pass: 8 : 2 where every wave has several items (1344 items, G = 128, 11.7 us against
    // 12.5 with 4 : 2; 512 units x 12 items 22.5 against 23.3).  4 : 2 where the ranges would be too few for the compute units (64
    // units x 8 items 13.8 -> 11.8; 8 units x 42, G = 16, 17.9 -> 15.1), and where a wave has one or two items, so that one
    // with a residual item should hold nothing else (2816 items 18.8 -> 16.9, 3072 items 18.7 -> 17.2, but 5376 19.7 -> 20.2).
    // Time with 8 : 2 over that with 4 : 2, 880 calls of 32 to 768 units with residual tokens, mean (least .. most):
    //   items      1500 .. 2048       2049 .. 3584       3585 .. 4600       4601 .. 7000
    //   G = 16     1.02 (0.89..1.15)  1.01 (0.90..1.15)  0.98 (0.93..1.05)  1.00 (0.87..1.11)
    //   G > 16     1.04 (0.92..1.16)  1.04 (0.94..1.16)  1.02 (0.94..1.12)  1.02 (0.91..1.17)
    // so the window is where 4 : 2 gains most for what it can lose; outside it single calls gain as much and lose more.
    const long units = (long)a.units * a.hsets;
    const long weight = units * (2 * ((a.Tcap + kPass - 1) / kPass) + 8 * ((a.Rcap + 63) / 64));
    const bool light = weight < 8 * kComputeUnits || (cap_items > 2048 && cap_items <= 3584);
    a.wq_log = mode == 2 ? 0 : 1, a.wr_log = mode == 2 ? 0 : mode == 0 && light ? 2 : 3;
    // Two sets of heads read the same words: their workgroups on one die find them in its L2 (128 units x 102 items 35.1 ->
    // 32.0 us, x 42 22.0 -> 20.6), if a die's eighth holds both; small calls lose (8 units x 22 items 13.8 -> 14.4).
    a.by_die = a.hsets > 1 && cap_items > 2048 && units >= 16;
    // More than 16 workgroups a unit (a merge of two loops) only where each has eight items (8 units x 102 items, G = 128, 15.1
    // us with 32 workgroups a unit, 13.6 with 16; but 8 x 784 28.3 against 31.0).
    long groups = cap_items < kComputeUnits ? cap_items : kComputeUnits;
    const long few = 16 * units > cap_items / 8 ? 16 * units : cap_items / 8;
    groups = groups < few ? groups : few;
    // Streaming loads where the packed cache (by its capacity) is larger than a third of the 256 MB memory-side cache and a
    // call reads it once.  Twice, with two sets of heads, the hint loses at every size (8 heads per KV head, G = 32, 200 MB
    // 71.8 -> 75.1 us, 300 MB 101 -> 105; 6 heads the same, G = 16 1 % less, G = 128 3 % from 300 MB on).  Once, with three
    // caches in turn and 90 / 120 / 300 MB (4 heads per KV head, then one; 128 units):
    //   G = 16   31.3 -> 30.9 / 37.9 -> 35.4 / 74.3 -> 70.5        (320 units) 39.6 -> 35.2 at 120, 77.5 -> 73.3 at 300
    //   G = 32   27.9 -> 27.7 / 33.6 -> 30.6 / 67.3 -> 62.3        33.5 -> 29.4, 65.8 -> 60.9
    //   G = 64   26.5 -> 26.3 / 32.9 -> 31.3 / 64.9 -> 60.6        (2 heads) 26.1 -> 25.5 at 90
    //   G = 128  26.2 -> 26.0 / 32.5 -> 31.9 / 64.2 -> 61.5        (320 units) 36.4 -> 32.6, 70.1 -> 60.2
    // Smaller ones may still be there from the call before, and are then read faster with ordinary loads (65 MB: G = 128 24.8
    // against 25.8, 2 heads 20.8 against 22.0, G = 64 24.3 against 25.1, G = 16 and 32 within 1 %), unless ten of them take
    // turns (the hint gains 1-5 % from 65 MB on).  That is also what a cache sees that is allocated long and filled short:
    // 40 MB in 160 17.7 -> 17.9 us at G = 32, 18.1 -> 18.6 at G = 64, 17.7 -> 18.5 at G = 128 if it is among the last three,
    // and nothing otherwise.  The lengths are not known here.  Choosing in the kernel by the total of the work line costs
    // more than that (a branch at each pair of loads: 65 MB 21.7 -> 24.2 us; a second copy of the pass loop does not fit the
    // registers).
    constexpr long kStreamBytes = 88L << 20;
    const bool streams = (long)a.units * a.Tcap * (64 + 8 * kD / G) > kStreamBytes && a.hsets == 1;
    if (mode == 0 && unit_per_workgroup(a, G, PAIRED))
        return streams ? launch_form<G, LO, PAIRED, APPEND, true, true>(a, units, st) : launch_form<G, LO, PAIRED, APPEND, true, false>(a, units, st);
    return streams ? launch_form<G, LO, PAIRED, APPEND, false, true>(a, groups, st) : launch_form<G, LO, PAIRED, APPEND, false, false>(a, groups, st);
}

template <bool LO, bool PAIRED>
static int launch_stream_g(const DecArgs &a, int G, hipStream_t st)
{
    if (a.append) {
        switch (G) {
        case 16: return launch_stream<16, LO, PAIRED, true>(a, st);
        case 32: return launch_stream<32, LO, PAIRED, true>(a, st);
        case 64: return launch_stream<64, LO, PAIRED, true>(a, st);
        case 128: return launch_stream<128, LO, PAIRED, true>(a, st);
        }
        return MINIKV_EUNSUPPORTED;
    }
    switch (G) {
    case 16: return launch_stream<16, LO, PAIRED, false>(a, st);
    case 32: return launch_stream<32, LO, PAIRED, false>(a, st);
    case 64: return launch_stream<64, LO, PAIRED, false>(a, st);
    case 128: return launch_stream<128, LO, PAIRED, false>(a, st);
    }
    return MINIKV_EUNSUPPORTED;
}

int launch_decode_tiled(const DecArgs &a, int G, int units, int variant, hipStream_t st)
{
    (void)units;
    if (variant != 3) return MINIKV_EINVAL;
    return a.rep <= 2 ? launch_stream_g<true, true>(a, G, st) : launch_stream_g<true, false>(a, G, st);
}

}  // namespace minikv
