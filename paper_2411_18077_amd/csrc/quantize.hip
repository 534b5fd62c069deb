// kv_quantize_pack / kv_flush_residual / kv_append_residual kernels (gfx950).
//
// Quantizer: Section 3.1.1 and Section 3.3 of the MiniKV paper -- asymmetric 2-bit codes, K grouped
// along tokens per channel, V grouped along channels per token, fp16 scale and zero-point, 16 codes per
// 32-bit word.  Residual buffer: Algorithm 1 lines 9-15.
//
// A wave takes the keys or the values of a block of 64 consecutive retained tokens of one unit and keeps them in registers:
// lane 16 q + p holds channels 8 p .. 8 p + 7 of tokens 16 q .. 16 q + 15, sixteen 128-bit loads that are all in flight at
// once (Algorithm 1 line 3: only retained rows are read).  Statistics, codes and words are formed where the data is; local
// memory carries only the group parameters and the finished words on their way to coalesced stores, and the waves of a
// workgroup meet at no barrier (but one where a group of 128 tokens spans two of them).
//
// What bounds it: memory.  An element costs about 8.9 vector instructions (5 of them the quantizer's own roundings), half of
// the time.  Rows and words pass the caches once, so both carry the streaming hint: a call on 128 units x 13088 of 32768
// rows, G = 32, three sets of inputs in turn, takes 209 us without it, 200 with it on the loads or the stores alone, 180 (5.7
// TB/s) with it on both (188 while the code words went through a private segment).  An earlier form, blocks in local memory
// and four waves on each with barriers between the passes, took 214 there (129 -> 61 us at G = 128, 32 units x 17664, where
// half its threads had no statistics to do; 151 -> 132 at G = 64, 32 x 40000; 71 -> 62 at G = 16, 256 units x 2048; a flush of
// 256 x 128 rows at G = 16 10.9 -> 9.8).
#include "common.h"

#include <hip/hip_fp16.h>

#include <utility>

namespace minikv {

struct QuantArgs {
    const uint16_t *K, *V;       // [U][L][D] fp16
    const int32_t *idx;          // [U][idx_stride] or null
    const int32_t *n_tok;        // [U]  (flush: r_len)
    uint32_t *Kc, *Vc;
    uint16_t *Ks, *Kz, *Vs, *Vz;
    int32_t *q_len, *r_len;
    int64_t L, idx_stride;
    int Tcap, Rcap, flush;
    int max_tok;                 // host-side bound of n_tok the launch was sized for
    int units;
};

__device__ inline float h2f(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// Tokens this unit appends, or 0 when the request is not a positive multiple of G that fits.
template <int G>
__device__ inline int tokens_to_append(const QuantArgs &a, int u, int &q0)
{
    int n = a.n_tok[u];
    q0 = a.q_len[u];
    if (a.flush) n = (n == a.Rcap) ? a.Rcap : 0;
    if (n <= 0 || (n % G) || q0 < 0 || (q0 % G) || q0 + n > a.Tcap || n > a.L || n > a.max_tok) return 0;
    return n;
}

// scale (fp16 bits), zero (fp16 bits), 1/scale (binary32) of a group with extrema mn, mx.
__device__ inline void group_params(float mn, float mx, uint16_t &sh, uint16_t &zh, float &inv, float &zf)
{
    __half z = __float2half_rn(mn);                   // exact: mn is an fp16 value
    zh = __half_as_ushort(z);
    if ((zh & 0x7fffu) == 0) zh = 0;                  // -0 is stored as +0
    zf = h2f(zh);
    float range = mx - mn;
    float step = range / 3.0f;                        // IEEE binary32 division
    __half s = __float2half_rn(step);
    sh = __half_as_ushort(s);
    float sf = __half2float(s);
    inv = (sf == 0.0f) ? 0.0f : 1.0f / sf;
}

typedef _Float16 qh2 __attribute__((ext_vector_type(2)));
__device__ inline qh2 as_qh2(uint32_t u) { return __builtin_bit_cast(qh2, u); }
__device__ inline qh2 pk_min(qh2 a, qh2 b) { return __builtin_elementwise_min(a, b); }
__device__ inline qh2 pk_max(qh2 a, qh2 b) { return __builtin_elementwise_max(a, b); }

// code of x as a float 0..3 (round half to even, clamped): every operation a separately rounded binary32 one.
// nzi = (-zero, 1/scale).  x - zero is written as the fused x * one + (-zero) with `one` a 1.0 the compiler cannot
// see through: the conversion of the fp16 x then folds into the instruction (v_fma_mix_f32) and the result is
// the same single rounding of x - zero.
__device__ inline float quant_codef(_Float16 x, float2 nzi, float one)
{
    const float d = __builtin_fmaf((float)x, one, nzi.x);
    const float u = d * nzi.y;
    return __builtin_amdgcn_fmed3f(rintf(u), 0.0f, 3.0f);
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Orders this wave's local-memory writes before its reads (the hardware keeps them in order; this is for the compiler).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Lane I of every row of 16 lanes, to the whole row.
template <int I>
__device__ __forceinline__ int row_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + I, 0xf, 0xf, false); }
__device__ __forceinline__ uint32_t neighbour(uint32_t v)        // of the lane next door (lane ^ 1)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, false);
}
// Tokens 16 q .. 16 q + 15 of the block, this lane's 16-byte piece of each; lane t knows where token t's row is.
template <int... I>
__device__ __forceinline__ void load_rows(u32x4 (&x)[16], const uint16_t *src, int row, std::integer_sequence<int, I...>)
{
    const int piece = (threadIdx.x & 15) * 8;
    ((x[I] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + (size_t)(uint32_t)row_lane<I>(row) * kD + piece))), ...);
}

// Where a wave's tokens go: nt of them (a multiple of min(G, 64)), to token t0 of unit u.  With PAIR (units of at most 32
// tokens, groups of at most 32) the lower half of the wave is one unit and the upper half the next.
struct Place { int u, nt, t0; };

// Half of the workgroup's waves take keys, the others values; both kinds of one block sit next to each other.
constexpr int kBlock = 64;                               // tokens of a wave
template <int G> constexpr int kKGroups = G < kBlock ? kBlock / G : 1;
constexpr int kKPitch = 164, kKPitchQ = 40;              // words: code words of the keys on their way out (banks differ by q, word half)
constexpr int kStatPitch = 68, kVPitch = 36, kParPitch = 72, kParPitchQ = 18;
template <int G> constexpr int kKeyLds = kKGroups<G> * 1024 + 4 * kKPitch * 4;            // bytes
template <int G> constexpr int kValueLds = 16 * kStatPitch * 4 + kD / G * kParPitch * 8;

// Keys: groups of G tokens of one channel.
//   statistics  packed fp16 minima and maxima (exact) down the lane's 16 tokens, then between the rows of lanes of a group
//               by exchanging halves: each step halves the channels a lane is left with, so that every lane ends with its
//               share of the groups and computes scale, zero-point and reciprocal once per group
//   words       16 channels of a token are two lanes' work: 8 codes as one exact binary32 sum each (below 2^24), joined
//               with the neighbour's
template <int G, bool PAIR>
__device__ __forceinline__ void quantize_keys(const QuantArgs &a, const u32x4 (&x)[16], char *lds, uint32_t *exchange, int sub,
                                              const Place &lower, const Place &upper)
{
    const int lane = threadIdx.x & 63, q = lane >> 4, p = lane & 15;
    float one = 1.0f;
    asm volatile("" : "+v"(one));                        // (see quant_codef)
    qh2 mn[4], mx[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        mn[k] = mx[k] = as_qh2(x[0][k]);
#pragma unroll
        for (int i = 1; i < 16; i++) mn[k] = pk_min(mn[k], as_qh2(x[i][k])), mx[k] = pk_max(mx[k], as_qh2(x[i][k]));
    }
    constexpr int NP = G == 16 ? 4 : G == 32 ? 2 : 1;     // channel pairs a lane is left with
    auto meet16 = [](qh2 v, qh2 w, auto op) -> qh2 {     // rows 0, 2 of lanes: v over rows 2j, 2j + 1; rows 1, 3: w
        const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, w), false, false);
        return op(as_qh2(s[0]), as_qh2(s[1]));
    };
    auto meet32 = [](qh2 v, qh2 w, auto op) -> qh2 {     // lower half of the wave: v over both halves; upper half: w
        const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, v), __builtin_bit_cast(uint32_t, w), false, false);
        return op(as_qh2(s[0]), as_qh2(s[1]));
    };
    if constexpr (G >= 32) {
#pragma unroll
        for (int k = 0; k < 2; k++) mn[k] = meet16(mn[k], mn[k + 2], pk_min), mx[k] = meet16(mx[k], mx[k + 2], pk_max);
    }
    if constexpr (G >= 64) mn[0] = meet32(mn[0], mn[1], pk_min), mx[0] = meet32(mx[0], mx[1], pk_max);
    if constexpr (G == 128) {                            // the other half of the tokens is with the next wave of keys
        uint32_t *mine = exchange + sub * 128 + lane, *other = exchange + (sub ^ 1) * 128 + lane;
        mine[0] = __builtin_bit_cast(uint32_t, mn[0]), mine[64] = __builtin_bit_cast(uint32_t, mx[0]);
        __syncthreads();
        mn[0] = pk_min(mn[0], as_qh2(other[0])), mx[0] = pk_max(mx[0], as_qh2(other[64]));
    }
    // this lane's channel pairs are first, first + 1, ... of the four of piece p
    const int first = G == 16 ? 0 : G == 32 ? 2 * (q & 1) : 2 * (q & 1) + (q >> 1);
    const int group = G == 16 ? q : G == 32 ? q >> 1 : 0;
    float4 *par = reinterpret_cast<float4 *>(lds) + group * 64 + p;        // [group][pair][piece]: (-zero, 1/scale) of two channels
    auto place = [&](int half) -> Place { return PAIR && half ? upper : lower; };
    uint32_t sw[NP], zw[NP];
#pragma unroll
    for (int k = 0; k < NP; k++) {
        uint16_t sh[2], zh[2];
        float inv[2], zf[2];
#pragma unroll
        for (int e = 0; e < 2; e++) group_params((float)mn[k][e], (float)mx[k][e], sh[e], zh[e], inv[e], zf[e]);
        sw[k] = sh[0] | (uint32_t)sh[1] << 16, zw[k] = zh[0] | (uint32_t)zh[1] << 16;
        par[(first + k) * 16] = float4{-zf[0], inv[0], -zf[1], inv[1]};
    }
    const Place dst = place(q >> 1);
    const int of_unit = PAIR ? group % (32 / (G < 32 ? G : 32)) : group;
    if (of_unit * G < dst.nt && (G < 128 || (sub & 1) == 0)) {
        const size_t row = ((size_t)dst.u * (a.Tcap / G) + (size_t)(dst.t0 / G + of_unit)) * kD;      // (G = 128: t0 of the even wave)
        if constexpr (NP == 1) {
            const size_t o = row + k_meta_pos(G, 8 * p + 2 * first);
            *reinterpret_cast<uint32_t *>(a.Ks + o) = sw[0], *reinterpret_cast<uint32_t *>(a.Kz + o) = zw[0];
        } else {
#pragma unroll
            for (int k = 0; k < NP; k += 2) {            // a quad of channels is contiguous
                const size_t o = row + k_meta_pos(G, 8 * p + 2 * (first + k));
                *reinterpret_cast<uint2 *>(a.Ks + o) = uint2{sw[k], sw[k + 1]};
                *reinterpret_cast<uint2 *>(a.Kz + o) = uint2{zw[k], zw[k + 1]};
            }
        }
    }
    wave_sync();
    float4 pv[4];
    {
        const float4 *mine = reinterpret_cast<const float4 *>(lds) + group * 64 + p;
#pragma unroll
        for (int k = 0; k < 4; k++) pv[k] = mine[k * 16];
    }
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const qh2 v = as_qh2(x[i][k]);
            acc = __builtin_fmaf(quant_codef(v[0], float2{pv[k].x, pv[k].y}, one), (float)(1 << 2 * k), acc);
            acc = __builtin_fmaf(quant_codef(v[1], float2{pv[k].z, pv[k].w}, one), (float)(65536 << 2 * k), acc);
        }
        w[i] = (uint32_t)acc << 8 * (p & 1);             // channels 8.. of the word sit 8 bits up
        w[i] |= neighbour(w[i]);
    }
    // lanes of a pair share the store of their words: the even one the first eight tokens, the odd one the others
    uint32_t *words = reinterpret_cast<uint32_t *>(lds + kKGroups<G> * 1024);
    const int wd = p >> 1, odd = p & 1, at = (wd >> 2) * kKPitch + q * kKPitchQ + (wd & 3) + odd * 16;
    const uint32_t second = 0u - (uint32_t)odd;          // (a mask: of `odd ? :` the compiler makes an index, and of w memory)
#pragma unroll
    for (int i = 0; i < 8; i++) words[at + (i & 1) * 2 * kKPitch + (i >> 1) * 4] = w[i] ^ ((w[i] ^ w[i + 8]) & second);
    wave_sync();
#pragma unroll
    for (int s = 0; s < 2; s++) {                        // piece (token parity, word half, token pair): four words of a token
        const int ch = 2 * s + (lane >> 5), pr = lane & 31, t = 2 * (PAIR ? pr & 15 : pr) + s;
        const Place to = place(pr >> 4);
        const u32x4 v = *reinterpret_cast<const u32x4 *>(words + ch * kKPitch + (pr >> 3) * kKPitchQ + (pr & 7) * 4);
        uint32_t *Kc = a.Kc + (size_t)to.u * kc_words(a.Tcap);
        if (t < to.nt) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(Kc + k_word_index(to.t0 + t, (ch & 1) * 4)));
    }
}

// Values: groups of G channels of one token.
//   statistics  (minimum, -maximum) of the lane's eight channels as one packed pair per token, turned through local memory
//               so that lane t finishes the groups of token t
//   words       16 tokens of a channel are one lane's work; the words of a 64-token tile go out together
template <int G, bool PAIR>
__device__ __forceinline__ void quantize_values(const QuantArgs &a, const u32x4 (&x)[16], char *lds, const Place &lower, const Place &upper)
{
    constexpr int NCG = kD / G, kPieces = G / 8;
    const int lane = threadIdx.x & 63, q = lane >> 4, p = lane & 15;
    float one = 1.0f;
    asm volatile("" : "+v"(one));
    uint32_t *stats = reinterpret_cast<uint32_t *>(lds);                   // [piece][token], pitch kStatPitch
    float2 *par = reinterpret_cast<float2 *>(lds + 16 * kStatPitch * 4);   // [group][token], 16 tokens per kParPitchQ
#pragma unroll
    for (int i4 = 0; i4 < 4; i4++) {
        u32x4 m;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const u32x4 v = x[4 * i4 + j];
            const qh2 x0 = as_qh2(v[0]), x1 = as_qh2(v[1]), x2 = as_qh2(v[2]), x3 = as_qh2(v[3]);
            const qh2 lo = pk_min(pk_min(x0, x1), pk_min(x2, x3)), hi = pk_max(pk_max(x0, x1), pk_max(x2, x3));
            m[j] = __builtin_bit_cast(uint32_t, pk_min(qh2{lo[0], -hi[0]}, qh2{lo[1], -hi[1]}));
        }
        *reinterpret_cast<u32x4 *>(stats + p * kStatPitch + 16 * q + 4 * i4) = m;
    }
    wave_sync();
    qh2 m[16];
#pragma unroll
    for (int k = 0; k < 16; k++) m[k] = as_qh2(stats[k * kStatPitch + lane]);
    uint16_t sh[NCG], zh[NCG];
#pragma unroll
    for (int g = 0; g < NCG; g++) {
        qh2 r = m[g * kPieces];
#pragma unroll
        for (int k = 1; k < kPieces; k++) r = pk_min(r, m[g * kPieces + k]);
        float inv, zf;
        group_params((float)r[0], -(float)r[1], sh[g], zh[g], inv, zf);
        par[g * kParPitch + q * kParPitchQ + p] = float2{-zf, inv};
    }
    auto place = [&](int half) -> Place { return PAIR && half ? upper : lower; };
    const Place dst = place(lane >> 5);
    const int token = PAIR ? lane & 31 : lane;
    if (token < dst.nt) {
        const size_t o = ((size_t)dst.u * a.Tcap + (size_t)(dst.t0 + token)) * NCG;
        __builtin_memcpy(__builtin_assume_aligned(a.Vs + o, 2 * NCG), sh, 2 * NCG);
        __builtin_memcpy(__builtin_assume_aligned(a.Vz + o, 2 * NCG), zh, 2 * NCG);
    }
    wave_sync();
    float4 pv[8];                                        // tokens 2j, 2j + 1 of this lane's sixteen
    {
        const float4 *mine = reinterpret_cast<const float4 *>(par + (p / kPieces) * kParPitch + q * kParPitchQ);
#pragma unroll
        for (int j = 0; j < 8; j++) pv[j] = mine[j];
    }
    uint32_t *words = stats;                             // (the statistics have been read)
#pragma unroll
    for (int e = 0; e < 8; e++) {
        float lo = 0.0f, hi = 0.0f;                      // even and odd tokens: exact sums below 2^16
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const float wgt = (float)(1 << 2 * j);
            lo = __builtin_fmaf(quant_codef(as_qh2(x[2 * j][e >> 1])[e & 1], float2{pv[j].x, pv[j].y}, one), wgt, lo);
            hi = __builtin_fmaf(quant_codef(as_qh2(x[2 * j + 1][e >> 1])[e & 1], float2{pv[j].z, pv[j].w}, one), wgt, hi);
        }
        words[p * kVPitch + e * 4 + q] = (uint32_t)lo | (uint32_t)hi << 16;
    }
    wave_sync();
    if (!PAIR && lower.nt == kBlock && (lower.t0 & 63) == 0) {            // a whole tile: four blocks of a channel are contiguous
        uint32_t *Vc = a.Vc + (size_t)lower.u * vc_words(a.Tcap);
#pragma unroll
        for (int s = 0; s < 2; s++) {
            const int c = lane + 64 * s;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(words + (c >> 3) * kVPitch + (c & 7) * 4);
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(Vc + v_word_index(lower.t0 / 16, c)));
        }
    } else {
        const Place to = place((lane >> 1) & 1);
        const int bl = PAIR ? lane & 1 : lane & 3;       // block of 16 tokens of the unit
        uint32_t *Vc = a.Vc + (size_t)to.u * vc_words(a.Tcap);
#pragma unroll
        for (int s = 0; s < 8; s++) {
            const int c = (lane >> 2) + 16 * s;
            if (bl * 16 < to.nt) Vc[v_word_index(to.t0 / 16 + bl, c)] = words[(c >> 3) * kVPitch + (c & 7) * 4 + (lane & 3)];
        }
    }
}

// NBLK blocks of 64 tokens per workgroup, two waves each.  WHOLE: the workgroup is a whole unit of at most NBLK blocks (PAIR:
// two units of at most half a block) and leaves the new lengths; otherwise update_lengths_kernel follows.
template <int G, int NBLK, bool WHOLE, bool PAIR>
__global__ __launch_bounds__(128 * NBLK, 4) void quantize_pack_kernel(QuantArgs a)
{
    static_assert(G < 128 || NBLK % 2 == 0, "a group of 128 tokens is two blocks of one workgroup");
    static_assert(!PAIR || (WHOLE && NBLK == 1 && G <= 32), "halves of a block hold whole groups");
    __shared__ __attribute__((aligned(16))) char lds[NBLK * (kKeyLds<G> + kValueLds<G>)];
    __shared__ uint32_t exchange[G == 128 ? NBLK * 128 : 1];

    const int lane = threadIdx.x & 63, half = PAIR ? lane >> 5 : 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = wave >> 1;
    const bool values = wave & 1;
    const int u0 = PAIR ? 2 * (int)blockIdx.y : (int)blockIdx.y, u1 = PAIR ? min(u0 + 1, a.units - 1) : u0;
    const int i0 = (WHOLE ? 0 : (int)blockIdx.x * NBLK * kBlock) + sub * kBlock;
    // the position of this lane's token (requested together with the lengths; the address lies inside the list whatever they are)
    const int u = half ? u1 : u0, token = PAIR ? lane & 31 : lane;
    int row = i0 + token;
    if (a.idx) row = a.idx[(size_t)u * a.idx_stride + min(row, a.max_tok - 1)];
    int q0, q1 = 0;
    const int n = tokens_to_append<G>(a, u0, q0), n1 = PAIR && u1 > u0 ? tokens_to_append<G>(a, u1, q1) : 0;
    if (WHOLE ? (n | n1) == 0 : (int)blockIdx.x * NBLK * kBlock >= n) return;      // (uniform in the workgroup)
    if (WHOLE) {
        __syncthreads();                                 // (every wave has read the lengths)
        if (threadIdx.x == 0 && n) {
            a.q_len[u0] = q0 + n;
            if (a.flush) a.r_len[u0] = 0;
        }
        if (PAIR && threadIdx.x == 0 && n1) {
            a.q_len[u1] = q1 + n1;
            if (a.flush) a.r_len[u1] = 0;
        }
    }
    const Place lower = {u0, max(min(n - i0, kBlock), 0), q0 + i0}, upper = {u1, n1, q1};      // nt = 0: nothing for this wave
    if (!PAIR && G < 128 && lower.nt == 0) return;
    if (token >= (half ? upper.nt : lower.nt)) row = 0;
    row = min(max(row, 0), (int)min(a.L - 1, (int64_t)0x7fffffff));
    u32x4 x[16];
    load_rows(x, (values ? a.V : a.K) + (size_t)u * a.L * kD, row, std::make_integer_sequence<int, 16>());
    char *const mine = lds + sub * (kKeyLds<G> + kValueLds<G>);
    if (!values) {
        quantize_keys<G, PAIR>(a, x, mine, exchange, sub, lower, upper);
    } else {
        if constexpr (G == 128) __syncthreads();         // (the two waves of keys exchange their halves' statistics)
        quantize_values<G, PAIR>(a, x, mine + kKeyLds<G>, lower, upper);
    }
}

// Runs after every workgroup of quantize_pack_kernel has finished (next kernel on the stream).
template <int G>
__global__ void update_lengths_kernel(QuantArgs a)
{
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= a.units) return;
    int q0;
    const int n = tokens_to_append<G>(a, u, q0);
    if (n == 0) return;
    a.q_len[u] = q0 + n;
    if (a.flush) a.r_len[u] = 0;
}

// One workgroup of 64 threads per group of 2 units: thread = (unit, K or V, 16-byte piece).  The new rows
// are requested together with the length, so the kernel costs one memory round trip plus the store.
__global__ __launch_bounds__(64) void append_residual_kernel(const uint16_t *k_new, const uint16_t *v_new,
                                                             uint16_t *Rk, uint16_t *Rv, int32_t *r_len,
                                                             int Rcap, int units)
{
    const int tid = threadIdx.x;
    const int u = blockIdx.x * 2 + (tid >> 5);
    if (u >= units) return;
    const int which = (tid >> 4) & 1, piece = tid & 15;
    const uint4 row = reinterpret_cast<const uint4 *>((which ? v_new : k_new) + (size_t)u * kD)[piece];
    const int r = r_len[u];
    if (r < 0 || r >= Rcap) return;
    uint16_t *dst = (which ? Rv : Rk) + ((size_t)u * Rcap + r) * kD;
    reinterpret_cast<uint4 *>(dst)[piece] = row;
    // every thread of the unit has its r in a register by now (the loads above were waited for), so the
    // length can be bumped without a barrier
    if ((tid & 31) == 0) r_len[u] = r + 1;
}

template <int G>
static int launch_quantize_g(const QuantArgs &a, hipStream_t st)
{
    constexpr int NB = G == 128 ? 2 : 1;                 // blocks per workgroup
    const int units = a.units, nblk = (a.max_tok + kBlock - 1) / kBlock;
    // Up to four blocks: one workgroup per unit, no launch of update_lengths_kernel behind this one (2.5 us of a call); its waves
    // wait for each other only for the lengths.  One or two blocks always (the call, against two launches, 64 units x 128 rows
    // 12.3 -> 9.7 us, 1024 x 128 20.3 -> 18.7, 4096 x 128 60 -> 58).  Three or four take a workgroup of four, of which a compute
    // unit holds two, the fourth with nothing to do for three: only while each has a compute unit (256 x 144 12.3 -> 10.4, x 256
    // 13.1 -> 11.7) or most compute units have as many as the others (320 x 144 12.4 -> 14.4, x 256 15.4 -> 16.7, but 512 x 144
    // 16.8 -> 15.3, x 256 21.2 -> 19.4, 768 x 192 23.1 -> 22.3), and, beyond two on each, while their waves have mostly full
    // blocks (1024 x 144 23.4 -> 25.8, x 256 34.9 -> 34.4) and few rounds to go (2048 x 192 47.9 -> 49.8, 4096 x 256 114 -> 117).
    // Up to 32 tokens: two units share a block (16-token groups, 1024 units x 32 rows 10.4 -> 10.2 us, 2048 15.9 -> 13.0, 4096
    // 24.9 -> 19.8; 256 units the same: there the waves' own instructions count, and half of every wave would idle).
    const bool even_rounds = units >= kComputeUnits * 3 / 2 && units <= (a.max_tok > 160 ? 4 : 2) * kComputeUnits;
    if (nblk <= 2 || (nblk <= 4 && (units <= kComputeUnits || even_rounds))) {
        if (nblk > 2) {
            hipLaunchKernelGGL((quantize_pack_kernel<G, 4, true, false>), dim3(1, units), dim3(512), 0, st, a);
        } else if (nblk == 2 || G == 128) {
            hipLaunchKernelGGL((quantize_pack_kernel<G, 2, true, false>), dim3(1, units), dim3(256), 0, st, a);
        } else if constexpr (G <= 32) {
            if (a.max_tok <= 32)
                hipLaunchKernelGGL((quantize_pack_kernel<G, 1, true, true>), dim3(1, (units + 1) / 2), dim3(128), 0, st, a);
            else
                hipLaunchKernelGGL((quantize_pack_kernel<G, 1, true, false>), dim3(1, units), dim3(128), 0, st, a);
        } else if constexpr (G == 64) {
            hipLaunchKernelGGL((quantize_pack_kernel<G, 1, true, false>), dim3(1, units), dim3(128), 0, st, a);
        }
        return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
    }
    hipLaunchKernelGGL((quantize_pack_kernel<G, NB, false, false>), dim3((nblk + NB - 1) / NB, units), dim3(128 * NB), 0, st, a);
    hipLaunchKernelGGL(update_lengths_kernel<G>, dim3((units + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

int launch_quantize(const minikv_shape &s, const minikv_f16 *K, const minikv_f16 *V, int64_t L,
                    const int32_t *idx, int64_t idx_stride, const int32_t *n_tok, int32_t max_tok,
                    const minikv_cache &c, bool flush, hipStream_t st)
{
    QuantArgs a;
    a.K = K; a.V = V; a.idx = idx; a.n_tok = n_tok;
    a.Kc = c.Kc; a.Vc = c.Vc; a.Ks = c.Ks; a.Kz = c.Kz; a.Vs = c.Vs; a.Vz = c.Vz;
    a.q_len = c.q_len; a.r_len = c.r_len;
    a.L = L; a.idx_stride = idx_stride; a.Tcap = s.Tcap; a.Rcap = s.Rcap; a.flush = flush ? 1 : 0;
    a.max_tok = max_tok;
    a.units = s.B * s.Hkv;
    switch (s.G) {
    case 16: return launch_quantize_g<16>(a, st);
    case 32: return launch_quantize_g<32>(a, st);
    case 64: return launch_quantize_g<64>(a, st);
    case 128: return launch_quantize_g<128>(a, st);
    }
    return MINIKV_EUNSUPPORTED;
}

int launch_append(const minikv_shape &s, const minikv_f16 *k_new, const minikv_f16 *v_new,
                  const minikv_cache &c, hipStream_t st)
{
    const int units = s.B * s.Hkv;
    hipLaunchKernelGGL(append_residual_kernel, dim3((units + 1) / 2), dim3(64), 0, st, k_new, v_new, c.Rk,
                       c.Rv, c.r_len, s.Rcap, units);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

}  // namespace minikv
