// Per-token quantized KV cache: the token-wise quantization the paper's appendix studies (8, 4 and 2 bits for
// keys and values alike; 2 bits is the case it reports as failing) and its 4-bit baseline, whose size the
// appendix on KV cache compression ratios works out.  Keys are quantized like values: the G channels of one
// token share a zero-point and a scale.  Entry points: kv_quantize_pack_pt, minikv_decode_attn_pt.
//
// Storage (per unit; cpw = 32 / bits codes per word, code i of a word at bits [bits*i, bits*i + bits)):
//   Kc [Tcap][D/cpw]   token major (a token's codes are contiguous: the score phase has one token per thread)
//   Vc [Tcap/cpw][D]   channel major (a word = cpw consecutive tokens of one channel: the value phase has one
//                      channel per thread and consecutive threads read consecutive words)
//   Ks, Kz, Vs, Vz fp16 [Tcap][D/G];  q_len int32, a multiple of 16.
#include "common.h"

#include <hip/hip_fp16.h>

namespace minikv {

constexpr int kPtBlockTok = 64;      // tokens one workgroup of the quantizer takes
constexpr int kPtMinChunk = 256;     // least tokens of a decode workgroup
constexpr int kPtMaxRep = 8;

struct PtQuantArgs {
    const uint16_t *K, *V;
    const int32_t *idx, *n_tok;
    uint32_t *Kc, *Vc;
    uint16_t *Ks, *Kz, *Vs, *Vz;
    int32_t *q_len;
    int64_t L, idx_stride;
    int Tcap, max_tok;
};

__device__ inline float pt_h2f(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// Tokens this unit appends, or 0 when the request is not a positive multiple of 16 that fits.
__device__ inline int pt_tokens_to_append(const PtQuantArgs &a, int u, int &q0)
{
    const int n = a.n_tok[u];
    q0 = a.q_len[u];
    if (n <= 0 || (n & 15) || q0 < 0 || (q0 & 15) || q0 + n > a.Tcap || n > a.L || n > a.max_tok) return 0;
    return n;
}

// The quantizer of one group: zero = min (fp16, -0 stored as +0), scale = fp16((max - min) / levels) in
// binary32, 1/scale of the STORED scale; every operation separately rounded (this file is compiled without
// floating-point contraction).
__device__ inline void pt_group_params(float mn, float mx, float levels, uint16_t &sh, uint16_t &zh, float &inv, float &zf)
{
    zh = __half_as_ushort(__float2half_rn(mn));
    if ((zh & 0x7fffu) == 0) zh = 0;
    zf = pt_h2f(zh);
    const float range = mx - mn;
    const float step = range / levels;
    const __half s = __float2half_rn(step);
    sh = __half_as_ushort(s);
    const float sf = __half2float(s);
    inv = (sf == 0.0f) ? 0.0f : 1.0f / sf;
}
__device__ inline uint32_t pt_code(float x, float zf, float inv, float levels)
{
    const float d = x - zf;
    const float u = d * inv;
    return (uint32_t)(int)__builtin_amdgcn_fmed3f(rintf(u), 0.0f, levels);
}

// One thread = 16 consecutive channels of one token; a group of G channels = G/16 neighbouring threads.
// Returns the thread's 16 codes; the group's first thread stores scale and zero-point at meta_at.
template <int BITS, int G>
__device__ inline void pt_quantize_slice(const uint16_t *row16, uint16_t *sc, uint16_t *zp, int slice, uint32_t (&codes)[16])
{
    constexpr float levels = (float)((1 << BITS) - 1);
    const uint4 a = reinterpret_cast<const uint4 *>(row16)[0], b = reinterpret_cast<const uint4 *>(row16)[1];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    float x[16];
#pragma unroll
    for (int i = 0; i < 8; i++) {
        x[2 * i] = pt_h2f((uint16_t)(w[i] & 0xffffu));
        x[2 * i + 1] = pt_h2f((uint16_t)(w[i] >> 16));
    }
    float mn = x[0], mx = x[0];
#pragma unroll
    for (int i = 1; i < 16; i++) { mn = fminf(mn, x[i]); mx = fmaxf(mx, x[i]); }
#pragma unroll
    for (int d = 1; d < G / 16; d <<= 1) {           // the G/16 threads of the group are neighbours in the wave
        mn = fminf(mn, __shfl_xor(mn, d));
        mx = fmaxf(mx, __shfl_xor(mx, d));
    }
    uint16_t sh, zh;
    float inv, zf;
    pt_group_params(mn, mx, levels, sh, zh, inv, zf);
    if ((slice & (G / 16 - 1)) == 0) { sc[slice / (G / 16)] = sh; zp[slice / (G / 16)] = zh; }
#pragma unroll
    for (int i = 0; i < 16; i++) codes[i] = pt_code(x[i], zf, inv, levels);
}

template <int BITS, int G>
__global__ __launch_bounds__(256) void quantize_pack_pt_kernel(PtQuantArgs a)
{
    constexpr int CPW = 32 / BITS, NG = kD / G;
    __shared__ uint8_t vcode[kPtBlockTok][kD + 4];     // V codes of the block, one byte each (row pitch 132)

    const int u = blockIdx.y, tid = threadIdx.x;
    int q0;
    const int n = pt_tokens_to_append(a, u, q0);
    const int i0 = blockIdx.x * kPtBlockTok;
    if (i0 >= n) return;
    const int nt = min(kPtBlockTok, n - i0);           // multiple of 16
    const int t0 = q0 + i0;

    const int slice = tid & 7;                         // 16-channel slice of the token
    for (int i = tid >> 3; i < nt; i += 32) {
        long row = a.idx ? (long)a.idx[(size_t)u * a.idx_stride + i0 + i] : (long)(i0 + i);
        row = row < 0 ? 0 : (row >= a.L ? a.L - 1 : row);
        const size_t src = ((size_t)u * a.L + row) * kD + slice * 16;
        const size_t meta = ((size_t)u * a.Tcap + (size_t)(t0 + i)) * NG;
        uint32_t codes[16];
        // keys: the codes of a token are contiguous, 16 codes = 16 * BITS / 32 words
        pt_quantize_slice<BITS, G>(a.K + src, a.Ks + meta, a.Kz + meta, slice, codes);
        uint32_t *kdst = a.Kc + ((size_t)u * a.Tcap + (size_t)(t0 + i)) * (kD / CPW) + slice * (16 / CPW);
#pragma unroll
        for (int wv = 0; wv < 16 / CPW; wv++) {
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < CPW; j++) word |= codes[wv * CPW + j] << (BITS * j);
            kdst[wv] = word;
        }
        // values: codes go through LDS, the words run along the tokens
        pt_quantize_slice<BITS, G>(a.V + src, a.Vs + meta, a.Vz + meta, slice, codes);
#pragma unroll
        for (int j = 0; j < 16; j++) vcode[i][slice * 16 + j] = (uint8_t)codes[j];
    }
    __syncthreads();
    uint32_t *vdst = a.Vc + (size_t)u * (size_t)(a.Tcap / CPW) * kD + (size_t)(t0 / CPW) * kD;
    for (int wi = tid; wi < (nt / CPW) * kD; wi += 256) {
        const int r = wi / kD, c = wi % kD;
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < CPW; j++) word |= (uint32_t)vcode[r * CPW + j][c] << (BITS * j);
        vdst[(size_t)r * kD + c] = word;
    }
}

__global__ void update_lengths_pt_kernel(PtQuantArgs a, int units)
{
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    int q0;
    const int n = pt_tokens_to_append(a, u, q0);
    if (n) a.q_len[u] = q0 + n;
}

// ------------------------------------------------------------------------------------------------ decode
struct PtDecArgs {
    const uint16_t *q;
    const uint32_t *Kc, *Vc;
    const uint16_t *Ks, *Kz, *Vs, *Vz;
    const int32_t *q_len;
    uint16_t *out;
    float *ws;                    // partials (nchunk > 1) [B*Hq][nchunk][kPartialStride]: m, l, 2 pad, o[128]
    float c1;                     // sm_scale * log2(e)
    int Hq, Hkv, rep, Tcap, chunk, nchunk;
};

// A 16-bit half of a packed word holds NF = 16 / BITS codes.  A code field moved to the top of its half's ten mantissa bits
// under the exponent of 2^BITS is the fp16 number 2^BITS + code: a shift and one v_and_or_b32 "convert" two codes, one per
// half, exactly, and every field's place counts the same, so that one accumulator takes them all and the other operand is
// used as it is.  (Two bits: neighbouring fields share a shift, the lower one is 16 + code.)  The constant is taken out by
// what the accumulator starts from: minus the sum of the other operand times it.  Masked in place, without the exponent,
// the fields are fp16 subnormals, at 4 bits half the shifts.  But a matrix instruction aligns its sum by the exponent field,
// 2^-14 for a subnormal, and cuts what is 24 bits below, always downwards; and the power of two that then belongs to a
// field's place has to go somewhere: with the weights it pushed those of small values below what fp16 holds, error
// 5e-4 -> 1.8e-3 at 4 bits on values of deviation 1/64.
typedef _Float16 pt_half8 __attribute__((ext_vector_type(8)));
typedef float pt_float4 __attribute__((ext_vector_type(4)));
template <int BITS> struct PtFields {
    static constexpr int CPW = 32 / BITS, NF = 16 / BITS, P = NF / 2;
    __device__ static constexpr int bit(int f) { return BITS == 2 && !(f & 1) ? 6 : 10 - BITS; }   // where field f goes
    // the fields of operand p are this + code
    __device__ static constexpr float base(int p) { return (float)(1 << (10 - bit(p))); }
    __device__ static uint32_t pair(uint32_t w, int f)   // field f of both halves
    {
        const int up = bit(f) - BITS * f;
        const uint32_t m = (((1u << BITS) - 1u) << bit(f)) * 0x00010001u;
        const uint32_t e = (uint32_t)(15 + 10 - bit(f)) * 0x04000400u;
        return ((up >= 0 ? w << up : w >> -up) & m) | e;
    }
    // operand p (0 .. P-1) from two words: codes p, NF+p, P+p, NF+P+p of each, in this order
    __device__ static pt_half8 operand(uint32_t w0, uint32_t w1, int p)
    {
        return __builtin_bit_cast(pt_half8, make_uint4(pair(w0, p), pair(w0, P + p), pair(w1, p), pair(w1, P + p)));
    }
    // code index (0 .. CPW-1) of half i (0..3) of a word's share of the operand
    __device__ static constexpr int code_at(int p, int i) { return p + (i & 1) * NF + (i >> 1) * P; }
};

// One workgroup = one (unit, chunk of tokens), all query heads of the unit; its four waves take blocks of TB tokens in
// turn, each with an online softmax of its own, and meet once at the end.  Both products run on 16x16x32 matrix
// instructions: scores with 16 tokens as rows and the query heads as columns, outputs with 16 channels as rows, the
// heads as columns and the tokens in between.  The order of the tokens inside a block is chosen so that the lane that
// gets a score is the lane that needs its weight as an operand, and the order of channels so that codes are loaded
// 128 bits at a time.  Column n of a score product holds head n % REPT and, where a token has several channel groups,
// only group (n / REPT) % NG of it (the query is zero elsewhere), so that every group meets its own scale; the groups
// are added across lanes afterwards.
// What bounds it: memory (136 bytes per token at 4 bits with one group) and, nearly as much, the vector instructions that
// make operands of codes and weights; a form with one dot2 per pair of codes and head was bound by those alone.  Calls of
// 128 units x 13088 tokens, 4 heads each, G = 128: 4 bits 79 -> 52 us (4.4 TB/s; a plain copy reaches 5.0), 2 bits
// 82 -> 46.5, 8 bits 110 -> 83; 16 units 23 -> 16 us; G = 32, 128 units x 8192 tokens 63 -> 41 us.
// STREAM: code words, read once per call, are loaded with the streaming hint (see pt_streams()).
typedef uint32_t pt_word2 __attribute__((ext_vector_type(2)));
typedef uint32_t pt_word4 __attribute__((ext_vector_type(4)));
template <bool STREAM, class T> __device__ __forceinline__ T pt_load(const T *p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    return *p;
}
template <int BITS, int G, int REPT, bool STREAM>
__global__ __launch_bounds__(256, 2) void decode_pt_kernel(PtDecArgs a)
{
    typedef PtFields<BITS> F;
    constexpr int CPW = F::CPW, P = F::P, NG = kD / G, W = kD / CPW;
    constexpr int KW = W / 4;                            // key words of one lane and token: 32 channels
    constexpr int TB = 8 * CPW, NT = TB / 16;            // tokens of a block, score tiles of a block
    constexpr int NS = NG * REPT > 16 ? 2 : 1;           // column sets of a score product
    constexpr int NB = NG == 1 ? 1 : 2;                  // weight operands: the channel halves may differ in scale
    constexpr int E = TB * NG / 64 ? TB * NG / 64 : 1;   // scales of a block and array that one lane loads
    constexpr bool HINT_K = STREAM && KW <= 4;           // (see pt_streams())
    __shared__ __align__(16) _Float16 meta[4][4][NG][TB];                  // wave; Ks, Kz, Vs, Vz; group; token
    __shared__ float part_o[4][REPT][kD], part_m[4][REPT], part_l[4][REPT], zsum[4][NG][REPT];

    const int u = blockIdx.y, ch = blockIdx.x, tid = threadIdx.x, lane = tid & 63, rep = a.rep;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kg = lane >> 4, h = col % REPT;
    const int b = u / a.Hkv, kvh = u % a.Hkv;
    const int bq0 = b * a.Hq + kvh * rep;
    const int T = min(max(a.q_len[u], 0), a.Tcap);
    const int t_begin = ch * a.chunk, t_end = min(T, t_begin + a.chunk);
    if (t_begin >= t_end && a.nchunk > 1) return;       // the merge kernel skips this slot

    const uint32_t *Kc = a.Kc + (size_t)u * a.Tcap * W;
    const uint32_t *Vc = a.Vc + (size_t)u * (size_t)(a.Tcap / CPW) * kD;
    const uint16_t *mt[4] = {a.Ks + (size_t)u * a.Tcap * NG, a.Kz + (size_t)u * a.Tcap * NG,
                             a.Vs + (size_t)u * a.Tcap * NG, a.Vz + (size_t)u * a.Tcap * NG};

    // requests of a block, made one block ahead (addresses stay inside the buffers; what lies past t_end is masked)
    uint32_t kw[NT][KW];
    pt_word4 vw[2][2];                                     // [half of the channels][s]: words of tokens CPW (kg + 4 s) ..
    uint16_t mr[4][E];
    auto request = [&](int t0) {
#pragma unroll
        for (int tau = 0; tau < NT; tau++) {
            const int s = tau / (CPW / 4), q4 = tau % (CPW / 4);
            const int t = min(t0 + CPW * (col >> 2) + 4 * CPW * s + 4 * q4 + (col & 3), a.Tcap - 1);
            const uint32_t *src = Kc + (size_t)t * W + kg * KW;
            if constexpr (KW == 2) {
                const pt_word2 v = pt_load<HINT_K>(reinterpret_cast<const pt_word2 *>(src));
                kw[tau][0] = v.x, kw[tau][1] = v.y;
            } else {
#pragma unroll
                for (int i = 0; i < KW / 4; i++) {
                    const pt_word4 v = pt_load<HINT_K>(reinterpret_cast<const pt_word4 *>(src) + i);
                    kw[tau][4 * i] = v.x, kw[tau][4 * i + 1] = v.y, kw[tau][4 * i + 2] = v.z, kw[tau][4 * i + 3] = v.w;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 2; s++) {
            const int row = min(t0 / CPW + kg + 4 * s, a.Tcap / CPW - 1);
#pragma unroll
            for (int half = 0; half < 2; half++)
                vw[half][s] = pt_load<STREAM>(reinterpret_cast<const pt_word4 *>(Vc + (size_t)row * kD + half * 64 + col * 4));
        }
        const int e0 = min(t0 * NG + lane * E, a.Tcap * NG - E);
#pragma unroll
        for (int k = 0; k < 4; k++) __builtin_memcpy(mr[k], __builtin_assume_aligned(mt[k] + e0, 2 * E), 2 * E);
    };

    const int t_first = t_begin + wave * TB;
    if (t_first < t_end) request(t_first);

    // the query as operand: [column set][pair of words][position]; heads beyond rep repeat the last one, unused
    pt_half8 qb[NS][KW / 2][P];
    float qz[NS], minus_q[NS];                          // sum of the query over the column's group; minus that of its bases
    {
        const _Float16 *qr = reinterpret_cast<const _Float16 *>(a.q) + (size_t)(bq0 + min(h, rep - 1)) * kD + kg * 32;
        pt_half8 qv[4];
#pragma unroll
        for (int i = 0; i < 4; i++) qv[i] = reinterpret_cast<const pt_half8 *>(qr)[i];
        float sum = 0.f, based = 0.f;
#pragma unroll
        for (int c = 0; c < 32; c++) {
            sum += (float)qv[c >> 3][c & 7];
            based = __builtin_fmaf((float)qv[c >> 3][c & 7], F::base(c % CPW % P), based);
        }
#pragma unroll
        for (int ns = 0; ns < NS; ns++) {
            const bool mine = kg * 32 / G == ((ns * 16 + col) / REPT) % NG;
#pragma unroll
            for (int wp = 0; wp < KW / 2; wp++)
#pragma unroll
                for (int p = 0; p < P; p++)
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        const int c = (2 * wp + (i >> 2)) * CPW + F::code_at(p, i & 3);
                        qb[ns][wp][p][i] = mine ? qv[c >> 3][c & 7] : (_Float16)0;
                    }
            qz[ns] = mine ? sum : 0.f;
            qz[ns] += __shfl_xor(qz[ns], 16);
            qz[ns] += __shfl_xor(qz[ns], 32);
            minus_q[ns] = mine ? -based : 0.f;
            minus_q[ns] += __shfl_xor(minus_q[ns], 16);
            minus_q[ns] += __shfl_xor(minus_q[ns], 32);
        }
    }

    float m = -1e30f, l = 0.f, pz[NS];
    pt_float4 o[2][4];                                  // o[half][i][j]: channel 64 half + 4 (4 kg + j) + i of head h
#pragma unroll
    for (int ns = 0; ns < NS; ns++) pz[ns] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; i++) o[i >> 2][i & 3] = pt_float4{0.f, 0.f, 0.f, 0.f};

    for (int t0 = t_first; t0 < t_end; t0 += 4 * TB) {
        // ---- scales and zero-points to LDS by (group, token); zero past the end
        if (TB * NG >= 64 || lane < TB * NG) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                const int t = (lane * E + e) / NG, g = (lane * E + e) % NG;
                const bool in = t0 + t < t_end;
#pragma unroll
                for (int k = 0; k < 4; k++) meta[wave][k][g][t] = __builtin_bit_cast(_Float16, in ? mr[k][e] : (uint16_t)0);
            }
        }
        asm volatile("" ::: "memory");                  // (one wave: LDS operations stay in order)
        __builtin_amdgcn_wave_barrier();
        // the four tokens of lane kg in tile tau start here
        auto at = [&](int tau) { return CPW * kg + 4 * CPW * (tau / (CPW / 4)) + 4 * (tau % (CPW / 4)); };
        typedef _Float16 h4 __attribute__((ext_vector_type(4)));

        // ---- scores
        float s[NT][4];
#pragma unroll
        for (int tau = 0; tau < NT; tau++) {
#pragma unroll
            for (int j = 0; j < 4; j++) s[tau][j] = 0.f;
#pragma unroll
            for (int ns = 0; ns < NS; ns++) {
                pt_float4 acc = {minus_q[ns], minus_q[ns], minus_q[ns], minus_q[ns]};
#pragma unroll
                for (int p = 0; p < P; p++)
#pragma unroll
                    for (int wp = 0; wp < KW / 2; wp++)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(F::operand(kw[tau][2 * wp], kw[tau][2 * wp + 1], p),
                                                                     qb[ns][wp][p], acc, 0, 0, 0);
                const int g = ((ns * 16 + col) / REPT) % NG;
                const h4 ks = *reinterpret_cast<const h4 *>(&meta[wave][0][g][at(tau)]);
                const h4 kz = *reinterpret_cast<const h4 *>(&meta[wave][1][g][at(tau)]);
#pragma unroll
                for (int j = 0; j < 4; j++)
                    s[tau][j] += __builtin_fmaf((float)ks[j], acc[j], (float)kz[j] * qz[ns]);
            }
#pragma unroll
            for (int d = REPT; d < (NG * REPT > 16 ? 16 : NG * REPT); d <<= 1)       // the other groups of the token
#pragma unroll
                for (int j = 0; j < 4; j++) s[tau][j] += __shfl_xor(s[tau][j], d);
            if (NT == 8)                                 // (all tiles' operands at once do not fit the registers)
                asm volatile("" : "+v"(s[tau][0]), "+v"(s[tau][1]), "+v"(s[tau][2]), "+v"(s[tau][3])::"memory");
        }
        pt_word4 vc[2][2];
#pragma unroll
        for (int i = 0; i < 4; i++) vc[i >> 1][i & 1] = vw[i >> 1][i & 1];
        if (t0 + 4 * TB < t_end) request(t0 + 4 * TB);
        // ---- online softmax over the block (base-2 domain)
        const bool whole = t0 + TB <= t_end;
        float bm = m;
#pragma unroll
        for (int tau = 0; tau < NT; tau++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                s[tau][j] *= a.c1;
                if (!whole && t0 + at(tau) + j >= t_end) s[tau][j] = -INFINITY;
                bm = fmaxf(bm, s[tau][j]);
            }
        bm = fmaxf(bm, __shfl_xor(bm, 16));
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const float alpha = __builtin_amdgcn_exp2f(m - bm);
        m = bm;
        if (__any(alpha != 1.0f)) {
#pragma unroll
            for (int i = 0; i < 8; i++) o[i >> 2][i & 3] *= alpha;
        }
        float sum = 0.f;
        pt_half8 wb[NB][P];                              // weights times V scale, in the order of the value operands
#pragma unroll
        for (int ns = 0; ns < NS; ns++) pz[ns] *= alpha;
#pragma unroll
        for (int tau = 0; tau < NT; tau++) {
            const h4 vsA = *reinterpret_cast<const h4 *>(&meta[wave][2][NG == 4 ? (col / REPT) & 1 : 0][at(tau)]);
            h4 vsB = vsA;
            if constexpr (NB == 2)
                vsB = *reinterpret_cast<const h4 *>(&meta[wave][2][NG == 4 ? 2 + ((col / REPT) & 1) : 1][at(tau)]);
            float w[4];
#pragma unroll
            for (int j = 0; j < 4; j++) sum += w[j] = __builtin_amdgcn_exp2f(s[tau][j] - m);
#pragma unroll
            for (int ns = 0; ns < NS; ns++) {
                const h4 vz = *reinterpret_cast<const h4 *>(&meta[wave][3][((ns * 16 + col) / REPT) % NG][at(tau)]);
#pragma unroll
                for (int j = 0; j < 4; j++) pz[ns] = __builtin_fmaf(w[j], (float)vz[j], pz[ns]);
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int sw = tau / (CPW / 4), e = 4 * (tau % (CPW / 4)) + j;       // code e of word sw
                const int hi = e / F::NF, up = (e % F::NF) / P, p = e % P;
                const int at_op = sw * 4 + up * 2 + hi;
                wb[0][p][at_op] = (_Float16)(w[j] * (float)vsA[j]);
                if constexpr (NB == 2) wb[NB - 1][p][at_op] = (_Float16)(w[j] * (float)vsB[j]);
            }
        }
        l = __builtin_fmaf(l, alpha, sum);
        // ---- weighted values: 16 channels a tile, from minus the sum of the (rounded) weights times the codes' bases
        pt_float4 minus[NB];
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
            minus[nb] = pt_float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < P; p++) {
                const _Float16 n = (_Float16)-F::base(p);
                minus[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pt_half8{n, n, n, n, n, n, n, n}, wb[nb][p], minus[nb], 0, 0, 0);
            }
        }
#pragma unroll
        for (int half = 0; half < 2; half++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const pt_word4 q0 = vc[half][0], q1 = vc[half][1];
                const uint32_t w0 = i == 0 ? q0.x : i == 1 ? q0.y : i == 2 ? q0.z : q0.w;
                const uint32_t w1 = i == 0 ? q1.x : i == 1 ? q1.y : i == 2 ? q1.z : q1.w;
                pt_float4 acc = minus[NB == 2 ? half : 0];
#pragma unroll
                for (int p = 0; p < P; p++)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(F::operand(w0, w1, p), wb[NB == 2 ? half : 0][p], acc, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; j++) o[half][i][j] += acc[j];
                if (NT == 8) asm volatile("" : "+v"(o[half][i])::"memory");
            }
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    }

    // ---- the four waves' parts meet
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
#pragma unroll
    for (int ns = 0; ns < NS; ns++) {
        pz[ns] += __shfl_xor(pz[ns], 16);
        pz[ns] += __shfl_xor(pz[ns], 32);
        if (kg == 0) zsum[wave][((ns * 16 + col) / REPT) % NG][h] = pz[ns];          // (equal columns write equal values)
    }
    // with four groups a column of the value product is right for the channels of its own group parity only
    if (NG == 4 ? (col < 2 * REPT && col / REPT == kg >> 1) : col < REPT) {
#pragma unroll
        for (int half = 0; half < 2; half++)
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 4; j++) part_o[wave][h][64 * half + 4 * (4 * kg + j) + i] = o[half][i][j];
    }
    if (lane < REPT) part_m[wave][lane] = m, part_l[wave][lane] = l;
    __syncthreads();
    const int c = tid & (kD - 1);
    for (int hh = tid >> 7; hh < rep; hh += 2) {
        float M = part_m[0][hh];
#pragma unroll
        for (int w = 1; w < 4; w++) M = fmaxf(M, part_m[w][hh]);
        float Ls = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < 4; w++) {
            const float e = __builtin_amdgcn_exp2f(part_m[w][hh] - M);
            Ls = __builtin_fmaf(part_l[w][hh], e, Ls);
            O = __builtin_fmaf(part_o[w][hh][c] + zsum[w][c / G][hh], e, O);
        }
        if (a.nchunk == 1) {
            a.out[(size_t)(bq0 + hh) * kD + c] = __half_as_ushort(__float2half_rn(Ls > 0.f ? O / Ls : 0.f));
        } else {
            float *pp = a.ws + ((size_t)(bq0 + hh) * a.nchunk + ch) * kPartialStride;
            pp[4 + c] = O;
            if (c == 0) pp[0] = M, pp[1] = Ls;
        }
    }
}

// One workgroup of 128 threads per query row: combine the partials of the chunks that hold tokens.  Eight
// chunks at a time, all their loads requested before the first is used; the running maximum is carried from
// batch to batch (online, like the kernel above).
__global__ __launch_bounds__(128) void merge_pt_kernel(PtDecArgs a)
{
    const int bq = blockIdx.x, c = threadIdx.x;
    const int u = (bq / a.Hq) * a.Hkv + (bq % a.Hq) / a.rep;
    const float *base = a.ws + (size_t)bq * a.nchunk * kPartialStride;
    float pm[8], pl[8], po[8];
    // (the first batch is requested before the unit's length is known: slots beyond it are ignored below)
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const float *p = base + (size_t)min(j, a.nchunk - 1) * kPartialStride;
        pm[j] = p[0], pl[j] = p[1], po[j] = p[4 + c];
    }
    const int T = min(max(a.q_len[u], 0), a.Tcap);
    const int nq = (T + a.chunk - 1) / a.chunk;
    float M = -1e30f, L = 0.f, O = 0.f;
    for (int c0 = 0; c0 < nq; c0 += 8) {
        if (c0) {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float *p = base + (size_t)min(c0 + j, nq - 1) * kPartialStride;
                pm[j] = p[0], pl[j] = p[1], po[j] = p[4 + c];
            }
        }
        float bm = M;
#pragma unroll
        for (int j = 0; j < 8; j++) bm = c0 + j < nq ? fmaxf(bm, pm[j]) : bm;
        const float sc = exp2f(M - bm);
        L *= sc, O *= sc, M = bm;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const bool in = c0 + j < nq;                   // (a slot beyond the unit's chunks holds anything, NaN included)
            const float w = exp2f(pm[j] - M);
            L = in ? __builtin_fmaf(pl[j], w, L) : L;
            O = in ? __builtin_fmaf(po[j], w, O) : O;
        }
    }
    a.out[(size_t)bq * kD + c] = __half_as_ushort(__float2half_rn(L > 0.f ? O / L : 0.f));
}

static int pt_validate_shape(const minikv_pt_shape *s)
{
    if (!s) return MINIKV_EINVAL;
    if (s->D != kD) return MINIKV_EUNSUPPORTED;
    if (!(s->G == 32 || s->G == 64 || s->G == 128)) return MINIKV_EUNSUPPORTED;
    if (!(s->bits == 2 || s->bits == 4 || s->bits == 8)) return MINIKV_EUNSUPPORTED;
    if (s->B <= 0 || s->Hq <= 0 || s->Hkv <= 0 || s->Hq % s->Hkv) return MINIKV_EINVAL;
    if (s->Hq / s->Hkv > kPtMaxRep) return MINIKV_EUNSUPPORTED;
    if (s->Tcap <= 0 || s->Tcap % 64) return MINIKV_EINVAL;
    if ((int64_t)s->B * s->Hkv > 65535) return MINIKV_EINVAL;
    return MINIKV_OK;
}

static int pt_validate_cache(const minikv_pt_cache *c)
{
    if (!c) return MINIKV_EINVAL;
    if (!aligned16(c->Kc) || !aligned16(c->Ks) || !aligned16(c->Kz) || !aligned16(c->Vc) || !aligned16(c->Vs) ||
        !aligned16(c->Vz) || !c->q_len)
        return MINIKV_EINVAL;
    return MINIKV_OK;
}

// Chunks per unit the workspace is sized for.
static int pt_ws_chunks(const minikv_pt_shape &s)
{
    const long units = (long)s.B * s.Hkv;
    int chunk = kPtMinChunk;
    while (chunk < 8192 && units * ((s.Tcap + 2 * chunk - 1) / (2 * chunk)) >= 1024) chunk *= 2;
    return (s.Tcap + chunk - 1) / chunk;
}

// Token chunk of one decode workgroup: a multiple of 256 tokens, as few chunks as keep kPtTargetWgs workgroups in the
// launch -- the two per compute unit that the registers allow, so that all run at once and each sets up its query operands
// once (1024: 49.7 instead of 44.7 us on 128 units x 13088 tokens, 38 instead of 32 on 16 x 65536) -- and never more
// chunks than the workspace holds (a unit's share of 1024 workgroups).
// One chunk a unit, and with it no merge launch, where splitting saves less than that costs: up to 512 tokens (at 2 bits one round
// of the four waves' blocks: 24 units 10.4 -> 8.3 us, 192 units 12.3 -> 8.1, 1024 tokens 10.4 against 12.6; at 4 bits two, G = 128
// 7.9 -> 7.3, but G = 32 8.5 against 8.6 and with 8 units 8.0 against 8.3; at 8 bits four, 9.2 against 9.6), and up to 1536 on
// more than 170 units, which could have two (192 units, G = 32, 1024 tokens: 2 bits 15.0 -> 13.6, 4 bits 15.9 -> 14.5, 8 bits 18.8 ->
// 15.9; 1536 tokens 21.2 -> 18.2, 20.2 -> 19.1, 21.8 -> 21.4; 2048 21.4 against 22.5, 23.5 against 23.6, 26.5 against 27.2).
constexpr int kPtTargetWgs = 512;
static int pt_chunk(const minikv_pt_shape &s)
{
    const long units = (long)s.B * s.Hkv;
    const long most = kPtTargetWgs / units > 1 ? kPtTargetWgs / units : 1;
    const long blocks = ((long)s.Tcap + kPtMinChunk - 1) / kPtMinChunk;
    const int whole = most <= 2 ? 1536 : s.bits == 2 || (s.bits == 4 && s.G == kD) ? 512 : 0;     // most tokens in one chunk
    if (s.Tcap <= whole) return (int)blocks * kPtMinChunk;
    return (int)((blocks + most - 1) / most) * kPtMinChunk;
}

template <int BITS>
static int pt_launch_quantize(const PtQuantArgs &a, int G, dim3 grid, int units, hipStream_t st)
{
    switch (G) {
    case 32: hipLaunchKernelGGL((quantize_pack_pt_kernel<BITS, 32>), grid, dim3(256), 0, st, a); break;
    case 64: hipLaunchKernelGGL((quantize_pack_pt_kernel<BITS, 64>), grid, dim3(256), 0, st, a); break;
    case 128: hipLaunchKernelGGL((quantize_pack_pt_kernel<BITS, 128>), grid, dim3(256), 0, st, a); break;
    default: return MINIKV_EUNSUPPORTED;
    }
    hipLaunchKernelGGL(update_lengths_pt_kernel, dim3((units + 255) / 256), dim3(256), 0, st, a, units);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

// Whether a call loads its codes with the streaming hint: where the packed cache (by its capacity) is larger than three
// eighths of the 256 MB memory-side cache.  128 units x 13088 tokens at 4 bits (228 MB) 51.7 -> 49.9 us, 8 bits x 8192
// (272 MB) 55.6 -> 50.7, 104 MB 28.7 -> 28.0; what is smaller may still be cached from the call before (three caches in
// turn, 84 MB 21.8 against 22.3, 36 .. 80 MB a tie).  A cache that is larger than what it holds is judged by its capacity all
// the same: 60 MB in 240, ten such caches in turn, 50.4 -> 49.8 us (three in turn 49.4 -> 49.5).  Not with the hint on the keys
// at 8 bits: there a lane's 32 bytes of a key are two loads, half of every sector each, and a sector that the first has marked as
// used up comes from memory again for the second where few waves run (120 MB in 240: 38.2 us without a hint, 42.7 with it on
// both, 36.7 on the values only; full caches of 120 and 250 MB 28.7, 28.3, 25.8 and 51.9, 49.5, 47.7).
static bool pt_streams(const PtDecArgs &a, int bits, int G, unsigned units)
{
    return (long)units * a.Tcap * (2 * (kD * bits / 8 + 4 * kD / G)) > (96L << 20);
}

template <int BITS, int REPT, bool STREAM>
static int pt_launch_decode_g(const PtDecArgs &a, int G, dim3 grid, hipStream_t st)
{
    switch (G) {
    case 32: hipLaunchKernelGGL((decode_pt_kernel<BITS, 32, REPT, STREAM>), grid, dim3(256), 0, st, a); break;
    case 64: hipLaunchKernelGGL((decode_pt_kernel<BITS, 64, REPT, STREAM>), grid, dim3(256), 0, st, a); break;
    case 128: hipLaunchKernelGGL((decode_pt_kernel<BITS, 128, REPT, STREAM>), grid, dim3(256), 0, st, a); break;
    default: return MINIKV_EUNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

// heads per unit rounded up to 1, 2, 4 or 8 (the spare ones repeat the last head and are not written)
template <int BITS, bool STREAM>
static int pt_launch_decode_s(const PtDecArgs &a, int G, dim3 grid, hipStream_t st)
{
    if (a.rep <= 1) return pt_launch_decode_g<BITS, 1, STREAM>(a, G, grid, st);
    if (a.rep <= 2) return pt_launch_decode_g<BITS, 2, STREAM>(a, G, grid, st);
    if (a.rep <= 4) return pt_launch_decode_g<BITS, 4, STREAM>(a, G, grid, st);
    return pt_launch_decode_g<BITS, 8, STREAM>(a, G, grid, st);
}
template <int BITS>
static int pt_launch_decode(const PtDecArgs &a, int G, dim3 grid, hipStream_t st)
{
    return pt_streams(a, BITS, G, grid.y) ? pt_launch_decode_s<BITS, true>(a, G, grid, st) : pt_launch_decode_s<BITS, false>(a, G, grid, st);
}

}  // namespace minikv

using namespace minikv;

extern "C" {

size_t minikv_pt_cache_bytes(const minikv_pt_shape *s, int which)
{
    if (pt_validate_shape(s) != MINIKV_OK) return 0;
    const size_t U = (size_t)s->B * s->Hkv;
    switch (which) {
    case MINIKV_BUF_KC:
    case MINIKV_BUF_VC: return U * (size_t)s->Tcap * (size_t)(kD * s->bits / 8);
    case MINIKV_BUF_KS:
    case MINIKV_BUF_KZ:
    case MINIKV_BUF_VS:
    case MINIKV_BUF_VZ: return U * (size_t)s->Tcap * (size_t)(kD / s->G) * 2;
    case MINIKV_BUF_QLEN: return U * 4;
    default: return 0;
    }
}

size_t minikv_pt_workspace_bytes(const minikv_pt_shape *s)
{
    if (pt_validate_shape(s) != MINIKV_OK) return 0;
    return (size_t)s->B * s->Hq * (size_t)pt_ws_chunks(*s) * kPartialStride * sizeof(float);
}

int kv_quantize_pack_pt(const minikv_pt_shape *s, const minikv_f16 *K, const minikv_f16 *V, int64_t L,
                        const int32_t *idx, int64_t idx_stride, const int32_t *n_tok, int32_t max_tok,
                        minikv_pt_cache *c, void *stream)
{
    int rc = pt_validate_shape(s);
    if (rc) return rc;
    if ((rc = pt_validate_cache(c))) return rc;
    if (!aligned16(K) || !aligned16(V) || !n_tok || L <= 0) return MINIKV_EINVAL;
    if (max_tok < 0 || max_tok % 16 || max_tok > s->Tcap || max_tok > L) return MINIKV_EINVAL;
    if (idx && idx_stride < max_tok) return MINIKV_EINVAL;
    if (max_tok == 0) return MINIKV_OK;
    PtQuantArgs a;
    a.K = K; a.V = V; a.idx = idx; a.n_tok = n_tok;
    a.Kc = c->Kc; a.Vc = c->Vc; a.Ks = c->Ks; a.Kz = c->Kz; a.Vs = c->Vs; a.Vz = c->Vz; a.q_len = c->q_len;
    a.L = L; a.idx_stride = idx_stride; a.Tcap = s->Tcap; a.max_tok = max_tok;
    const int units = s->B * s->Hkv;
    const dim3 grid((max_tok + kPtBlockTok - 1) / kPtBlockTok, units);
    switch (s->bits) {
    case 2: return pt_launch_quantize<2>(a, s->G, grid, units, (hipStream_t)stream);
    case 4: return pt_launch_quantize<4>(a, s->G, grid, units, (hipStream_t)stream);
    case 8: return pt_launch_quantize<8>(a, s->G, grid, units, (hipStream_t)stream);
    }
    return MINIKV_EUNSUPPORTED;
}

int minikv_decode_attn_pt(const minikv_pt_shape *s, const minikv_f16 *q, const minikv_pt_cache *c, float sm_scale,
                          minikv_f16 *out, void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = pt_validate_shape(s);
    if (rc) return rc;
    if ((rc = pt_validate_cache(c))) return rc;
    if (!aligned16(q) || !aligned16(out) || !aligned16(workspace)) return MINIKV_EINVAL;
    if (!(sm_scale == sm_scale) || sm_scale - sm_scale != 0.0f) return MINIKV_EINVAL;
    if (workspace_bytes < minikv_pt_workspace_bytes(s)) return MINIKV_EWORKSPACE;
    PtDecArgs a;
    a.q = q; a.Kc = c->Kc; a.Vc = c->Vc; a.Ks = c->Ks; a.Kz = c->Kz; a.Vs = c->Vs; a.Vz = c->Vz; a.q_len = c->q_len;
    a.out = out;
    a.ws = reinterpret_cast<float *>(workspace);
    a.c1 = sm_scale * 1.44269504088896340736f;
    a.Hq = s->Hq; a.Hkv = s->Hkv; a.rep = s->Hq / s->Hkv; a.Tcap = s->Tcap;
    a.chunk = pt_chunk(*s);
    a.nchunk = (s->Tcap + a.chunk - 1) / a.chunk;
    const dim3 grid(a.nchunk, s->B * s->Hkv);
    switch (s->bits) {
    case 2: rc = pt_launch_decode<2>(a, s->G, grid, (hipStream_t)stream); break;
    case 4: rc = pt_launch_decode<4>(a, s->G, grid, (hipStream_t)stream); break;
    case 8: rc = pt_launch_decode<8>(a, s->G, grid, (hipStream_t)stream); break;
    default: return MINIKV_EUNSUPPORTED;
    }
    if (rc || a.nchunk == 1) return rc;                 // (a single chunk is the result)
    hipLaunchKernelGGL(merge_pt_kernel, dim3(s->B * s->Hq), dim3(128), 0, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
}

}  // extern "C"
