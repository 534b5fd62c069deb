// Prefill attention that also returns the cumulative attention score of every prompt token, in memory linear
// in the prompt length (Section 3.2; Algorithm 1 line 2): X_O = softmax(sm_scale Q K^T) V on the causal part,
// LSE per query row, A_cumul = column sums of the softmax matrix.
//
// Two kernels, as in Section 3.2, re-tiled for 64-lane waves and the 32x32x16 fp16 matrix instruction:
//   prefill_fwd_kernel     row blocks in parallel.  A workgroup owns 32 queries per wave and walks the keys in tiles
//                          of 64 through LDS.  Scores are computed TRANSPOSED, S^T = K Q^T, so that a lane holds one
//                          query column: the running max / sum of the online softmax are per-lane scalars (one
//                          exchange between the two half-waves per tile), the rescale of the output is a per-lane
//                          multiply, and the fp32 scores, once turned into fp16 weights, ARE the B operand of
//                          O^T = V^T P^T without any shuffle (the key order inside a 16-key step is whatever the
//                          accumulator layout gives; the V^T operand is read in the same order).
//   prefill_colsum_kernel  column blocks in parallel.  A workgroup owns 128 or 64 keys (their K rows held in registers as
//                          the B operand), walks the queries from the diagonal down in tiles of 64 or 128 through LDS,
//                          recomputes S = Q K^T, normalises with the saved LSE and adds the weights of its key column
//                          in the lane: no atomics, one exchange at the end.
// A prompt of at most 128 tokens is one row block: its workgroup of the first kernel forms the column sums as well.
#include "common.h"

#include <type_traits>

namespace minikv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kPfD = 128;            // head dimension
constexpr int kPfN = 64;             // keys (forward) / queries (column sums) per LDS tile
constexpr int kWaitVm0 = 0x0F70;      // s_waitcnt vmcnt(0), other counters untouched
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct PrefillArgs {
    const _Float16 *Q, *K, *V;
    _Float16 *XO;
    float *lse, *A_cumul;
    int Hq, rep, nblk;
    long L;
    float scale_log2;                // sm_scale * log2(e): the softmax runs on powers of two
};

__device__ __forceinline__ float16v mfma32(half8 a, half8 b, float16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Row of accumulator element i (0..15) inside a 32x32 result tile, for a lane of half-wave g.
__device__ __forceinline__ int acc_row(int i, int g) { return (i >> 2) * 8 + g * 4 + (i & 3); }

// 64 lanes x 16 bytes from base + off (per lane) straight to LDS at lds + 16 * lane: no registers and no LDS store
// instructions in between.  The compiler does not count this load: wait with s_waitcnt vmcnt before the barrier that
// hands the data over.  (m0, which it sets, is a register the compiler reserves and holds no value in from one statement to
// the next -- it refuses it as a clobber --, and nothing else in this file reads it.)
__device__ __forceinline__ void load_to_lds(const void *base, unsigned off, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds), "v"(off), "s"(base)
                 : "memory");
}
__device__ __forceinline__ unsigned lds_offset(const void *p)
{
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
// Tiles loaded this way have unpadded rows of 256 bytes; chunk k (16 bytes) of row r sits at place k ^ (r & 15), so
// that the fragment reads of 32 consecutive rows use all banks evenly.
__device__ __forceinline__ int tile_place(int row, int chunk) { return row * kPfD + ((chunk ^ (row & 15)) << 3); }

// A workgroup of WAVES waves owns 32 queries per wave (their Q rows in registers) and walks the keys in tiles of 64.
// Scores are computed TRANSPOSED, S^T = K Q^T, so that a lane holds one query column (see the top of the file).  One
// step of the loop, for tile n, is one instruction stream of two halves:
//   first   the 16 score products of tile n+1, between them the weights of the first 48 keys of tile n
//   second  the 16 output products of tile n, between them the weights of the last 16 keys and the maximum of the
//           scores of tile n+1
// so that the matrix unit and the vector unit of a SIMD work at the same time whatever the other wave does.  One
// barrier per step, between the halves: there tile n's V and tile n+2's K are in place, tile n+1's K has been read.
// K and V tiles go straight to LDS from their own row-major layout; the output product's A operand V^T is read with
// the transposing LDS read.
// What bounds it: the energy of the products (the clock falls to 1.55-1.8 GHz on N(0,1) data with the matrix unit 60 % busy;
// 2.4 GHz on zeros).  So what moves data was taken out: no staging of tiles through registers and LDS stores, no
// transposed copy of V in memory.  32 heads x 32768 tokens 9.7 -> 8.4 ms (1.05 PFLOP/s; a plain library product of
// 16384^3 reaches 1.29 on this card), 2 x 32 x 4096 364 -> 320 us, 32 x 777 26.7 -> 19.9 us.  Letting the reference of the
// weights lag behind the running maximum (fewer rescales) is another 2-3 %, but then the key that dominates a row no
// longer has the weight 1 that fp16 holds exactly, and the error grows by 1 %.
constexpr int kPfTile = kPfN * kPfD;                    // halves of one unpadded tile in LDS

// Place (in halves) of 16-byte chunk k of row `key` in a V tile: the rows 4j .. 4j+3 that one transposing read takes
// fall on different banks.
__device__ __forceinline__ int v_swizzle(int key) { return 4 * (key & 3) + 2 * ((key >> 1) & 1); }

typedef __fp16 fp16x4 __attribute__((__vector_size__(8)));
__device__ __forceinline__ half4 read_transposed(const _Float16 *p)
{
    return (half4)__builtin_amdgcn_ds_read_tr16_b64_v4f16((__attribute__((address_space(3))) fp16x4 *)p);
}

// SPLIT == 2: two sets of WAVES waves take the even and the odd tiles of the same queries, each through LDS buffers of
// its own, and meet at the end; for launches that leave a compute unit a single set.  The launch gives the LDS: where the
// compiler knows that 128 KB leave room for one workgroup, it spreads two sets of two waves over the registers of two
// waves per SIMD, half of them reachable for matrix instructions only, and moves 160 registers per tile (3700 cycles a
// tile, 2400 without; 8 heads x 2048 32.2 -> 26.3 us).  With the second launch bound no instance has a register of that
// kind, nor a private segment.
//
// BUF == 1: one K and one V buffer per set instead of two, so that a compute unit has room for two workgroups of two sets.
// K tile n+2 is requested between the halves and V tile n+1 at the end of step n, each into the buffer that has just been
// read, at a second barrier; what a wave then waits the other workgroup's wave of its SIMD fills.
//
// SCORES: the prompt is one row block, whose workgroup then has every row's LSE and returns the column sums as well: the
// scores once more, as S = Q K^T with the Q rows it still holds, so that a lane adds up one key's weights; the waves' sums
// meet in LDS.  What bounds short prompts is the launch and its two round trips to memory, and a second one repeats them:
// 8 heads x 48 tokens 9.8 -> 6.7 us, 8 x 128 13.3 -> 10.2, 1024 x 64 26.7 -> 21.4, 2048 x 128 95.6 -> 71.7.
constexpr unsigned fwd_lds_bytes(int split, int buffers, int scored_queries = 0)
{
    return split * 2 * buffers * kPfTile * sizeof(_Float16) + scored_queries * (1 + scored_queries / 32) * sizeof(float);
}

template <int WAVES, int SPLIT, int BUF, bool SCORES>
__global__ __launch_bounds__(64 * WAVES * SPLIT, 2) void prefill_fwd_kernel(PrefillArgs a)
{
    constexpr int kRows = kPfN / WAVES, kLoads = kRows / 4;     // rows of a tile one wave loads, four per instruction
    extern __shared__ __align__(16) _Float16 tiles[];

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % WAVES;
    const int set = SPLIT == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / WAVES;
    _Float16 *Ks = tiles + set * 2 * BUF * kPfTile, *Vs = Ks + BUF * kPfTile;
    // heaviest row blocks (the last ones: they see the most keys) first
    const int nbh = (int)gridDim.x / a.nblk, head = (int)blockIdx.x % nbh;
    const int qb = a.nblk - 1 - (int)blockIdx.x / nbh;
    const long bh = head, kvh = (head / a.Hq) * (a.Hq / a.rep) + (head % a.Hq) / a.rep;
    const int L = (int)a.L;
    const _Float16 *Qh = a.Q + bh * L * kPfD, *Kh = a.K + kvh * L * kPfD, *Vh = a.V + kvh * L * kPfD;

    const int q0 = qb * (32 * WAVES) + wave * 32;      // first query of this wave
    const int query = q0 + r;                          // this lane's query column
    half8 qf[8];                                       // B operand of S^T = K Q^T: Q[query][16 ks + 8 g ..]
    {
        const _Float16 *qp = Qh + (long)min(query, L - 1) * kPfD + g * 8;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qf[ks] = *(const half8 *)(qp + ks * 16);
    }
    // Tile n of this set is tile n * SPLIT + set of the prompt.  Steps of the workgroup (every wave meets each barrier),
    // this set's tiles some query of this wave sees, and those every query of the wave sees whole:
    auto of_set = [&](int n) { return max((n - set + SPLIT - 1) / SPLIT, 0); };
    const int all = (min((qb + 1) * (32 * WAVES), L) + kPfN - 1) / kPfN;
    const int ntiles = (all + SPLIT - 1) / SPLIT;
    const int mytiles = of_set(min((q0 + 31) / kPfN + 1, all)), nfull = min(of_set((q0 + 1) / kPfN), mytiles);

    // tile loads
    const unsigned v_off = (lane >> 4) * 256u + (((lane & 15) ^ v_swizzle(lane >> 4)) << 4);
    // (of the first load; the i-th one is four rows further for each i, which flips bits 2 and 3 of the chunk)
    const unsigned k_off = (lane >> 4) * 256u + (((lane & 15) ^ ((wave * kRows + (lane >> 4)) & 15)) << 4);
    const unsigned k_lds = lds_offset(Ks) + wave * (kRows * 256u), v_lds = lds_offset(Vs) + wave * (kRows * 256u);
    // (no branch: code motion across one would take the interleaving below apart.  Lanes whose row lies past the
    // prompt load the last chunk of its last row, any finite value will do: their weights are 0.  For a tile past the
    // last one that counts every lane loads the same bytes, into a buffer nobody reads any more: nearly nothing moves.)
    auto request = [&](const _Float16 *base, int n, bool is_v) {
        const int t = n * SPLIT + set, row0 = min(t, all - 1) * kPfN + wave * kRows;
        const char *tile = (const char *)(base + (long)min(row0, L - 1) * kPfD);
        const unsigned lds = (is_v ? v_lds : k_lds) + (BUF == 2 ? (n & 1) * (kPfTile * 2u) : 0u);
        const int end = t < all ? max(L - 1 - row0, 0) * 256 + 240 : 0;
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            load_to_lds(tile, (unsigned)min((int)(is_v ? v_off : k_off ^ ((i & 3) << 6)) + i * 1024, end), lds + i * 1024u);
    };
    // all loads of this wave have landed and its fragment reads have returned (their buffer is about to be refilled); then
    // the barrier that hands every wave's share over
    auto hand_over = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // fragment reads
    int k_place[8], v_place[4];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) k_place[ks] = tile_place(r, 2 * ks + g);
    {
        const int i = lane & 15, row = 4 * g + (i >> 2), c0 = 2 * ((lane >> 4) & 1) + ((i & 3) >> 1);
#pragma unroll
        for (int db = 0; db < 4; ++db)
            v_place[db] = row * kPfD + (((4 * db + c0) ^ v_swizzle(row)) << 3) + (i & 1) * 4;
    }
    auto read_k = [&](int j, int odd) -> half8 {       // fragment j of an even / odd tile: keys 32 (j & 1) .., channels 16 (j >> 1) ..
        return *(const half8 *)(Ks + (BUF == 2 ? odd * kPfTile : 0) + (j & 1) * 32 * kPfD + k_place[j >> 1]);
    };
    auto read_v = [&](int j, int odd) -> half8 {         // fragment j: keys 16 (j >> 2) + 4 g + {0..3, 8..11}, channels 32 (j & 3) + r
        const _Float16 *p = Vs + (BUF == 2 ? odd * kPfTile : 0) + (j >> 2) * 16 * kPfD + v_place[j & 3];
        const half4 lo = read_transposed(p), hi = read_transposed(p + 8 * kPfD);
        return half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };

    float16v o[4];                                     // O^T: o[db][i] = out[query][32 db + acc_row(i, g)]
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.0f;
    const float c = a.scale_log2;                      // > 0: the running max is kept on the raw scores
    float m = -INFINITY, mc = 0.0f;                    // reference of the weights (shared by both half-waves), -m c
    float l = 0.0f;                                    // this lane's part of the sum of weights
    half8 kf[4], vf[4];                                // the next four fragments

    // the maximum mx of a tile's scores (this lane's half of the keys) settles the reference of its weights
    auto settle = [&](float mx) {
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));   // (the other half-wave holds the column's other keys)
        if (__any(mx > m)) {                           // (m = -inf at the first tile)
            const float top = fmaxf(mx, m), alpha = __builtin_amdgcn_exp2f((m - top) * c);
            m = top, mc = -top * c;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
        }
    };
    // keys after the query do not count: their scores become -inf
    auto mask = [&](float16v (&s)[2], int n) {
        const int rel = query - (n * SPLIT + set) * kPfN - 4 * g;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (t * 32 + acc_row(i, 0) > rel) s[t][i] = -INFINITY;
    };

    // tile n: scores in cur, their maximum settled, K fragments 0-3 of tile n+1 in kf.  `multiply`: there is a tile n+1
    // for this wave.
    auto step = [&](float16v (&cur)[2], float16v (&next)[2], int n, auto multiply, auto parity, auto masked) {
        constexpr int odd = decltype(parity)::value;
        half8 pb[4];                                   // B operands of the output product: the weights as fp16
        float x[2], y[2], sum[2] = {0.0f, 0.0f};
        // weights 2e, 2e+1 of this lane pass through three stages (exponent, power, sum) in three consecutive slots
        auto slot = [&](int e) {
            if (e >= 2 && e <= 17) {
                const int w = 2 * (e - 2);
                sum[0] += y[0], sum[1] += y[1];
                asm volatile("" : "+v"(sum[0]), "+v"(sum[1]));      // (else the sums of the last step sink to where they are used, and every weight lives until then)
                pb[w >> 3][w & 7] = (_Float16)y[0], pb[w >> 3][(w & 7) + 1] = (_Float16)y[1];
            }
            if (e >= 1 && e <= 16) y[0] = __builtin_amdgcn_exp2f(x[0]), y[1] = __builtin_amdgcn_exp2f(x[1]);
            if (e <= 15) {
                const int w = 2 * e;
                x[0] = __builtin_fmaf(cur[w >> 4][w & 15], c, mc), x[1] = __builtin_fmaf(cur[w >> 4][(w & 15) + 1], c, mc);
            }
        };
        if (decltype(multiply)::value) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) next[t][i] = 0.0f;
        }
        slot(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (decltype(multiply)::value) {
                next[j & 1] = mfma32(kf[j & 3], qf[j >> 1], next[j & 1]);
                if (j < 12) kf[j & 3] = read_k(j + 4, !odd);
            }
            if (j < 13) slot(j + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        hand_over();
#pragma unroll
        for (int j = 0; j < 4; ++j) vf[j] = read_v(j, odd);
        if (BUF == 2) request(Vh, n + 1, true);
        request(Kh, n + BUF + 1, false);
        float mx[4];
        if (decltype(multiply)::value && decltype(masked)::value) mask(next, n + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            o[j & 3] = mfma32(vf[j & 3], pb[j >> 2], o[j & 3]);
            if (j < 12) vf[j & 3] = read_v(j + 4, odd);
            if (BUF == 2 && decltype(multiply)::value && j >= 12) kf[j & 3] = read_k(j & 3, odd);   // (past the last tile: unused)
            if (j < 4) slot(j + 14);
            if (decltype(multiply)::value && j >= 4 && j < 12) {
                const int e = 4 * (j - 4), t = e >> 4, i = e & 15, k = j & 3;
                const float a0 = fmaxf(next[t][i], next[t][i + 1]), a1 = fmaxf(next[t][i + 2], next[t][i + 3]);
                mx[k] = j < 8 ? fmaxf(a0, a1) : fmaxf(mx[k], fmaxf(a0, a1));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        l += sum[0] + sum[1];
        if (BUF == 1) {
            hand_over();
            request(Vh, n + 1, true);
            if (decltype(multiply)::value) {
#pragma unroll
                for (int j = 0; j < 4; ++j) kf[j] = read_k(j, 0);
            }
        }
        if (decltype(multiply)::value) settle(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])));
    };

    request(Kh, 0, false);
    if (BUF == 2) request(Kh, 1, false);
    request(Vh, 0, true);
    hand_over();                                       // (the Q rows have arrived as well)
    float16v sa[2], sb[2];
    if (SPLIT == 1 || mytiles > 0) {                   // (the second set may have nothing for the first rows)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) sa[t][i] = 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) sa[j & 1] = mfma32(read_k(j, 0), qf[j >> 1], sa[j & 1]);
        if (nfull < 1) mask(sa, 0);
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sa[t][i]);
        settle(mx);
        if (BUF == 2) {
#pragma unroll
            for (int j = 0; j < 4; ++j) kf[j] = read_k(j, 1);  // (with a single tile: unused)
        }
    }
    hand_over();
    request(Kh, BUF, false);
    if (BUF == 1) {
        hand_over();
#pragma unroll
        for (int j = 0; j < 4; ++j) kf[j] = read_k(j, 0);
    }

    const std::true_type yes{};
    const std::false_type no{};
    if (SPLIT == 1 || mytiles > 0) {
        int n = 0;
        for (; n + 2 < nfull; n += 2) {
            step(sa, sb, n, yes, no, no);
            step(sb, sa, n + 1, yes, yes, no);
        }
        for (; n + 2 < mytiles; n += 2) {
            step(sa, sb, n, yes, no, yes);
            step(sb, sa, n + 1, yes, yes, yes);
        }
        // (one copy of the last step: with one for either parity the compiler keeps state of both and spills)
        if (n + 1 < mytiles) {
            step(sa, sb, n, yes, no, yes);
            sa[0] = sb[0], sa[1] = sb[1];
            if (BUF == 2) Vs += kPfTile;
            ++n;
        }
        step(sa, sb, n, no, no, no);
    }
    for (int n = mytiles; n < ntiles; ++n) {           // tiles only other waves see: this one still loads its share
        hand_over();
        if (BUF == 2) request(Vh, n + 1, true);
        request(Kh, n + BUF + 1, false);
        if (BUF == 1) {
            hand_over();
            request(Vh, n + 1, true);
        }
    }
    if constexpr (SPLIT == 2) {
        // the second set's state goes to the first through LDS (every tile has been read, every load has landed)
        float *xch = (float *)tiles + wave * (66 * 64) + lane;
        hand_over();
        if (set == 1) {
            xch[0] = m, xch[64] = l;
#pragma unroll
            for (int i = 0; i < 64; ++i) xch[(2 + i) * 64] = o[i >> 4][i & 15];
        }
        __syncthreads();
        if (set == 1) return;
        const float m1 = xch[0], top = fmaxf(m, m1);   // (m is finite: the first set has the prompt's first tile)
        const float f0 = __builtin_amdgcn_exp2f((m - top) * c), f1 = __builtin_amdgcn_exp2f((m1 - top) * c);
        l = l * f0 + xch[64] * f1;
#pragma unroll
        for (int i = 0; i < 64; ++i) o[i >> 4][i & 15] = o[i >> 4][i & 15] * f0 + xch[(2 + i) * 64] * f1;
        m = top;
    }

    l += __shfl_xor(l, 32, 64);
    const float inv = 1.0f / l, lse2 = m * c + log2f(l);
    float *row_lse2 = (float *)(tiles + SPLIT * 2 * BUF * kPfTile), *part = row_lse2 + 32 * WAVES;
    if constexpr (SCORES) {                            // the prompt's one or two K tiles again, and every row's LSE
        static_assert(!SCORES || (WAVES == 4 && SPLIT == 1 && BUF == 2), "two tiles, one set of waves");
        hand_over();
        request(Kh, 0, false);
        request(Kh, 1, false);
        if (g == 0) row_lse2[wave * 32 + r] = lse2;
        hand_over();
    }
    if (query < L) {
        if (g == 0) a.lse[bh * L + query] = lse2 * kLn2;
        _Float16 *orow = a.XO + (bh * L + query) * kPfD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int iq = 0; iq < 4; ++iq) {
                half4 h;
#pragma unroll
                for (int j = 0; j < 4; ++j) h[j] = (_Float16)(o[db][iq * 4 + j] * inv);
                *(half4 *)(orow + db * 32 + iq * 8 + g * 4) = h;
            }
    }
    if constexpr (SCORES) {
        float ls[16];
#pragma unroll
        for (int iq = 0; iq < 4; ++iq) {
            const float4 v = *(const float4 *)&row_lse2[wave * 32 + iq * 8 + g * 4];
            ls[iq * 4] = v.x, ls[iq * 4 + 1] = v.y, ls[iq * 4 + 2] = v.z, ls[iq * 4 + 3] = v.w;
        }
        const int end = L - q0 - 4 * g;                // rows of the wave's block that exist, this half-wave's share
        for (int n = 0; n < mytiles; ++n) {
            float16v s[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) s[t][i] = 0.0f;
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j & 1] = mfma32(qf[j >> 1], read_k(j, n), s[j & 1]);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int key = n * kPfN + t * 32 + r, first = key - q0 - 4 * g;     // first row that sees the key
                float sum = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][i], c, -ls[i]));
                    sum += acc_row(i, 0) >= first && acc_row(i, 0) < end ? w : 0.0f;
                }
                sum += __shfl_xor(sum, 32, 64);
                if (g == 0) part[wave * (32 * WAVES) + key] = sum;
            }
        }
        __syncthreads();
        if (tid < L) {                                 // (the waves of the rows before the key have nothing to add)
            float total = 0.0f;
            for (int w = tid >> 5; w < WAVES; ++w) total += part[w * (32 * WAVES) + tid];
            a.A_cumul[bh * L + tid] = total;
        }
    }
}

// A workgroup of four waves owns 64 KW keys and walks the queries from the diagonal down in tiles of 128 / KW through LDS.
// Wave (kw, qw) holds the K rows of 64 of the keys as B operands and takes 32 of a tile's queries, so that every Q fragment
// read from LDS feeds two products.  The products of tile n+1 and the exponentials of tile n stand side by side in one
// instruction stream (one 32x32x16 product, then the two weights whose exponent is ready): 43 cycles per product and
// two weights with two waves on a SIMD, where products and weights in separate phases took their sum.
// What bounds it: on N(0,1) data the clock falls to 1.8 GHz under this load (2.4 GHz on zeros, same cycles), so what
// counts is energy as well as issue slots.  Q tiles therefore go straight to LDS: staging them through registers cost
// 12 % of the cycles (the LDS stores stall the stream).  32 heads x 32768 tokens 4.85 -> 4.47 ms (980 TFLOP/s),
// 32 x 2048 32 -> 25 us, 32 x 777 15.6 -> 12.3 us.  Three LDS buffers instead of two: the same.  The sums are pinned where
// they are formed: without that the weights of every other step stood after its products, in front of the next ones (32
// heads x 16384 1.185 -> 1.156 ms, 32 x 777 12.7 -> 12.1 us, 8 x 2048 21.6 -> 20.2).  Two sets of waves on the even and the
// odd tiles, as in the first pass, gain on long prompts of few heads and lose on the others (8 x 2048 20.3 -> 19.2, 8 x 4096 36.0
// -> 33.2, but 32 x 400 9.1 -> 10.3, 32 x 777 12.2 -> 13.0, 32 x 4096 80 -> 95).
constexpr int kColWaves = 4;

template <int KW>
__global__ __launch_bounds__(64 * kColWaves, 2) void prefill_colsum_kernel(PrefillArgs a)
{
    constexpr int kKeys = 64 * KW, QW = kColWaves / KW, kTile = 32 * QW;   // keys of the workgroup, queries of a tile
    constexpr int kRows = kTile / kColWaves, kLoads = kRows / 4;   // rows of a tile one wave loads, four per instruction
    __shared__ __align__(16) _Float16 Qs[2 * kTile * kPfD];
    __shared__ __align__(16) float lse2[4 * kTile];    // LSE of a tile's queries in powers of two; read one iteration
                                                       // after the tile's rows, so kept longer
    __shared__ float part_sum[(QW - 1) * kKeys];

    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave % KW, qw = wave / KW;
    // column blocks in natural order: block 0 is seen by every query and is the heaviest
    const int nbh = (int)gridDim.x / a.nblk, kb = (int)blockIdx.x / nbh, head = (int)blockIdx.x % nbh;
    const long bh = head, kvh = (head / a.Hq) * (a.Hq / a.rep) + (head % a.Hq) / a.rep;
    const int L = (int)a.L;
    const _Float16 *Qh = a.Q + bh * L * kPfD, *Kh = a.K + kvh * L * kPfD;
    const float *lseh = a.lse + bh * L;

    const int k0 = kb * kKeys + kw * 64;               // first key of this wave
    half8 kf[2][8];                                    // B operands of S = Q K^T: K[key][16 ks + 8 g ..]
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const _Float16 *kr = Kh + (long)min(k0 + t * 32 + r, L - 1) * kPfD + g * 8;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kf[t][ks] = *(const half8 *)(kr + ks * 16);
    }

    const float c = a.scale_log2;
    const int tile0 = kb * kKeys / kTile, ntiles = (L + kTile - 1) / kTile;
    // A wave loads kRows consecutive rows of a tile; lanes whose row lies past the prompt load the last chunk of its last
    // row (their weights are masked), and for a tile past the last every lane loads the same bytes: nearly nothing moves.
    const unsigned q_lds = lds_offset(Qs) + wave * (kRows * 256u);
    const unsigned q_off = (wave * kRows + (lane >> 4)) * 256u + (((lane & 15) ^ (lane >> 4)) << 4);    // of the first load
    const int lse0 = wave % (kTile / 64) * 64;   // (uniform)
    auto request = [&](int n) -> float {               // returns the LSE of query lse0 + lane of the tile
        const unsigned tile = (unsigned)min(n, ntiles - 1) * (kTile * 256u);
        const unsigned end = n < ntiles ? (unsigned)(L - 1) * 256u + 240u : 0u;
        unsigned off = q_off;
        if (KW == 1) asm volatile("" : "+v"(off));     // (opaque: its four forms are not kept over the loop, which has no register for them)
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            load_to_lds(Qh, min((off ^ ((i & 3) << 6)) + i * 1024u + tile, end), q_lds + (n & 1) * (kTile * 256u) + i * 1024u);
        return lseh[min((n * kTile + lse0) + lane, L - 1)];  // (some waves the same 64: no branch in the stream)
    };
    float lr = 0.0f;
    auto settle = [&](int n) {                         // tile n is in LDS (this wave's share): then a barrier
        lse2[(n & 3) * kTile + lse0 + lane] = lr * kLog2e;
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
    };
    const int frag_row = qw * 32 + r;
    half8 qf[8];                                       // A operands: the next tile's Q rows
    float ls[16];                                      // LSE of the current tile's rows
    int q_place[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q_place[ks] = tile_place(frag_row, 2 * ks + g);
    auto read_q = [&](int ks, int n) { qf[ks] = *(const half8 *)(Qs + (n & 1) * (kTile * kPfD) + q_place[ks]); };
    auto read_lse = [&](int iq, int n) {
        const float4 v = *(const float4 *)&lse2[(n & 3) * kTile + qw * 32 + iq * 8 + g * 4];
        ls[iq * 4] = v.x, ls[iq * 4 + 1] = v.y, ls[iq * 4 + 2] = v.z, ls[iq * 4 + 3] = v.w;
    };
    // scores that do not count (query before the key, or past the prompt) become -inf: weight 0.  Few tiles have any.
    auto mask = [&](float16v (&s)[2], int n) {
        const int row0 = n * kTile + qw * 32;
        if (row0 >= k0 + 63 && row0 + 32 <= L) return;
        const int hi = L - row0 - 4 * g;               // rows of the block that exist, this half-wave's share
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int lo = k0 + t * 32 + r - row0 - 4 * g;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (acc_row(i, 0) < lo || acc_row(i, 0) >= hi) s[t][i] = -INFINITY;
        }
    };
    float cs[2] = {0.0f, 0.0f};                        // column sums of keys k0 + r and k0 + 32 + r

    // Scores of tile n+1 into `next` while the weights of tile n are formed from `cur` and added up.  Every fragment
    // and LSE register is refilled for the step after as soon as its last use is issued, so that no product waits
    // for LDS; tile n+3 goes into the buffer of tile n+1, whose rows were last read before the barrier.
    auto step = [&](float16v (&cur)[2], float16v (&next)[2], int n) {
        mask(cur, n);
        float x[2], y[2];
        x[0] = __builtin_fmaf(cur[0][0], c, -ls[0]), x[1] = __builtin_fmaf(cur[0][1], c, -ls[1]);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) next[t][i] = 0.0f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {                 // element pair 2m, 2m+1 of the 32 weights of a lane
            next[m & 1] = mfma32(qf[m >> 1], kf[m & 1][m >> 1], next[m & 1]);
            if (m & 1) read_q(m >> 1, n + 2);
            const float y0 = __builtin_amdgcn_exp2f(x[0]), y1 = __builtin_amdgcn_exp2f(x[1]);
            if (m) cs[(m - 1) >> 3] += y[0];
            if (m < 15) {
                const int t = (2 * m + 2) >> 4, i = (2 * m + 2) & 15;
                x[0] = __builtin_fmaf(cur[t][i], c, -ls[i]), x[1] = __builtin_fmaf(cur[t][i + 1], c, -ls[i + 1]);
            }
            if (m) {
                cs[(m - 1) >> 3] += y[1];
                asm volatile("" : "+v"(cs[(m - 1) >> 3]));    // (else every other step's weights sink behind the next one's mask test)
            }
            y[0] = y0, y[1] = y1;
            if (m == 0) lr = request(n + 3);
            if (m == 15) settle(n + 3);
            if (m >= 8 && !(m & 1)) read_lse((m - 8) >> 1, n + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        cs[1] += y[0];
        cs[1] += y[1];
    };
    auto finish = [&](float16v (&cur)[2], int n) {     // the last tile: nothing left to multiply
        mask(cur, n);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) cs[t] += __builtin_amdgcn_exp2f(__builtin_fmaf(cur[t][i], c, -ls[i]));
    };

    lr = request(tile0);
    const float lr1 = request(tile0 + 1);
    lse2[((tile0 + 1) & 3) * kTile + lse0 + lane] = lr1 * kLog2e;
    settle(tile0);                                     // (the second tile and the K rows have arrived as well)
    __syncthreads();
    float16v sa[2], sb[2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) read_q(ks, tile0);
#pragma unroll
    for (int iq = 0; iq < 4; ++iq) read_lse(iq, tile0);
    __syncthreads();
    lr = request(tile0 + 2);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) sa[t][i] = 0.0f;
#pragma unroll
    for (int m = 0; m < 16; ++m) sa[m & 1] = mfma32(qf[m >> 1], kf[m & 1][m >> 1], sa[m & 1]);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) read_q(ks, tile0 + 1);
    settle(tile0 + 2);
    __syncthreads();
    // At the top of iteration n the fragments of tile n+1 and the LSE of tile n are in registers and tile n+2 is
    // in LDS.
    int n = tile0;
    for (; n + 2 < ntiles; n += 2) {
        step(sa, sb, n);
        __syncthreads();
        step(sb, sa, n + 1);
        __syncthreads();
    }
    if (n + 1 < ntiles) {
        step(sa, sb, n);
        finish(sb, n + 1);
    } else {
        finish(sa, n);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) cs[t] += __shfl_xor(cs[t], 32, 64);
    const float sum = g ? cs[1] : cs[0];               // lane (r, g) stores key k0 + 32 g + r = k0 + lane
    if (qw) part_sum[(qw - 1) * kKeys + kw * 64 + lane] = sum;
    __syncthreads();
    if (qw || k0 + lane >= L) return;
    float total = sum;
#pragma unroll
    for (int w = 0; w < QW - 1; ++w) total += part_sum[w * kKeys + kw * 64 + lane];
    a.A_cumul[bh * L + k0 + lane] = total;
}

int launch_prefill(int32_t B, int32_t Hq, int32_t Hkv, int64_t L, const minikv_f16 *Q, const minikv_f16 *K,
                   const minikv_f16 *V, float sm_scale, minikv_f16 *XO, float *lse, float *A_cumul, hipStream_t st)
{
    PrefillArgs a;
    a.Q = (const _Float16 *)Q, a.K = (const _Float16 *)K, a.V = (const _Float16 *)V;
    a.XO = (_Float16 *)XO, a.lse = lse, a.A_cumul = A_cumul;
    a.Hq = Hq, a.rep = Hq / Hkv, a.L = L, a.scale_log2 = sm_scale * kLog2e;
    // Queries per workgroup and whether two sets of waves share them.  256 queries halve what a tile costs to load; on long
    // prompts, while they leave four workgroups per compute unit, that is 1-3 % (64 heads x 16384: 4.32 -> 4.25 ms), on
    // shorter ones the waves that are done wait for the others (512 heads x 257: 47 -> 59 us).  Else 128, but a launch of
    // few workgroups lasts as long as its longest row block, and that is shorter
    //   with 64 queries shared by two sets, if there is one workgroup per compute unit (8 heads x 2048: 37.4 -> 27.2 us, 32 x
    //   512 14.7 -> 11.9, 64 x 200 9.7 -> 9.2, 32 x 128 8.0 -> 7.4, but 8 x 65 6.8 -> 7.3), or, of few heads, not many more:
    //   the second ones are then blocks that see a short part of the prompt (16 x 1200 24.2 -> 19.6, 8 x 3000 50.7 -> 38.3);
    //   the same with one buffer each, if all run at once, two per compute unit (32 x 777 19.0 -> 16.9, 32 x 1000 22.9 ->
    //   20.7, 48 x 512 14.9 -> 14.5, 16 x 2048 38.5 -> 32.2 against 34.6 with two buffers, which are better by themselves:
    //   16 x 1200 19.6 against 20.6; 64 x 320 10.9 -> 12.3, 48 x 777, at 624 workgroups, 21.7 -> 24.7);
    //   with 128 shared by two sets, if there are not many more than one per compute unit on long prompts of few heads (8 x
    //   6000: 110.8 -> 98.5, 16 x 3000 59.3 -> 52.9, 32 x 1200 27.5 -> 26.4; but 24 x 2100 45.2 -> 46.1, 48 x 1000 26.2 -> 29.7).
    // In the second pass eight waves per workgroup lose (4.36 -> 4.62 ms): they wait for each other at every tile.
    const int64_t heads = (int64_t)B * Hq;
    auto blocks = [&](int queries) { return heads * ((L + queries - 1) / queries); };
    if (A_cumul && L <= 128) {                         // one row block a head: always faster in one launch (see SCORES)
        a.nblk = 1;
        hipLaunchKernelGGL((prefill_fwd_kernel<4, 1, 2, true>), dim3((unsigned)heads), dim3(256), fwd_lds_bytes(1, 2, 128), st, a);
        return hipGetLastError() == hipSuccess ? MINIKV_OK : MINIKV_ELAUNCH;
    }
    const bool two_buffers = L > 96 && 2 * blocks(64) <= (heads <= 20 ? 3 : 2) * kComputeUnits;
    const bool two_sets_64 = two_buffers || (L > 384 && blocks(64) <= 2 * kComputeUnits);
    const bool two_sets_128 = L >= 1024 && heads <= 32 && 2 * blocks(128) <= (heads <= 20 ? 4 : 3) * kComputeUnits;
    const int queries = L >= 4096 && blocks(256) >= 4 * kComputeUnits ? 256 : two_sets_64 ? 64 : 128;
    a.nblk = (int)((L + queries - 1) / queries);
    const dim3 grid((unsigned)(heads * a.nblk));
    if (queries == 256)
        hipLaunchKernelGGL((prefill_fwd_kernel<8, 1, 2, false>), grid, dim3(512), fwd_lds_bytes(1, 2), st, a);
    else if (two_sets_64 && !two_buffers)
        hipLaunchKernelGGL((prefill_fwd_kernel<2, 2, 1, false>), grid, dim3(256), fwd_lds_bytes(2, 1), st, a);
    else if (two_sets_64)
        hipLaunchKernelGGL((prefill_fwd_kernel<2, 2, 2, false>), grid, dim3(256), fwd_lds_bytes(2, 2), st, a);
    else if (two_sets_128)
        hipLaunchKernelGGL((prefill_fwd_kernel<4, 2, 2, false>), grid, dim3(512), fwd_lds_bytes(2, 2), st, a);
    else
        hipLaunchKernelGGL((prefill_fwd_kernel<4, 1, 2, false>), grid, dim3(256), fwd_lds_bytes(1, 2), st, a);
    if (hipGetLastError() != hipSuccess) return MINIKV_ELAUNCH;
    if (A_cumul) {
        // 64 keys per workgroup, its four waves side by side on 128 queries, while the launch lasts as long as its longest walk:
        // one workgroup per compute unit, or two of few heads, where the second ones walk a short part of the prompt.
        // Whole call, 128 keys -> 64 keys, us: 8 heads x 160 14.9 -> 14.2, x 777 25.4 -> 23.3, x 2048 45.1 -> 39.9, x 4096 (512
        // workgroups) 89.6 -> 84.0; 16 x 2048 51.6 -> 49.4, 32 x 512 20.3 -> 19.0; beyond, the second read of Q by twice the
        // workgroups loses: 32 x 777 (416) the same, 64 x 384 (384) 20.9 -> 21.7, 16 x 3000 83.8 -> 86.7, 32 x 1500 53.5 -> 57.5.
        // At the lines: 17 x 1868 (510 workgroups) 54.2 -> 54.2, 18 x 1778 49.9 -> 49.3, 19 x 1605 49.7 -> 50.8, 20 x 1575 46.1 -> 45.2
        // (each side varies by 2-4 % there), 20 x 1369 (440) 39.7 -> 37.7; 21 x 747 (252) 28.5 -> 27.1, 32 x 493 (256) 21.5 -> 19.9, 64 x 209
        // 16.9 -> 15.9.  (Eight waves on 256 queries lose to four everywhere: 8 x 384 16.9 -> 19.5, 8 x 2048 39.9 -> 40.7.)
        if (blocks(64) <= (heads <= 20 ? 2 : 1) * kComputeUnits) {
            a.nblk = (int)((L + 63) / 64);
            hipLaunchKernelGGL((prefill_colsum_kernel<1>), dim3((unsigned)(heads * a.nblk)), dim3(64 * kColWaves), 0, st, a);
        } else {
            a.nblk = (int)((L + 127) / 128);
            hipLaunchKernelGGL((prefill_colsum_kernel<2>), dim3((unsigned)(heads * a.nblk)), dim3(64 * kColWaves), 0, st, a);
        }
        if (hipGetLastError() != hipSuccess) return MINIKV_ELAUNCH;
    }
    return MINIKV_OK;
}

}  // namespace minikv
