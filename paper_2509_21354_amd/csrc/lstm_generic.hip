// Recurrent gate, Eq. 3 of the paper: a standard LSTM cell (gate rows i,f,g,o)
// over the chunk summaries [Kbar_t ; Vbar_t] with a scalar utility head on h_t.
// fp32-arithmetic kernel for fp32 storage and for gate widths that the
// matrix-core kernels do not take (lstm_mfma.hip has the bf16 fast path).  No
// workspace is used: one workgroup walks one sequence through its steps.
//
// What bounds it is the chain of dependent steps, so everything that does not
// depend on h_{t-1} is taken out of the step, and the step itself is spread over
// a whole workgroup of 16 waves:
//   * the steps are cut into blocks of up to 16.  The input projections
//     W_ih x_t + b_ih + b_hh of a block are one 4 d_g x 2d x 16 product on the fp32
//     matrix instruction (v_mfma_f32_16x16x4_f32: fp32 operands, products and
//     sums), kept in LDS;
//   * a group of 16 lanes owns a hidden unit (or several): lane c holds elements
//     4 c .. 4 c + 3 (mod 64) of that unit's four rows of W_hh and of h, and the
//     four partial dot products are folded over the 16 lanes by a transposing
//     reduction that leaves one gate's sum in each lane of a quad, where its
//     nonlinearity is evaluated; c_t and h_t follow in the same lanes, so a
//     step has one barrier;
//   * up to d_g = 128 the four rows stay in registers for the whole call (RES > 0),
//     and up to 192 with bf16 storage, as the pairs that they are (two shifts and masks
//     per pair and step; what bounds the streamed form there is its chain of dependent
//     loads, of single elements where d_g is no multiple of 4: d_g = 163, 32 sequences x
//     32 steps 586 -> 131 us, 512 x 32 1173 -> 262, 1024 x 32 772 (four a workgroup) ->
//     521; short calls of many sequences keep the streamed form: see launch_t); wider
//     gates read them from L2 every step, 16 bytes per lane;
//   * the utility head runs after each block over the block's 16 states.
// Measured (fp32, d_g = 64, d = 64, 4 sequences x 64 steps): 1346 us with one
// row of W_ih and W_hh at a time per lane group, dependent loads from L2 in every
// step; 64 us (1 us per step, the projections included); lstm_chain_kernel below takes 42 us.  d_g = 256, d = 128, 32 sequences x 64 steps: 11.4 ms
// -> 0.69 ms, bound by the 1 MiB of W_hh that a workgroup streams per step.
#include <utility>
#include "common.hpp"
#include "kernels.hpp"
#include "lstm_common.hpp"

namespace kvev {

constexpr int kGenThreads = 1024, kGenCols = 16;      // (sequence, step) pairs of a block: one column tile of the projection
constexpr size_t kGenLdsMax = 160 * 1024;

// LDS of a block of tb steps of mb sequences: inputs, projections, states (step 0: the state before the block), cell state
constexpr int gen_hp(int dg) { return (dg + 63) / 64 * 64; }
constexpr size_t gen_lds(int d, int dg, int mb, int tb)
{
    return sizeof(float) * mb * ((size_t)tb * (2 * d + 4) + (size_t)tb * 4 * dg + (size_t)(tb + 1) * gen_hp(dg) + dg);
}
// most steps of a block that LDS holds (0: not even one)
static int gen_tb(int d, int dg, int mb)
{
    int tb = kGenCols / mb;
    while (tb > 0 && gen_lds(d, dg, mb, tb) > kGenLdsMax) --tb;
    return tb;
}

// Four bf16 elements of R rows `pitch` elements apart, from each of k, k + 64, .. on, as the pairs that they are, zeros at and past n.
// Rows that allow no wider load are read by the element, without a branch: all requests leave before the first is waited for.
template <int R, int KC, bool VEC> __device__ __forceinline__ void load_pairs(const bf16_t *mat, uint32_t at, uint32_t pitch, int k, int n, float (*o)[KC][2])
{
    if constexpr (VEC) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                const uint2 v = 64 * c + k < n ? *reinterpret_cast<const uint2 *>(mat + (at + r * pitch + 64 * c + k)) : make_uint2(0u, 0u);
                o[r][c][0] = __uint_as_float(v.x);
                o[r][c][1] = __uint_as_float(v.y);
            }
    } else {
        uint32_t v[R][KC][4];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[r][c][e] = mat[at + r * pitch + (uint32_t)min(64 * c + k + e, n - 1)];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int j = 64 * c + k + 2 * e;
                    o[r][c][e] = __uint_as_float((j < n ? v[r][c][2 * e] : 0u) | (j + 1 < n ? v[r][c][2 * e + 1] << 16 : 0u));
                    asm volatile("" : "+v"(o[r][c][e]));         // (the pair is kept, not its elements until it is used)
                }
    }
}

// MB: sequences of one layer per workgroup.  RES: hidden units per lane group whose rows of W_hh stay in registers, KC
// chunks of 64 elements each (0: the rows are streamed).  VEC: d_g is a multiple of 4, so every row of W_hh starts where
// a 4-element load may.
template <typename T, int D, int MB, int RES, int KC, bool VEC>
__global__ __launch_bounds__(kGenThreads, RES == 1 && MB == 1 ? 8 : 4) void lstm_generic_kernel(LstmArgs a, int tb)
{
    constexpr int XP = 2 * D + 4;       // padded input row: the columns of a block start in different banks
    static_assert(MB == 1 || MB == 4, "what cell() folds");
    extern __shared__ __align__(16) float smem[];
    const int dg = a.d_g, G = 4 * dg, HP = gen_hp(dg);
    float *x = smem;                                 // [MB * tb][XP]
    float *pre = x + (size_t)MB * tb * XP;           // [MB * tb][4 d_g]
    float *hs = pre + (size_t)MB * tb * G;           // [MB][tb + 1][HP]   zeros from d_g on
    float *cs = hs + (size_t)MB * (tb + 1) * HP;     // [MB][d_g]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cl = tid & 15, grp = tid >> 4;
    const int gpl = (a.BH + MB - 1) / MB;
    const int l = blockIdx.x / gpl, m0 = (blockIdx.x % gpl) * MB;
    const int live = min(MB, a.BH - m0);             // (a group never straddles layers; the rest repeat the last sequence)
    auto seq = [&](int m) __attribute__((always_inline)) { return (size_t)l * a.BH + m0 + min(m, live - 1); };
    const T *W_ih = static_cast<const T *>(a.W_ih) + (size_t)l * G * 2 * D;
    const T *W_hh = static_cast<const T *>(a.W_hh) + (size_t)l * G * dg;
    const T *b_ih = static_cast<const T *>(a.b_ih) + (size_t)l * G;
    const T *b_hh = static_cast<const T *>(a.b_hh) + (size_t)l * G;
    const T *w_s = static_cast<const T *>(a.w_s) + (size_t)l * dg;
    const float b_s = Storage<T>::load(static_cast<const T *>(a.b_s) + l);
    const int gate = value_of_lane(cl);

    const bool fresh = a.c0 == 0;        // the recurrence starts from a zero state at chunk 0, whatever the buffers hold
    for (int j = tid; j < MB * (tb + 1) * HP; j += kGenThreads) {
        const int m = j / ((tb + 1) * HP), e = j % ((tb + 1) * HP);
        hs[j] = e < dg && !fresh ? a.h[seq(m) * dg + e] : 0.f;
    }
    for (int j = tid; j < MB * dg; j += kGenThreads) cs[j] = fresh ? 0.f : a.c[seq(j / dg) * dg + j % dg];

    // (at three units of three chunks only as the bf16 pairs that they are)
    constexpr bool PACKED = RES == 3;
    static_assert(!PACKED || sizeof(T) == 2, "two elements of a row in a register");
    constexpr int WN = PACKED ? 2 : 4;
    float w[RES > 0 ? RES : 1][4][KC][WN];
    if constexpr (RES > 0) {
#pragma unroll
        for (int i = 0; i < RES; ++i) {
            const int u = min(grp + kGenThreads / 16 * i, dg - 1);
            if constexpr (PACKED) {
                load_pairs<2, KC, VEC>(W_hh, (uint32_t)u * dg, (uint32_t)dg * dg, 4 * cl, dg, w[i]);
                load_pairs<2, KC, VEC>(W_hh, (uint32_t)(2 * dg + u) * dg, (uint32_t)dg * dg, 4 * cl, dg, w[i] + 2);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int c = 0; c < KC; ++c) load4<T, VEC>(W_hh + (size_t)(q * dg + u) * dg, 64 * c + 4 * cl, dg, w[i][q][c]);
            }
        }
    }

    for (int t0 = a.c0; t0 < a.c1; t0 += tb) {
        const int nb = min(tb, a.c1 - t0), cols = MB * nb;      // column m * nb + j: step t0 + j of sequence m
        // ---- the block's inputs ----
        for (int p = tid; p < cols * (2 * D / 4); p += kGenThreads) {
            const int col = p / (2 * D / 4), e = (p % (2 * D / 4)) * 4;
            const size_t row = (seq(col / nb) * a.N_cap + t0 + col % nb) * D;
            float v[4];
            VecLoad<T, 4>::run((e < D ? static_cast<const T *>(a.Kbar) + e : static_cast<const T *>(a.Vbar) + (e - D)) + row, v);
            *reinterpret_cast<float4 *>(x + (size_t)col * XP + e) = make_float4(v[0], v[1], v[2], v[3]);
        }
        __syncthreads();
        // ---- their projections: 16 gate rows x 16 columns per wave and turn.  A contraction index may be permuted as
        // long as both operands agree: lane group g takes elements 16 c + 4 g .. + 3 of chunk c, one per instruction ----
        for (int r0 = wave * 16; r0 < G; r0 += 16 * (kGenThreads / 64)) {
            const int g = lane >> 4;
            const T *wr = W_ih + (size_t)min(r0 + cl, G - 1) * 2 * D + 4 * g;
            const float *xr = x + (size_t)min(cl, cols - 1) * XP + 4 * g;
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int c = 0; c < 2 * D / 16; ++c) {
                float wv[4];
                VecLoad<T, 4>::run(wr + 16 * c, wv);
                const float4 xv = *reinterpret_cast<const float4 *>(xr + 16 * c);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[0], xv.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[1], xv.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[2], xv.z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[3], xv.w, acc, 0, 0, 0);
            }
            if (cl < cols) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = r0 + 4 * g + r;
                    if (row < G) pre[(size_t)cl * G + row] = acc[r] + Storage<T>::load(b_ih + row) + Storage<T>::load(b_hh + row);
                }
            }
        }
        __syncthreads();
        // ---- the steps ----
        // unit u's partial sums are in `part`: the cell update and the new h.  With one sequence the four quads of a lane
        // group do the same work, with four each quad does that of a sequence of its own.
        const int mq = MB == 4 ? cl >> 2 : 0;
        auto cell = [&](int tt, int u, const float (&part)[MB][4]) __attribute__((always_inline)) {
            float z;
            if constexpr (MB == 4) z = fold16(part, cl);
            else z = fold4(part[0], cl);
            z += pre[(size_t)(mq * nb + tt) * G + gate * dg + u];
            const float act = gate == 2 ? tanhf(z) : 1.f / (1.f + expf(-z));
            // lanes 0, 2, 1, 3 of a quad hold i, f, g, o
            const float ig = dpp_move<0x00>(act), fg = dpp_move<0xAA>(act), gg = dpp_move<0x55>(act), og = dpp_move<0xFF>(act);
            const float cn = fg * cs[mq * dg + u] + ig * gg;
            const float hn = og * tanhf(cn);
            if (MB == 4 ? (cl & 3) == 0 : cl == 0) {     // (lanes with the same values, and all have read the old cell state)
                cs[mq * dg + u] = cn;
                hs[(size_t)(mq * (tb + 1) + tt + 1) * HP + u] = hn;
            }
        };
        for (int tt = 0; tt < nb; ++tt) {
            const float *hp = hs + (size_t)tt * HP + 4 * cl;        // + m * (tb + 1) * HP + 64 * chunk
            if constexpr (RES > 0) {
#pragma unroll
                for (int i = 0; i < RES; ++i) {
                    const int u = grp + kGenThreads / 16 * i;
                    if constexpr (PACKED) {          // (else the compiler unpacks them all once, before the steps, and spills)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int c = 0; c < KC; ++c) asm volatile("" : "+v"(w[i][q][c][0]), "+v"(w[i][q][c][1]));
                    }
                    if (u < dg) {
                        float part[MB][4];
#pragma unroll
                        for (int m = 0; m < MB; ++m) {
                            part[m][0] = part[m][1] = part[m][2] = part[m][3] = 0.f;
#pragma unroll
                            for (int c = 0; c < KC; ++c) {
                                float hv[4];
                                VecLoad<float, 4>::run(hp + (size_t)m * (tb + 1) * HP + 64 * c, hv);
#pragma unroll
                                for (int q = 0; q < 4; ++q)
#pragma unroll
                                    for (int e = 0; e < 4; ++e) {
                                        const float we = !PACKED ? w[i][q][c][e % WN] : e % 2 ? __uint_as_float(__float_as_uint(w[i][q][c][e / 2 % WN]) & 0xFFFF0000u)
                                                                                                : __uint_as_float(__float_as_uint(w[i][q][c][e / 2 % WN]) << 16);
                                        part[m][q] = fmaf(we, hv[e], part[m][q]);
                                    }
                            }
                        }
                        cell(tt, u, part);
                    }
                }
            } else {
                for (int u = grp; u < dg; u += kGenThreads / 16) {
                    const T *wr = W_hh + (size_t)u * dg;
                    float part[MB][4];
#pragma unroll
                    for (int m = 0; m < MB; ++m) part[m][0] = part[m][1] = part[m][2] = part[m][3] = 0.f;
#pragma unroll MB == 1 ? 4 : 2
                    for (int k = 0; k < dg; k += 64) {
                        float wv[4][4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) load4<T, VEC>(wr + (size_t)q * dg * dg, k + 4 * cl, dg, wv[q]);
#pragma unroll
                        for (int m = 0; m < MB; ++m) {
                            float hv[4];
                            VecLoad<float, 4>::run(hp + (size_t)m * (tb + 1) * HP + k, hv);
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int e = 0; e < 4; ++e) part[m][q] = fmaf(wv[q][e], hv[e], part[m][q]);
                        }
                    }
                    cell(tt, u, part);
                }
            }
            __syncthreads();
        }
        // ---- the block's scores: a wave per (sequence, step) ----
        for (int col = wave; col < live * nb; col += kGenThreads / 64) {
            const int m = col / nb, tt = col % nb;
            float u = 0.f;
            for (int j = lane; j < dg; j += kWave) u = fmaf(Storage<T>::load(w_s + j), hs[(size_t)(m * (tb + 1) + tt + 1) * HP + j], u);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) u += __shfl_xor(u, off);
            if (lane == 0) {
                u += b_s;
                a.util[seq(m) * a.N_cap + t0 + tt] = u;
                a.gate[seq(m) * a.N_cap + t0 + tt] = 1.f / (1.f + expf(-u));
            }
        }
        // the next block starts from this one's last state (step 0 is read by its first step only)
        for (int j = tid; j < MB * dg; j += kGenThreads) {
            float *hm = hs + (size_t)(j / dg) * (tb + 1) * HP + j % dg;
            hm[0] = hm[(size_t)nb * HP];
        }
    }
    __syncthreads();
    for (int j = tid; j < live * dg; j += kGenThreads) {
        const int m = j / dg, e = j % dg;
        a.h[seq(m) * dg + e] = hs[(size_t)m * (tb + 1) * HP + e];
        a.c[seq(m) * dg + e] = cs[j];
    }
}

// ---- d_g <= 64, one sequence per workgroup --------------------------------------------------------------------------
// Nonlinearities of the step below: the hardware exp2 and reciprocal, the latter with one Newton step, and for small
// arguments of tanh an odd polynomial (x + x^3 P(x^2), relative error 1.4e-9, a weighted least-squares fit iterated
// towards the minimax one), in a third of the instructions of expf, a division and tanhf and without branches.  The
// sigmoids add back what the product with log2 e was rounded by and stay within 3 ulp of themselves, however small (alone,
// that rounding grows with the argument: 8 ulp at -20).  tanh stays within 2 ulp: its share of 1 / (1 + e^2|x|) falls as
// the rounding grows.  NaN stays NaN.
__device__ __forceinline__ float rcp_newton(float d)
{
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.f), r, r);
}
// 1 / (1 + 2^y (1 + rest)); 0 where that is less than 2^-126 (the Newton step has no answer to an infinite 2^y)
__device__ __forceinline__ float inv_1p_exp2(float y, float rest)
{
    const float e = __builtin_amdgcn_exp2f(y);
    const float r = rcp_newton(fmaf(e, rest, 1.f + e));
    return y > 126.f ? 0.f : r;
}
__device__ __forceinline__ float inv_1p_exp2(float y)
{
    const float r = rcp_newton(1.f + __builtin_amdgcn_exp2f(y));
    return y > 126.f ? 0.f : r;
}
constexpr float kTanhSmall = 0.5625f;
__device__ __forceinline__ float tanh_small(float x)
{
    const float s = x * x;
    const float p = fmaf(fmaf(fmaf(fmaf(-0.006179808871800135f, s, 0.021007458045466547f), s, -0.05383742992718666f), s, 0.13332452268837372f), s, -0.3333331388797284f);
    return fmaf(x * s, p, x);
}
// tanh x from r = 1 / (1 + e^2|x|)
__device__ __forceinline__ float tanh_of(float x, float r)
{
    return fabsf(x) < kTanhSmall ? tanh_small(x) : copysignf(fmaf(-2.f, r, 1.f), x);
}

// What bounds a small launch is the chain of one step on one compute unit, so a step is as short as its dependences: a
// thread owns one gate row (its 64 weights in registers) and one nonlinearity, a quad of lanes the four gates of a unit.
// Four waves, one per SIMD, do nothing else.  Four more sit beside them and make the input projections of the next 16
// steps on the matrix cores, a sixteenth per step, and the scores; what they read from memory was asked for steps ahead
// (d = 64: their rows of W_ih stay in registers).  One barrier per step.
// Measured (fp32, d_g = 64, the kernel above and this one): d = 64, 4 sequences x 256 steps 248 and 142 us (0.52 us a step, of
// which about 0.1 are the products, 0.15 the nonlinearities, the rest LDS and the barrier), x 16 steps 18.7 and 16.0 us; d = 128,
// 256 x 64 steps 81 and 57 us; bf16, d_g = 50, d = 128, 96 x 128 steps 145 and 121 us.  One workgroup per compute unit: launches
// of more sequences than that are faster above (512 x 64 steps 78 and 108 us).
template <typename T, int D>
__global__ __launch_bounds__(512, 2) void lstm_chain_kernel(LstmArgs a)
{
    constexpr int NU = 64, TB = 16, CT = 2 * D / 16;         // units; steps of a block; 16-element chunks of an input row
    constexpr int TILES = 4 * NU / 16 / 4, CH = TILES * CT / TB;     // tiles of 16 gate rows per projecting wave; chunks per step
    constexpr int PPT = CT / CH;                             // steps per tile
    static_assert(CT % CH == 0 && PPT * TILES == TB, "a step stays within one tile");
    __shared__ __align__(16) float s_h[2][NU], s_pre[2][TB][4 * NU];
    const int dg = a.d_g, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = blockIdx.x / a.BH, n = a.c1 - a.c0;
    const size_t s = blockIdx.x;                             // (layers are contiguous)
    const T *W_ih = static_cast<const T *>(a.W_ih) + (size_t)l * 4 * dg * 2 * D;
    const bool fresh = a.c0 == 0;        // the recurrence starts from a zero state at chunk 0, whatever the buffers hold

    // ---- the projections, a tile of 16 gate rows x 16 steps at a time: gate row 4 u + q of the tile order is row q d_g + u
    //      of W_ih.  A contraction index may be permuted as long as both operands agree: lane group g takes elements
    //      16 c + 4 g .. + 3 of chunk c ----
    const int cl = lane & 15, g = lane >> 4;
    auto load_w = [&](int tile, int c, float (&o)[4]) __attribute__((always_inline)) {
        const int row = tile * 16 + cl, u = min(row >> 2, dg - 1);
        VecLoad<T, 4>::run(W_ih + ((size_t)(row & 3) * dg + u) * 2 * D + 16 * c + 4 * g, o);
    };
    auto load_x = [&](int block, float (&o)[CT][4]) __attribute__((always_inline)) {         // column cl: step cl of the block
        const size_t chunk = (s * a.N_cap + min(a.c0 + block * TB + cl, a.c1 - 1)) * D;
#pragma unroll
        for (int c = 0; c < CT; ++c) VecLoad<T, 4>::run(static_cast<const T *>(c < CT / 2 ? a.Kbar : a.Vbar) + chunk + 16 * (c % (CT / 2)) + 4 * g, o[c]);
    };
    // (two chains of sums: even and odd elements)
    auto multiply = [&](const float (&w)[4], const float (&x)[4], f32x4_t (&acc)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], acc[e & 1], 0, 0, 0);
    };
    auto load_bias = [&](int tile) __attribute__((always_inline)) {
        const int u = min((tile * 16 + 4 * g) >> 2, dg - 1);
        f32x4_t v;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[r] = Storage<T>::load(static_cast<const T *>(a.b_ih) + (size_t)l * 4 * dg + r * dg + u) +
                   Storage<T>::load(static_cast<const T *>(a.b_hh) + (size_t)l * 4 * dg + r * dg + u);
        return v;
    };
    auto put = [&](int block, int tile, const f32x4_t &v) __attribute__((always_inline)) {
        *reinterpret_cast<f32x4_t *>(&s_pre[block & 1][cl][tile * 16 + 4 * g]) = v;
    };
    constexpr bool RES = CT <= 8;                            // a projecting wave's weights all in registers, else WA steps ahead
    if constexpr (!RES) {       // the first block's, by all waves
        float x[CT][4];
        load_x(0, x);
        for (int tile = wave; tile < NU / 4; tile += 8) {
            float w[CT][4];
#pragma unroll
            for (int c = 0; c < CT; ++c) load_w(tile, c, w[c]);
            const f32x4_t bias = load_bias(tile);
            f32x4_t acc[2] = {};
#pragma unroll
            for (int c = 0; c < CT; ++c) multiply(w[c], x[c], acc);
            put(0, tile, acc[0] + acc[1] + bias);
        }
    }

    if (wave < 4) {
        // ---- the recurring waves: a quad of lanes has unit 16 wave + lane / 4; lane k of it multiplies elements 16 k .. + 15 of
        //      its four rows (each thread a row of its own would read four times as much of h from LDS) and ends, after
        //      a transposing reduction, with one gate ----
        const int kq = lane & 3, gate = value_of_lane(lane), unit = wave * 16 + (lane >> 2), u = min(unit, dg - 1);
        float w[4][16], c = 0.f, hn = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const T *row = static_cast<const T *>(a.W_hh) + ((size_t)l * 4 * dg + (size_t)r * dg + u) * dg;
#pragma unroll
            for (int k = 0; k < 16; k += 4) {
                float v[4];
                if (dg % 4 == 0) load4<T, true>(row, 16 * kq + k, dg, v);
                else load4<T, false>(row, 16 * kq + k, dg, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[r][k + e] = v[e];
            }
        }
        if (!fresh) {
            c = a.c[s * dg + u];
            hn = a.h[s * dg + u];
        }
        if (kq == 0) s_h[0][unit] = unit < dg ? hn : 0.f;
        const bool b0 = lane & 1, b1 = lane & 2, is_g = gate == 2;
        const float mul = is_g ? 2.8853900817779268f : -1.4426950408889634f;         // of |x| for tanh, of x for the sigmoids
        const float mul_rest = is_g ? 2.6699516e-8f : -1.3349758e-8f;               // what the constant lacks, times ln 2
        lds_barrier();
        for (int t = 0; t < n; ++t) {
            const float *h = s_h[t & 1] + 16 * kq;
            const float x = s_pre[(t / TB) & 1][t % TB][4 * unit + gate];
            float z[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 16; k += 4) {
                const float4 hv = *reinterpret_cast<const float4 *>(h + k);
#pragma unroll
                for (int r = 0; r < 4; ++r) z[r] = fmaf(w[r][k + 3], hv.w, fmaf(w[r][k + 2], hv.z, fmaf(w[r][k + 1], hv.y, fmaf(w[r][k], hv.x, z[r]))));
            }
            const float r0 = (b0 ? z[2] : z[0]) + dpp_move<kQuadXor1>(b0 ? z[0] : z[2]);
            const float r1 = (b0 ? z[3] : z[1]) + dpp_move<kQuadXor1>(b0 ? z[1] : z[3]);
            const float zz = (b1 ? r1 : r0) + dpp_move<kQuadXor2>(b1 ? r0 : r1) + x;
            const float arg = is_g ? fabsf(zz) : zz, y = mul * arg;
            const float off = fmaf(fmaf(mul, arg, -y), 0.69314718f, mul_rest * arg);
            const float r = inv_1p_exp2(y, y >= -126.f ? off : 0.f);         // (minus infinity has none)
            const float act = is_g ? tanh_of(zz, r) : r;
            // lanes 0, 2, 1, 3 of a quad hold i, f, g, o
            const float ig = dpp_move<0x00>(act), fg = dpp_move<0xAA>(act), gg = dpp_move<0x55>(act), og = dpp_move<0xFF>(act);
            c = fmaf(fg, c, ig * gg);
            hn = og * tanh_of(c, inv_1p_exp2(2.8853900817779268f * fabsf(c)));
            if (kq == 0) s_h[(t + 1) & 1][unit] = unit < dg ? hn : 0.f;
            lds_barrier();
        }
        if (kq == 0 && unit < dg) {
            a.h[s * dg + unit] = hn;
            a.c[s * dg + unit] = c;
        }
        return;
    }

    // ---- the projecting waves ----
    constexpr int WA = 2;
    const int tile0 = (wave - 4) * TILES;
    float w[RES ? TB : WA][CH][4], xc[CT][4], xn[CT][4];
    f32x4_t bias[TILES], acc[2];
    static_for<TILES>([&](auto ic) __attribute__((always_inline)) { bias[decltype(ic)::value] = load_bias(tile0 + decltype(ic)::value); });
    auto load_part = [&](int part, float (&o)[CH][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < CH; ++k) load_w(tile0 + part / PPT, part % PPT * CH + k, o[k]);
    };
    static_for<(RES ? TB : WA)>([&](auto ic) __attribute__((always_inline)) { load_part(decltype(ic)::value, w[decltype(ic)::value]); });
    // the score of step t from h_t: a unit per lane; the first of these waves writes a block's scores together
    const float w_s = lane < dg ? Storage<T>::load(static_cast<const T *>(a.w_s) + (size_t)l * dg + lane) : 0.f;
    const float b_s = Storage<T>::load(static_cast<const T *>(a.b_s) + l);
    float held = 0.f;
    auto score = [&](int t) __attribute__((always_inline)) {
        float u = w_s * s_h[(t + 1) & 1][lane];
        asm volatile("" : "+v"(u));      // the rounded product wherever this is inlined (never an fma with the next sum)
        u += dpp_move<kQuadXor1>(u);
        u += dpp_move<kQuadXor2>(u);
        u += dpp_move<kRowRor4>(u);
        u += dpp_move<kRowRor8>(u);
        // (lanes add their quads in different orders: the score is the first lane's, whichever lane will hold it)
        u = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rows_sum(u)))) + b_s;
        held = lane == (t & (TB - 1)) ? u : held;
    };
    auto write_scores = [&](int t) __attribute__((always_inline)) {          // of the block up to step t
        if (wave == 4 && lane <= (t & (TB - 1))) {
            const size_t at = s * a.N_cap + a.c0 + (t & ~(TB - 1)) + lane;
            a.util[at] = held;
            a.gate[at] = 1.f / (1.f + expf(-held));
        }
    };
    if constexpr (RES) {        // the first block's
        load_x(0, xc);
        if (n > TB) load_x(1, xn);
        static_for<TB>([&](auto pc) __attribute__((always_inline)) {
            constexpr int part = decltype(pc)::value;
            if constexpr (part % PPT == 0) acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            static_for<CH>([&](auto kc) __attribute__((always_inline)) { multiply(w[part][decltype(kc)::value], xc[part % PPT * CH + decltype(kc)::value], acc); });
            if constexpr (part % PPT == PPT - 1) put(0, tile0 + part / PPT, acc[0] + acc[1] + bias[part / PPT]);
        });
    } else if (n > TB) {
        load_x(1, xn);
    }
    lds_barrier();
    int t = 0;
    for (int block = 0; (block + 1) * TB < n; ++block) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) xc[c][e] = xn[c][e];
        if ((block + 2) * TB < n) load_x(block + 2, xn);
        static_for<TB>([&](auto pc) __attribute__((always_inline)) {
            constexpr int part = decltype(pc)::value, slot = RES ? part : part % WA;
            score(t - 1);           // (of no step at t = 0)
            if (part == 0 && t > 0) write_scores(t - 1);
            if constexpr (part % PPT == 0) acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            static_for<CH>([&](auto kc) __attribute__((always_inline)) { multiply(w[slot][decltype(kc)::value], xc[part % PPT * CH + decltype(kc)::value], acc); });
            if constexpr (!RES) load_part((part + WA) % TB, w[slot]);
            if constexpr (part % PPT == PPT - 1) put(block + 1, tile0 + part / PPT, acc[0] + acc[1] + bias[part / PPT]);
            lds_barrier();
            ++t;
        });
    }
    for (; t < n; ++t) {
        score(t - 1);
        if (t % TB == 0 && t > 0) write_scores(t - 1);
        lds_barrier();
    }
    score(n - 1);
    write_scores(n - 1);
}

template <typename T, int D, int MB, int RES, int KC>
static hipError_t launch_v(const LstmArgs &a, hipStream_t st)
{
    const int tb = gen_tb(D, a.d_g, MB);
    const size_t lds = gen_lds(D, a.d_g, MB, tb);
    const auto kernel = a.d_g % 4 == 0 ? lstm_generic_kernel<T, D, MB, RES, KC, true> : lstm_generic_kernel<T, D, MB, RES, KC, false>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.L * ((a.BH + MB - 1) / MB))), dim3(kGenThreads), lds, st, a, tb);
    return hipGetLastError();
}

LstmForm lstm_generic_form(const LstmArgs &a, int dtype)
{
    // (a workgroup takes a compute unit to itself: see lstm_chain_kernel)
    if (a.d_g <= 64 && (long long)a.L * a.BH <= a.compute_units) return LstmForm::chain;
    // Launches that give every compute unit four sequences put four into a workgroup: W_ih, and W_hh where it is
    // streamed, are then read once for all of them, and the nonlinearities, which bound a full chip, are evaluated once
    // instead of in four quads.  (fp32, one against four per workgroup: 2048 sequences x 64
    // steps at d_g = 64 359 -> 340 us, x 1 step 53 -> 20 us; x 8 steps at d_g = 256 843 -> 324 us.)
    // Above 128 units, where W_hh is streamed and a workgroup has a compute unit to itself, by rounds of the chip: a round of four
    // sequences each takes under two of one (32 steps, one against four: fp32, d_g = 256 369 and 630 us, 512 682 and 1000; bf16,
    // d_g = 200 373 and 681; fp32, 130 535 and 692), but for narrow aligned rows just over (fp32, d_g = 132 165 and 350).
    // 384 sequences, fp32, d_g = 256, once one each until 1024: 718 -> 629 us; 512 x 16 steps at d_g = 512 1365 -> 1000.
    const long long rounds1 = ((long long)a.L * a.BH + a.compute_units - 1) / a.compute_units;
    const long long rounds4 = ((long long)a.L * ((a.BH + 3) / 4) + a.compute_units - 1) / a.compute_units;
    const bool aligned = a.d_g % 4 == 0;
    if (dtype == KVEV_BF16 && a.d_g > 128 && a.d_g <= 192) {
        // Rows kept in registers, one sequence each (four take more registers than there are beside the rows), or read every step by
        // one or four: by their times for a round of the chip, start and steps, in steps of the first (2.9 us at d_g = 163).  They
        // add in the same order, so that a run cut into calls keeps its bits.  Kept / read, us, d = 128: aligned rows (d_g = 164) 32
        // sequences x 1 step 29.8 / 31.2, 1024 x 1 116 / 34 (by four), x 8 175 / 111, x 32 469 / 432; single elements (163) 32 x 1
        // 43 / 41, x 2 45 / 58, 1024 x 1 168 / 44, x 8 228 / 196, x 32 521 / 772.
        const long long n = a.c1 - a.c0, kept = rounds1 * ((aligned ? 9 : 14) + n);
        const long long one = rounds1 * (8 + (aligned ? 3 : 6) * n), four = rounds4 * (7 + (aligned ? 4 : 8) * n);
        return kept <= (one < four ? one : four) ? LstmForm::kept : one <= four ? LstmForm::one : LstmForm::four;
    }
    // (Of many layers of one sequence each there is nothing to share: 300, fp32, d_g = 200 1521 -> 1065; of two it still pays to read
    // each layer's weights once: bf16 1578, one each 1854.)
    const bool chip = (long long)a.L * ((a.BH + 3) / 4) >= a.compute_units;
    const bool rounds = rounds1 >= 2 * rounds4 + (a.d_g < 192 && aligned ? 1 : 0);
    const bool four = (a.d_g <= 128 ? chip : rounds || (chip && a.BH > 1)) && gen_tb(a.d, a.d_g, 4) > 0;
    return four ? LstmForm::four : LstmForm::one;
}

template <typename T, int D>
static hipError_t launch_t(const LstmArgs &a, hipStream_t st)
{
    if ((size_t)a.L * a.BH == 0 || a.c1 == a.c0) return hipSuccess;
    const LstmForm form = lstm_generic_form(a, sizeof(T) == 2 ? KVEV_BF16 : KVEV_F32);
    const bool four = form == LstmForm::four;
    if (form == LstmForm::chain) {
        hipLaunchKernelGGL((lstm_chain_kernel<T, D>), dim3((unsigned)((size_t)a.L * a.BH)), dim3(512), 0, st, a);
        return hipGetLastError();
    }
    if constexpr (sizeof(T) == 2) {
        if (form == LstmForm::kept) return launch_v<T, D, 1, 3, 3>(a, st);
    }
    if (a.d_g <= 64) return four ? launch_v<T, D, 4, 1, 1>(a, st) : launch_v<T, D, 1, 1, 1>(a, st);
    if (a.d_g <= 128) return four ? launch_v<T, D, 4, 2, 2>(a, st) : launch_v<T, D, 1, 2, 2>(a, st);
    return four ? launch_v<T, D, 4, 0, 1>(a, st) : launch_v<T, D, 1, 0, 1>(a, st);
}

hipError_t launch_lstm_generic(const LstmArgs &a, int dtype, hipStream_t st)
{
    if (dtype == KVEV_F32) return a.d == 64 ? launch_t<float, 64>(a, st) : launch_t<float, 128>(a, st);
    return a.d == 64 ? launch_t<bf16_t, 64>(a, st) : launch_t<bf16_t, 128>(a, st);
}

}  // namespace kvev
