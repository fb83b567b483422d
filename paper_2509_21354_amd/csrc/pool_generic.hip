// Chunk aggregation, Eq. 2 of the paper: mean of the chunk's C rows, then the
// d -> d_sum -> d MLP with exact GELU, for keys and values with their own
// weights.  fp32-arithmetic kernel for any storage dtype and any d_sum; the bf16
// fast path lives in pool_mfma.hip, this one serves fp32 storage and widths the
// MFMA tiling does not cover.
//
// A workgroup owns RB (sequence, chunk) rows of one layer: 4 where the launch
// still fills the chip, so that a weight row read from L2 serves four chunks (with
// one chunk per workgroup, fp32, d = d_sum = 128, a chunk of 32 rows asks L2 for eight
// times the bytes that it takes from HBM), else 1.  The rows are streamed by lane
// groups of 16 (16 or 32 bytes per lane and row).  Both layers give a lane group
// four weight rows at a time, 4 elements per lane and load, and fold the 4 (x RB)
// partial dot products over the lanes with a transposing reduction, after which
// every lane holds one output: a GELU is evaluated once, not in 16 lanes.
// Measured (fp32): d = 64, d_sum = 128, 4 sequences x 64 chunks of 16: 21.8 -> 6.1 us; d = 128, 512 x 64 chunks of 32: 713 -> 253 us (4.4 TB/s, the mean
// alone 184 us); the per-token MLP, 64 x 32 chunks of 32: 330 -> 96 us.
#include "common.hpp"
#include "kernels.hpp"

namespace kvev {

constexpr int pool_gen_ap(int ds) { return (ds + 63) / 64 * 64; }

enum { kGenPlain, kGenMlp, kGenTokenMlp };       // mean and maximum; the MLP on the mean; the MLP on every token

// VEC: d_sum is a multiple of 4, so every row of W2 starts where a 4-element load may.
template <typename T, int D, int FORM, int RB, bool VEC>
__global__ __launch_bounds__(256) void pool_generic_kernel(PoolArgs a, int stream)
{
    static_assert(RB == 1 || RB == 4, "a wave per row, or all waves on one");
    constexpr int EPL = D / 16, W = 16 / (int)sizeof(T) < EPL ? 16 / (int)sizeof(T) : EPL, NL = EPL / W;   // NL loads of W elements per row and lane
    constexpr int STRIDE = RB == 1 ? 16 : 4, U = 4, KC = D / 64;
    extern __shared__ __align__(16) float smem[];
    const int ds = a.d_sum, AP = pool_gen_ap(ds);
    float *red = smem;                            // [4 waves][2][D]   partial sums (RB == 1)
    float *mean = red + (RB == 1 ? 4 * 2 * D : 0);    // [RB][2][D]
    float *act = mean + RB * 2 * D;               // [RB][2][AP]   zeros from d_sum on

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, grp = tid >> 4, cl = tid & 15;
    const int nch = a.c1 - a.c0, rows_per_layer = a.BH * nch;
    const int gpl = (rows_per_layer + RB - 1) / RB;
    const int l = blockIdx.x / gpl, r0 = (blockIdx.x % gpl) * RB;
    const int live = min(RB, rows_per_layer - r0);
    const bool is_max = a.mode == KVEV_POOL_MAX;     // element-wise maximum instead of the mean
    // token rows and summary row of the workgroup's row m (past the end: the last one again)
    auto seq_of = [&](int m) __attribute__((always_inline)) { return (size_t)l * a.BH + (r0 + min(m, live - 1)) / nch; };
    auto chunk_of = [&](int m) __attribute__((always_inline)) { return a.c0 + (r0 + min(m, live - 1)) % nch; };
    auto tokens = [&](int m) __attribute__((always_inline)) { return (seq_of(m) * a.T_cap + (size_t)chunk_of(m) * a.C) * D; };
    auto out_row = [&](int m) __attribute__((always_inline)) { return (seq_of(m) * a.N_cap + chunk_of(m)) * D; };

    if constexpr (FORM != kGenPlain) {
        for (int i = tid; i < RB * 2 * AP; i += 256)
            if (i % AP >= ds) act[i] = 0.f;
    }
    if constexpr (FORM == kGenTokenMlp) {
        // the MLP on every token, outputs averaged; layer 2 is linear, so the average is taken over the hidden
        // activations: a lane group keeps four W1 rows in registers and takes four tokens at a time (RB == 1)
        for (int kv = 0; kv < 2; ++kv) {
            const T *X = static_cast<const T *>(kv ? a.V : a.K) + tokens(0) + 4 * cl;
            const T *W1 = static_cast<const T *>(kv ? a.W1V : a.W1K) + (size_t)l * ds * D + 4 * cl;
            const T *b1 = static_cast<const T *>(kv ? a.b1V : a.b1K) + (size_t)l * ds;
            for (int u0 = 4 * grp; u0 < ds; u0 += 64) {
                float w[4][KC][4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int c = 0; c < KC; ++c) VecLoad<T, 4>::run(W1 + (size_t)min(u0 + q, ds - 1) * D + 64 * c, w[q][c]);
                const int u = u0 + value_of_lane(cl);
                const float bias = Storage<T>::load(b1 + min(u, ds - 1));
                float total = 0.f;
                for (int j = 0; j < a.C; j += 4) {
                    float part[4][4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        part[m][0] = part[m][1] = part[m][2] = part[m][3] = 0.f;
#pragma unroll
                        for (int c = 0; c < KC; ++c) {
                            float x[4];
                            VecLoad<T, 4>::run(X + (size_t)min(j + m, a.C - 1) * D + 64 * c, x);
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int e = 0; e < 4; ++e) part[m][q] = fmaf(w[q][c][e], x[e], part[m][q]);
                        }
                    }
                    const float g = gelu_erf(fold16(part, cl) + bias);       // token j + cl / 4
                    total += j + (cl >> 2) < a.C ? g : 0.f;
                }
                total += dpp_move<kRowRor4>(total);
                total += dpp_move<kRowRor8>(total);
                if (cl < 4 && u < ds) act[kv * AP + u] = total / (float)a.C;
            }
        }
        __syncthreads();
    } else {
        // ---- mean (or maximum): lane group g of the wave takes tokens g, g + 4, ... of the wave's row (RB == 4), or
        // group g of the workgroup tokens g, g + 16, ... of the one row.  A token past the chunk is loaded from the last
        // one and gets weight 0 (the maximum needs no weight), so that a batch's loads are all in flight together ----
        const int g = RB == 1 ? grp : grp & 3, mrow = RB == 1 ? 0 : wave;
        const T *Kp = static_cast<const T *>(a.K) + tokens(mrow) + cl * W;
        const T *Vp = static_cast<const T *>(a.V) + tokens(mrow) + cl * W;
        float ak[EPL], av[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) ak[e] = av[e] = is_max ? -INFINITY : 0.f;
        for (int j0 = 0; j0 < a.C; j0 += STRIDE * U) {
            Raw<T, W> xk[U][NL], xv[U][NL];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t off = (size_t)min(j0 + g + STRIDE * u, a.C - 1) * D;
#pragma unroll
                for (int c = 0; c < NL; ++c) {
                    if (stream) { xk[u][c].load_stream(Kp + off + 16 * W * c); xv[u][c].load_stream(Vp + off + 16 * W * c); }
                    else { xk[u][c].load(Kp + off + 16 * W * c); xv[u][c].load(Vp + off + 16 * W * c); }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = j0 + g + STRIDE * u < a.C;
#pragma unroll
                for (int c = 0; c < NL; ++c) {
                    float fk[W], fv[W];
                    xk[u][c].get(fk);
                    xv[u][c].get(fv);
#pragma unroll
                    for (int e = 0; e < W; ++e) {
                        float &k = ak[c * W + e], &v = av[c * W + e];
                        k = is_max ? fmaxf(k, fk[e]) : in ? k + fk[e] : k;
                        v = is_max ? fmaxf(v, fv[e]) : in ? v + fv[e] : v;
                    }
                }
            }
        }
        const float cf = is_max ? 1.f : (float)a.C;
        float *dst = RB == 1 ? red + wave * 2 * D : mean + wave * 2 * D;
        if (is_max) {
            const auto mx = [](float x, float y) __attribute__((always_inline)) { return fmaxf(x, y); };
            rows_fold(ak, mx);
            rows_fold(av, mx);
        } else {
            const auto add = [](float x, float y) __attribute__((always_inline)) { return x + y; };
            rows_fold(ak, add);
            rows_fold(av, add);
        }
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i) {
            const int e = rows_value(i, lane >> 4), at = (e / W) * 16 * W + cl * W + e % W;
            dst[at] = RB == 1 ? ak[i] : ak[i] / cf;
            dst[D + at] = RB == 1 ? av[i] : av[i] / cf;
        }
        __syncthreads();
        if constexpr (RB == 1) {
            if (tid < 2 * D) {
                float sum = red[tid];
#pragma unroll
                for (int w = 1; w < 4; ++w) sum = is_max ? fmaxf(sum, red[w * 2 * D + tid]) : sum + red[w * 2 * D + tid];
                mean[tid] = sum / cf;
            }
            __syncthreads();
        }
        if constexpr (FORM == kGenPlain) {
            for (int i = tid; i < live * 2 * D; i += 256) {
                const int m = i / (2 * D), e = i % D;
                Storage<T>::store(static_cast<T *>(i % (2 * D) < D ? a.Kbar : a.Vbar) + out_row(m) + e, mean[i]);
            }
            return;
        }
        // ---- layer 1: four hidden units per lane group and turn ----
        for (int kv = 0; kv < 2; ++kv) {
            const T *W1 = static_cast<const T *>(kv ? a.W1V : a.W1K) + (size_t)l * ds * D + 4 * cl;
            const T *b1 = static_cast<const T *>(kv ? a.b1V : a.b1K) + (size_t)l * ds;
            for (int u0 = 4 * grp; u0 < ds; u0 += 64) {
                float part[RB][4];
#pragma unroll
                for (int m = 0; m < RB; ++m) part[m][0] = part[m][1] = part[m][2] = part[m][3] = 0.f;
#pragma unroll
                for (int c = 0; c < KC; ++c) {
                    float w[4][4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) VecLoad<T, 4>::run(W1 + (size_t)min(u0 + q, ds - 1) * D + 64 * c, w[q]);
#pragma unroll
                    for (int m = 0; m < RB; ++m) {
                        float x[4];
                        VecLoad<float, 4>::run(mean + (m * 2 + kv) * D + 64 * c + 4 * cl, x);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e) part[m][q] = fmaf(w[q][e], x[e], part[m][q]);
                    }
                }
                const int u = u0 + value_of_lane(cl), m = RB == 4 ? cl >> 2 : 0;
                float z;
                if constexpr (RB == 4) z = fold16(part, cl);
                else z = fold4(part[0], cl);
                z = gelu_erf(z + Storage<T>::load(b1 + min(u, ds - 1)));
                if (u < ds && (RB == 4 || cl < 4)) act[(m * 2 + kv) * AP + u] = z;
            }
        }
        __syncthreads();
    }
    // ---- layer 2: four output elements per lane group and turn ----
    for (int kv = 0; kv < 2; ++kv) {
        const T *W2 = static_cast<const T *>(kv ? a.W2V : a.W2K) + (size_t)l * D * ds;
        const T *b2 = static_cast<const T *>(kv ? a.b2V : a.b2K) + (size_t)l * D;
        for (int e0 = 4 * grp; e0 < D; e0 += 64) {
            float part[RB][4];
#pragma unroll
            for (int m = 0; m < RB; ++m) part[m][0] = part[m][1] = part[m][2] = part[m][3] = 0.f;
            for (int k = 0; k < ds; k += 64) {
                float w[4][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) load4<T, VEC>(W2 + (size_t)(e0 + q) * ds, k + 4 * cl, ds, w[q]);
#pragma unroll
                for (int m = 0; m < RB; ++m) {
                    float x[4];
                    VecLoad<float, 4>::run(act + (m * 2 + kv) * AP + k + 4 * cl, x);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) part[m][q] = fmaf(w[q][e], x[e], part[m][q]);
                }
            }
            const int e = e0 + value_of_lane(cl), m = RB == 4 ? cl >> 2 : 0;
            float z;
            if constexpr (RB == 4) z = fold16(part, cl);
            else z = fold4(part[0], cl);
            if (m < live && (RB == 4 || cl < 4))
                Storage<T>::store(static_cast<T *>(kv ? a.Vbar : a.Kbar) + out_row(m) + e, z + Storage<T>::load(b2 + e));
        }
    }
}

template <typename T, int D, int FORM, int RB>
static hipError_t launch_rb(const PoolArgs &a, hipStream_t st)
{
    const size_t blocks = (size_t)a.L * (((size_t)a.BH * (a.c1 - a.c0) + RB - 1) / RB);
    if (blocks == 0) return hipSuccess;
    const size_t lds = sizeof(float) * ((RB == 1 ? 4 * 2 * D : 0) + (size_t)RB * 2 * (D + (FORM == kGenPlain ? 0 : pool_gen_ap(a.d_sum))));
    // rows that the memory-side cache cannot hold until somebody reads them again carry the non-temporal hint
    const bool stream = (size_t)a.L * a.BH * (a.c1 - a.c0) * a.C * D * 2 * sizeof(T) > ((size_t)256 << 20);
    const auto kernel = a.d_sum % 4 == 0 || FORM == kGenPlain ? pool_generic_kernel<T, D, FORM, RB, true>
                                                              : pool_generic_kernel<T, D, FORM, RB, false>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), lds, st, a, stream ? 1 : 0);
    return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_t(const PoolArgs &a, hipStream_t st)
{
    if (a.mode == KVEV_POOL_TOKEN_MLP) return launch_rb<T, D, kGenTokenMlp, 1>(a, st);
    // four rows per workgroup once that leaves two workgroups for every compute unit (fp32, d = 128, 512 x 64 chunks of 32: 480 us
    // with one row, 255 us with four; the mean alone needs no weights)
    const bool four = (size_t)a.L * a.BH * (a.c1 - a.c0) >= (size_t)8 * a.compute_units;
    if (a.mode != KVEV_POOL_MLP) return launch_rb<T, D, kGenPlain, 1>(a, st);
    // (very wide hidden layers: their activations of four rows would leave one workgroup per compute unit)
    return four && pool_gen_ap(a.d_sum) <= 2048 ? launch_rb<T, D, kGenMlp, 4>(a, st) : launch_rb<T, D, kGenMlp, 1>(a, st);
}

hipError_t launch_pool_generic(const PoolArgs &a, int dtype, hipStream_t st)
{
    if (dtype == KVEV_F32) return a.d == 64 ? launch_t<float, 64>(a, st) : launch_t<float, 128>(a, st);
    return a.d == 64 ? launch_t<bf16_t, 64>(a, st) : launch_t<bf16_t, 128>(a, st);
}

}  // namespace kvev
