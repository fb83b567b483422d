// Retention: top-k by utility (or the threshold rule of section 3.2) over the
// candidate chunks of one sequence; the kept indices come out ascending.  Integer
// output, exact by construction (topk.hpp).
//
// One wave per sequence up to 1024 candidates (no barrier, the scores in
// registers), 16 waves above.  Bound by the chain of the bit search.  Measured
// against ranking every candidate by counting (from graphs): 8192 sequences, 64 of
// 248: 66 -> 8.4 us; 512 sequences, 64 of 504: 37.5 -> 5.5 us; 32 sequences, 32 of
// 120: 6.0 -> 3.0 us; 16 sequences, 1000 of 16384: 33.9 ms -> 17 us.
#include "common.hpp"
#include "kernels.hpp"
#include "topk.hpp"

namespace kvev {

template <int KPL, int NW>
__global__ __launch_bounds__(64 * NW) void select_kernel(SelectArgs a)
{
    using Top = TopK<KPL, NW>;
    __shared__ typename Top::Lds lds;
    const int s = blockIdx.x, tid = threadIdx.x;
    const float *src = (a.mode == KVEV_SELECT_TOPK ? a.util : a.gate) + (size_t)s * a.N_cap;
    float u[KPL];
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int c = Top::index(i);
        u[i] = c < a.n_cand ? src[c] : 0.f;
    }
    bool keep[KPL];
    if (a.mode == KVEV_SELECT_TOPK) {
        uint32_t key[KPL];
#pragma unroll
        for (int i = 0; i < KPL; ++i) key[i] = Top::index(i) < a.n_cand ? topk_key(u[i]) : 0u;
        Top::best(key, a.n_cand, a.k, keep, lds);
    } else {
#pragma unroll
        for (int i = 0; i < KPL; ++i) keep[i] = Top::index(i) < a.n_cand && u[i] >= a.tau;
    }
    int pos[KPL];
    const int kept = Top::before(keep, pos, lds);
    int32_t *out = a.idx + (size_t)s * a.k_cap;
#pragma unroll
    for (int i = 0; i < KPL; ++i)
        if (keep[i] && pos[i] < a.k_cap) out[pos[i]] = Top::index(i);
    if (tid == 0) a.count[s] = min(kept, a.k_cap);
}

hipError_t launch_select(const SelectArgs &a, hipStream_t st)
{
    if (a.S == 0) return hipSuccess;
    const dim3 grid((unsigned)a.S);
    if (a.n_cand <= 128) hipLaunchKernelGGL((select_kernel<2, 1>), grid, dim3(64), 0, st, a);
    else if (a.n_cand <= 256) hipLaunchKernelGGL((select_kernel<4, 1>), grid, dim3(64), 0, st, a);
    else if (a.n_cand <= 512) hipLaunchKernelGGL((select_kernel<8, 1>), grid, dim3(64), 0, st, a);
    else if (a.n_cand <= 1024) hipLaunchKernelGGL((select_kernel<16, 1>), grid, dim3(64), 0, st, a);
    else if (a.n_cand <= 4096) hipLaunchKernelGGL((select_kernel<4, 16>), grid, dim3(1024), 0, st, a);
    else hipLaunchKernelGGL((select_kernel<16, 16>), grid, dim3(1024), 0, st, a);        // (the ABI layer admits 16384 candidates)
    return hipGetLastError();
}

}  // namespace kvev
