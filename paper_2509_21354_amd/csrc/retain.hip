// Physical eviction (sections 3.2-3.3 of the paper: a chunk that is not kept is
// discarded, which is where the memory ratio n / (W + M) of section 3.3 comes
// from).  Per sequence a compact store holds at most k summaries, ascending by
// chunk id, with their ids and scores.  Freshly scored chunks (ids above every
// id in the store) are merged in and the best min(k, count + n_new) under the
// order of the top-k selection (score descending, NaN as minus infinity, ties to
// the lower id) stay.  A chunk that drops out can never return, because the
// scores of old chunks do not change, so the store always equals the top-k over
// every chunk seen so far.
//
// One workgroup per sequence.  Candidates are already in ascending id order
// (store entries, then the new chunks), so once the best k are known, a kept
// candidate's new slot is the number of kept candidates before it: surviving
// store rows only move towards slot 0 and the new rows are appended.  Rows move
// in batches of destination slots: every source of a batch is read into
// registers before the batch is written, and a batch only overwrites slots
// below the sources that later batches still need.
// Measured (from graphs; ranks by counting and 32 rows per pass, also those that stay -> now): 512 sequences, 240 new
// chunks into a store of 64: 13.9 -> 10.6 us, 8 new ones into a full store: 8.6 -> 6.9 us; 64 sequences, 1000 into 128:
// 111 -> 13.7 us; 8192 sequences (bound by HBM), 248 into 64: 121 -> 119 us, 8 into a full store: 92 -> 80 us; 2048
// sequences, 1000 into 256: 310 -> 124 us.  The bound of 8 waves per SIMD keeps the scheduler from holding the search
// and all the row addresses in registers at once: without it the kernel takes 124 registers (244 for more than 512
// candidates) and those three take 136, 94 and 171 us.
#include "common.hpp"
#include "kernels.hpp"
#include "topk.hpp"

namespace kvev {

typedef uint32_t piece_t __attribute__((ext_vector_type(4)));    // a 16-byte piece of a row

constexpr int kRetainPieces = 4;      // 16-byte pieces per thread, tensor and pass: 128, 64 or 32 destination rows of 128, 256 or 512 bytes

// KPL, NW: see topk.hpp.  NW = 1: every wave finds the best k by itself (up to 1024 candidates), which costs no barrier.
template <int KPL, int NW>
__global__ __launch_bounds__(256, 8) void retain_kernel(RetainArgs a)
{
    static_assert(NW == 1 || NW == 4, "one wave each, or the workgroup");
    using Top = TopK<KPL, NW>;
    extern __shared__ unsigned char smem_r[];
    __shared__ typename Top::Lds lds;
    const int s = blockIdx.x, tid = threadIdx.x;
    const int cnt = min(max(a.count[s], 0), a.k_cap);
    const int n = cnt + a.n_new;
    float *s_raw = reinterpret_cast<float *>(smem_r);                  // [n] score as stored (a NaN stays a NaN)
    int *s_src = reinterpret_cast<int *>(s_raw + a.k_cap + a.n_new);   // [k_cap] candidate that lands in each slot

    int32_t *ids = a.ids + (size_t)s * a.k_cap;
    float *uc = a.uc + (size_t)s * a.k_cap;
    const float *un = a.un + (size_t)s * a.n_new_cap;
    // the candidate index is the id order
    uint32_t key[KPL];
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
        const int c = Top::index(i);
        key[i] = 0;
        if (c < n) {
            const float u = c < cnt ? uc[c] : un[c - cnt];
            if (NW > 1 || tid < kWave) s_raw[c] = u;
            key[i] = topk_key(u);
        }
    }
    bool keep[KPL];
    int pos[KPL];
    Top::best(key, n, a.k, keep, lds);
    const int kept = Top::before(keep, pos, lds);             // <= k <= k_cap
#pragma unroll
    for (int i = 0; i < KPL; ++i)
        if (keep[i] && (NW > 1 || tid < kWave)) s_src[pos[i]] = Top::index(i);
    __syncthreads();

    // ids and scores of the new store: through registers, then a barrier, then the write
    for (int p0 = 0; p0 < kept; p0 += 256) {
        const int p = p0 + tid;
        int id = 0;
        float u = 0.f;
        if (p < kept) {
            const int c = s_src[p];
            id = c < cnt ? ids[c] : a.first_chunk + (c - cnt);
            u = s_raw[c];
        }
        __syncthreads();               // slots [p0, p0+256) are sources only of slots >= p0: all read before any is written
        if (p < kept) { ids[p] = id; uc[p] = u; }
    }

    // rows: 16-byte pieces (a row has 8, 16 or 32), `batch` destination slots per pass; a row that keeps its slot stays
    const int vec_shift = a.row_bytes == 128 ? 3 : a.row_bytes == 256 ? 4 : 5, batch = (256 * kRetainPieces) >> vec_shift;
    unsigned char *Kc = static_cast<unsigned char *>(a.Kc) + (size_t)s * a.k_cap * a.row_bytes;
    unsigned char *Vc = static_cast<unsigned char *>(a.Vc) + (size_t)s * a.k_cap * a.row_bytes;
    const unsigned char *Kn = static_cast<const unsigned char *>(a.Kn) + (size_t)s * a.n_new_cap * a.row_bytes;
    const unsigned char *Vn = static_cast<const unsigned char *>(a.Vn) + (size_t)s * a.n_new_cap * a.row_bytes;
    for (int p0 = 0; p0 < kept; p0 += batch) {
        piece_t rk[kRetainPieces], rv[kRetainPieces];
        uint32_t to[kRetainPieces];          // (byte offset in a store of at most 4000 rows)
        const int pieces = min(batch, kept - p0) << vec_shift;
#pragma unroll
        for (int i = 0; i < kRetainPieces; ++i) {
            const int e = tid + 256 * i, p = p0 + (e >> vec_shift), off = (e & ((1 << vec_shift) - 1)) * 16;
            const int c = e < pieces ? s_src[p] : p;
            to[i] = ~0u;
            if (e < pieces && (c != p || c >= cnt)) {           // (slot p < cnt with c == p: an old row that stays)
                to[i] = (uint32_t)(p * a.row_bytes + off);
                const uint32_t from = (uint32_t)((c < cnt ? c : c - cnt) * a.row_bytes + off);
                rk[i] = *reinterpret_cast<const piece_t *>((c < cnt ? Kc : Kn) + from);
                rv[i] = *reinterpret_cast<const piece_t *>((c < cnt ? Vc : Vn) + from);
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kRetainPieces; ++i) {
            if (to[i] != ~0u) {
                *reinterpret_cast<piece_t *>(Kc + to[i]) = rk[i];
                *reinterpret_cast<piece_t *>(Vc + to[i]) = rv[i];
            }
        }
        __syncthreads();
    }
    if (tid == 0) a.count[s] = kept;
}

hipError_t launch_retain(const RetainArgs &a, hipStream_t st)
{
    if (a.S == 0) return hipSuccess;
    const size_t n_max = (size_t)a.k_cap + a.n_new;          // (at most 4000: the ABI layer)
    const size_t lds = n_max * sizeof(float) + (size_t)a.k_cap * sizeof(int) + 16;
    if (n_max <= 128) hipLaunchKernelGGL((retain_kernel<2, 1>), dim3(a.S), dim3(256), lds, st, a);
    else if (n_max <= 256) hipLaunchKernelGGL((retain_kernel<4, 1>), dim3(a.S), dim3(256), lds, st, a);
    else if (n_max <= 512) hipLaunchKernelGGL((retain_kernel<8, 1>), dim3(a.S), dim3(256), lds, st, a);
    else if (n_max <= 1024) hipLaunchKernelGGL((retain_kernel<16, 1>), dim3(a.S), dim3(256), lds, st, a);
    else hipLaunchKernelGGL((retain_kernel<16, 4>), dim3(a.S), dim3(256), lds, st, a);
    return hipGetLastError();
}

}  // namespace kvev
