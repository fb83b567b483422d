// Decode attention (few queries per sequence): Eq. 1 of the paper evaluated
// over a row list that is either the whole cache (dense baseline) or the kept
// chunk summaries followed by the raw recent window (section 3.3, n' = W + M).
//
// The op moves 2*n*d elements per query and does 4*n*d flops: it is bound by
// HBM, so the kernel is a pure streaming design.  A 16-lane group owns one row
// at a time (one 16-byte load per lane covers a 128-wide bf16 row), a wave
// covers 4 consecutive rows per load instruction and a workgroup 16, so every
// wave-level load is one contiguous 1 KiB piece of the cache.  Each lane group
// keeps its own online-softmax state (m, l, o); the groups are merged by
// lane exchanges, the waves through LDS, and the splits of one sequence inside the
// same launch: every split leaves its partial (o, m, l) in scratch and draws an
// integer ticket; the workgroup that draws the last one merges all partials in
// split order (so the result does not depend on who arrives when, and no float
// atomics are involved) and puts the ticket back to zero.  A workgroup serves up
// to 4 queries that share the rows (the heads of a grouped-query group, a short
// frame).
#include "common.hpp"
#include "kernels.hpp"
#include <algorithm>
#include <type_traits>

namespace kvev {

constexpr float kNegBig = -1.0e30f;   // finite stand-in for -inf: exp2(kNegBig - x) == 0, no NaN
constexpr int kMaxSplit = KVEV_ATTN_MAX_SPLIT;   // most splits per query (the host plans within it)

// Device-scope accesses for what workgroups on different XCDs hand each other: the store writes through the
// XCD's L2, the load reads past the caches that are not coherent across XCDs.
__device__ __forceinline__ void store_device(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_device(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Queries that share a key-value sequence: the Tq queries of each of the G query
// heads of its group (grouped-query attention), numbered r = g * Tq + tq.  Row of
// query r in Q / O [L,B,H,Tq,d] for key-value sequence s of [L,B,H_kv].
__device__ __forceinline__ size_t query_row(const AttnArgs &a, int s, int r)
{
    const int g = r / a.Tq, tq = r - g * a.Tq;
    const size_t head = (size_t)(s / a.Hkv) * ((size_t)a.Hkv * a.G) + (size_t)(s % a.Hkv) * a.G + g;
    return head * a.Tq + tq;
}

// dot product of 16 / sizeof(T) (or fewer) elements of a query and a row, added to acc: bf16 pairs go through the
// two-element dot product (exact products, fp32 sums), which needs no conversion
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot_raw(const Raw<bf16_t, 8> &q, const Raw<bf16_t, 8> &k, float acc)
{
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.x), __builtin_bit_cast(bf16x2_t, k.v.x), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.y), __builtin_bit_cast(bf16x2_t, k.v.y), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.z), __builtin_bit_cast(bf16x2_t, k.v.z), acc, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.w), __builtin_bit_cast(bf16x2_t, k.v.w), acc, false);
}
__device__ __forceinline__ float dot_raw(const Raw<bf16_t, 4> &q, const Raw<bf16_t, 4> &k, float acc)
{
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.x), __builtin_bit_cast(bf16x2_t, k.v.x), acc, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, q.v.y), __builtin_bit_cast(bf16x2_t, k.v.y), acc, false);
}
__device__ __forceinline__ float dot_raw(const Raw<float, 4> &q, const Raw<float, 4> &k, float acc)
{
    return fmaf(q.v.w, k.v.w, fmaf(q.v.z, k.v.z, fmaf(q.v.y, k.v.y, fmaf(q.v.x, k.v.x, acc))));
}

// The scores of 4 rows x NQ queries, summed over the 16 lanes: a lane ends with one of them, of row value_of_lane(lane)
// and query 0 (NQ = 1, the four quads alike), lane / 8 (NQ = 2) or lane / 4 (NQ = 4).
__device__ __forceinline__ float fold_scores(const float (&v)[1][4], int lane) { return fold4(v[0], lane); }
__device__ __forceinline__ float fold_scores(const float (&v)[2][4], int lane) { return fold8(v, lane); }
__device__ __forceinline__ float fold_scores(const float (&v)[4][4], int lane) { return fold16(v, lane); }
// lane L of every 16-lane row to the whole row
template <int L> __device__ __forceinline__ float row_lane(float v) { return dpp_move<0x150 + L>(v); }

// NQ queries of one key-value sequence per workgroup: every row that is loaded
// serves all of them (what grouped-query heads and short query frames are for).
// NW waves per workgroup: 4 normally; 16 when the launch has no more workgroups than the chip has compute units
// (a short cache and few sequences: the rows of a sequence are then spread over four times the lanes).
// A lane group takes 4 rows at a time, with the loads of the next 4 in flight.  The scores of the 4 rows are folded over
// the lanes together (every lane is left with one score, so an exponential is taken once and not in 16 lanes), all on
// the vector unit: summing one score at a time with shuffles kept the LDS pipe busier than the memory.  Measured (from
// graphs): 2048 sequences x 333 rows for 4 queries each 87 -> 66 us (5.3 TB/s); 256 x 2000 rows, 8 queries 112 -> 89 us;
// 512 x 320 rows, one query 16.4 -> 15.7 us; fp32, one query 1024 x 544 rows 102 -> 86 us, four queries 2048 x 320 rows 132 -> 114
// us.  32 x 315 rows: 7.4 us -> 6.25 us, unsplit (launch and three round trips).
template <typename T, int D, int NQ, int NW>
__global__ __launch_bounds__(64 * NW) void attn_decode_kernel(AttnArgs a)
{
    constexpr int U = 4;
    constexpr int EPL = D / 16, GROUPS = 4 * NW;     // elements per lane; 16-lane row groups per workgroup
    constexpr int W = 16 / (int)sizeof(T) < EPL ? 16 / (int)sizeof(T) : EPL, NL = EPL / W;     // NL loads of W elements
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = tid >> 4;      // row group within the workgroup, 0 .. GROUPS-1
    const int cl = tid & 15;       // column lane within the group: elements 16 W c + W cl .. of a row
    const int R = a.G * a.Tq;
    const int qgroups = (R + NQ - 1) / NQ;
    int blk = blockIdx.x;
    const int split = blk % a.nsplit; blk /= a.nsplit;
    const int qg = blk % qgroups;
    const int s = blk / qgroups;

    const T *K = static_cast<const T *>(a.K) + cl * W, *V = static_cast<const T *>(a.V) + cl * W;
    const T *Kbar = static_cast<const T *>(a.Kbar) + cl * W, *Vbar = static_cast<const T *>(a.Vbar) + cl * W;

    // The raw rows are cut into nsplit runs of rows_per_split; the kept summaries go with the first run.  The cut thus
    // depends on the raw rows alone, and the compact form (same raw rows, another capacity for the summaries) walks
    // and merges exactly as the indexed form does.  A workgroup takes its raw rows first: their addresses need
    // nothing from memory, so their loads leave together with those of the queries, the kept count and the first
    // chunk indices, and the summaries' (whose addresses come out of the index list) leave before the raw rows are
    // waited for.
    const int wlen = a.T - a.win0;
    const int w0 = split * a.rows_per_split;
    const int w1 = min(wlen, w0 + a.rows_per_split);
    const int32_t *idx = a.idx ? a.idx + (size_t)s * a.k_cap : nullptr;   // null: the store is compact, row j is entry j
    int cnt_raw = 0;
    if (a.gated && split == 0) cnt_raw = a.count[s];
    int idx0[U];                  // the chunk indices of this lane group's first batch of summaries, asked for early
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int j = grp + GROUPS * u;
        idx0[u] = a.gated && split == 0 && idx && a.k_cap > 0 ? idx[min(j, a.k_cap - 1)] : j;
    }

    Raw<T, W> qv[NQ][NL];
    size_t qrow[NQ];
    bool qok[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int r = qg * NQ + i;
        qok[i] = r < R;
        qrow[i] = query_row(a, s, qok[i] ? r : R - 1);
#pragma unroll
        for (int c = 0; c < NL; ++c) qv[i][c].load(static_cast<const T *>(a.Q) + qrow[i] * D + cl * W + 16 * W * c);
    }
    // this lane's score: its row in a batch, its query, and the first raw row which that query must not see (causal frame:
    // the queries are the last Tq cached tokens and see nothing after their own position; a summary is older than every
    // raw row)
    const int my_u = value_of_lane(cl), my_i = NQ == 4 ? cl >> 2 : NQ == 2 ? cl >> 3 : 0;
    const int my_r = qg * NQ + my_i;
    const int lim = my_r >= R ? -1 : a.causal ? wlen - (a.Tq - 1 - my_r % a.Tq) : wlen;

    float m = kNegBig, l = 0.f;       // of this lane's query; l: of this lane's rows
    float o[NQ][EPL];
#pragma unroll
    for (int i = 0; i < NQ; ++i)
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[i][e] = 0.f;

    const size_t seq_raw = (size_t)s * a.T_cap;
    const size_t seq_sum = (size_t)s * a.N_cap;

    struct Batch { Raw<T, W> k[U][NL], v[U][NL]; int pos; };      // pos: see fold
    // One batch: 4 rows per lane group are scored against the NQ queries and folded into the running softmax.  pos is
    // the position of this lane's row for the causal test: its raw index, -1 for a summary (visible to every query), a
    // huge value for a slot past the end.
    auto fold = [&](const Batch &b) __attribute__((always_inline)) {
        float sc[NQ][U];
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sc[i][u] = 0.f;
#pragma unroll
                for (int c = 0; c < NL; ++c) sc[i][u] = dot_raw(qv[i][c], b.k[u][c], sc[i][u]);
            }
        const bool seen = b.pos < lim;
        const float folded = fold_scores(sc, cl) * a.scale_log2e;       // (by all lanes: they trade partial sums)
        const float x = seen ? folded : kNegBig;
        float mx = fmaxf(x, dpp_move<kQuadXor1>(x));
        mx = fmaxf(mx, dpp_move<kQuadXor2>(mx));
        const float m_new = fmaxf(m, mx);
        if (__any(m_new > m)) {       // (else every alpha is 1)
            const float alpha = exp2f(m - m_new);
            l *= alpha;
            static_for<NQ>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const float al = NQ == 1 ? alpha : row_lane<i * (16 / NQ)>(alpha);
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[i][e] *= al;
            });
            m = m_new;
        }
        const float p = seen ? exp2f(x - m_new) : 0.f;
        l += p;
        static_for<U>([&](auto uc) {
            constexpr int u = decltype(uc)::value, lane_u = (u & 1) * 2 + (u >> 1);     // (the lane of a quad that holds row u)
            float vv[EPL];
#pragma unroll
            for (int c = 0; c < NL; ++c) {
                float t[W];
                b.v[u][c].get(t);
#pragma unroll
                for (int e = 0; e < W; ++e) vv[c * W + e] = t[e];
            }
            static_for<NQ>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const float pi = row_lane<i * (16 / NQ) % 16 + lane_u>(p);
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[i][e] = fmaf(pi, vv[e], o[i][e]);
            });
        });
    };
    constexpr int kPast = 0x3fffffff;

    // Rows are read once per launch.  When a launch reads more than the memory-side cache holds (a.stream), the loads
    // carry the non-temporal hint: nothing of it can be kept anyway, and the read stream runs 13 % faster without
    // the allocations.  Smaller launches keep plain loads, so that the next decode step finds its rows in cache.
    const int nraw = w1 > w0 ? (w1 - w0 + GROUPS * U - 1) / (GROUPS * U) : 0;      // batches of raw rows, then of summaries
    auto walk = [&](auto stream_tag) __attribute__((always_inline)) {
        constexpr bool STREAM = decltype(stream_tag)::value;
        auto fetch = [&](Batch &b, const T *kp, const T *vp, int u, size_t off) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < NL; ++c) {
                if (STREAM) { b.k[u][c].load_stream(kp + off + 16 * W * c); b.v[u][c].load_stream(vp + off + 16 * W * c); }
                else { b.k[u][c].load(kp + off + 16 * W * c); b.v[u][c].load(vp + off + 16 * W * c); }
            }
        };
        // raw rows w0 .. w1-1 of the window (of the whole cache for the dense baseline)
        auto load_raw = [&](int n, Batch &b) __attribute__((always_inline)) {
            const int base = w0 + n * (GROUPS * U) + grp;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int r = a.win0 + min(base + GROUPS * u, w1 - 1) + a.ring_first;       // (ring_first is 0 unless the raw buffer is a ring)
                r = r >= a.T_cap ? r - a.T_cap : r;
                fetch(b, K, V, u, (seq_raw + r) * D);
            }
            const int w = base + GROUPS * my_u;
            b.pos = w < w1 ? w : kPast;
        };
        // the kept summaries (first run only)
        auto load_sum = [&](int n, int cnt, Batch &b) __attribute__((always_inline)) {
            const int base = n * (GROUPS * U) + grp;
            const int c_wave = __builtin_amdgcn_readfirstlane(idx0[0]);      // (all lanes are here)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = base + GROUPS * u, jc = min(j, cnt - 1);
                // idx0[u] is entry min(j, k_cap - 1) of the list: the right one whenever row j exists.  A slot past the
                // count takes the wave's first row instead (there is one: see total).  Its weight is 0, but what a stale
                // entry points to need not be finite (0 x NaN), and may never have been written.
                int c = idx ? (n == 0 ? (j < cnt ? idx0[u] : c_wave) : idx[jc]) : jc;
                c = min(max(c, 0), a.N_cap - 1);
                fetch(b, Kbar, Vbar, u, (seq_sum + c) * D);
            }
            b.pos = base + GROUPS * my_u < cnt ? -1 : kPast;
        };
        Batch b0, b1;
        if (nraw > 0) load_raw(0, b0);
        const int cnt = min(max(cnt_raw, 0), a.k_cap);
        const int wcnt = max(cnt - wave * 4, 0);         // entries from the wave's first on: its last batch holds a row of it
        const int total = nraw + (wcnt + GROUPS * U - 1) / (GROUPS * U);
        auto load = [&](int n, Batch &b) __attribute__((always_inline)) {
            if (n < nraw) load_raw(n, b);
            else load_sum(n - nraw, cnt, b);
        };
        if (nraw == 0 && total > 0) load_sum(0, cnt, b0);
        for (int n = 0; n < total; n += 2) {
            if (n + 1 < total) load(n + 1, b1);
            fold(b0);
            if (n + 1 >= total) break;
            if (n + 2 < total) load(n + 2, b0);
            fold(b1);
        }
    };
    if (a.stream) walk(std::true_type{}); else walk(std::false_type{});

    __shared__ float s_m[NQ][NW], s_l[NQ][NW], s_o[NQ][NW][D];
    {
        // merge the 4 lane groups of the wave
        const float M = rows_max(m), f = exp2f(m - M);
        float lf = l * f;
        lf += dpp_move<kQuadXor1>(lf);
        lf += dpp_move<kQuadXor2>(lf);
        lf = rows_sum(lf);
        if ((tid & 63) < 16 && cl % (16 / NQ) == 0) { s_m[my_i][wave] = M; s_l[my_i][wave] = lf; }
        static_for<NQ>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const float fi = NQ == 1 ? f : row_lane<i * (16 / NQ)>(f);
            float v[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) v[e] = o[i][e] * fi;
            rows_fold(v, [](float x, float y) __attribute__((always_inline)) { return x + y; });
#pragma unroll
            for (int k = 0; k < EPL / 4; ++k) {
                const int e = rows_value(k, (tid & 63) >> 4);
                s_o[i][wave][(e / W) * 16 * W + cl * W + e % W] = v[k];
            }
        });
    }
    __syncthreads();
    if (tid < D) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            if (!qok[i]) continue;
            float M = s_m[i][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[i][w]);
            float L = 0.f, acc = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float f = exp2f(s_m[i][w] - M);
                L += s_l[i][w] * f;
                acc += s_o[i][w][tid] * f;
            }
            if (a.nsplit == 1) {
                Storage<T>::store(static_cast<T *>(a.O) + qrow[i] * D + tid, L > 0.f ? acc / L : 0.f);
            } else {
                float *pp = a.part + (((size_t)s * R + (qg * NQ + i)) * a.nsplit + split) * (D + 2);
                store_device(pp + tid, acc);
                if (tid == 0) { store_device(pp + D, M); store_device(pp + D + 1, L); }
            }
        }
    }
    if (a.nsplit == 1) return;

    // ---- the splits of these queries meet here: the last one to arrive merges them all ----
    // Partials and tickets travel with device-scope accesses (stores that write through the XCD's L2, loads that
    // read past it), so no cache has to be written back or invalidated as a whole.  A workgroup waits until its
    // partial stores are acknowledged, then draws its ticket; the workgroup that draws number nsplit - 1 therefore
    // knows that all partials are in memory.  The merge walks the splits in their own order, whoever arrived last.
    __shared__ int s_last;
    // The wait is spelled out: neither relaxed device-scope stores nor a workgroup-scope release make the compiler wait for
    // vector stores, and the ticket is drawn by one wave for all of them.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this wave's stores have completed
    __syncthreads();
    int32_t *ticket = a.tickets + ((size_t)s * qgroups + qg);
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.nsplit - 1;
    __syncthreads();
    if (!s_last) return;
    // the splits' maxima and sums first, one (query, split) per thread: a single round trip for all of them
    __shared__ float s_pm[NQ][kMaxSplit], s_pl[NQ][kMaxSplit];
    for (int e = tid; e < NQ * a.nsplit; e += 64 * NW) {
        const int i = e / a.nsplit, sp = e - i * a.nsplit;
        const int r = qg * NQ + i;
        if (r < R) {
            const float *ps = a.part + (((size_t)s * R + r) * a.nsplit + sp) * (D + 2);
            s_pm[i][sp] = load_device(ps + D);
            s_pl[i][sp] = load_device(ps + D + 1);
        }
    }
    __syncthreads();
    const int t = tid % D;
    for (int i = tid / D; i < NQ; i += 64 * NW / D) {
        const int r = qg * NQ + i;
        if (r >= R) break;
        const float *p = a.part + ((size_t)s * R + r) * a.nsplit * (D + 2) + t;
        float M = kNegBig;
        for (int sp = 0; sp < a.nsplit; ++sp) M = fmaxf(M, s_pm[i][sp]);
        float L = 0.f, acc = 0.f;
        for (int sp0 = 0; sp0 < a.nsplit; sp0 += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = load_device(p + (size_t)min(sp0 + u, a.nsplit - 1) * (D + 2));
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (sp0 + u < a.nsplit) {
                    const float f = exp2f(s_pm[i][sp0 + u] - M);
                    L = fmaf(s_pl[i][sp0 + u], f, L);
                    acc = fmaf(v[u], f, acc);
                }
            }
        }
        Storage<T>::store(static_cast<T *>(a.O) + query_row(a, s, r) * D + t, L > 0.f ? acc / L : 0.f);
    }
    if (tid == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
}

template <typename T, int D, int NQ>
static hipError_t launch_decode_q(const AttnArgs &a, hipStream_t st)
{
    // waves of the large workgroups: 16 where two batches of rows, the queries and the sums fit 128 registers, else 8
    constexpr int BIG = 2 * 4 * 2 * D / 16 * (int)sizeof(T) / 4 + NQ * (D / 16) * (4 + (int)sizeof(T)) / 4 + 40 <= 124 ? 16 : 8;
    const int R = a.G * a.Tq;
    const size_t blocks = (size_t)a.S * ((R + NQ - 1) / NQ) * a.nsplit;
    if (blocks == 0) return hipSuccess;
    // (a large workgroup takes 128 or 256 rows at a time and is slower to start: runs of up to 320 rows go to 4 waves;
    // 128 sequences x 283 rows: 9.4 us against 11.0 us with 16)
    if (blocks <= 256 && a.rows_per_split > 320)
        hipLaunchKernelGGL((attn_decode_kernel<T, D, NQ, BIG>), dim3((unsigned)blocks), dim3(64 * BIG), 0, st, a);
    else
        hipLaunchKernelGGL((attn_decode_kernel<T, D, NQ, 4>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

// Queries per workgroup.  A workgroup that serves one query is the shortest (four queries: the fold of 16 sums, four weights per
// row), so queries that share rows only share a workgroup where there would be too many of them: one each up to half as many
// workgroups as compute units, then pairs up to three quarters.  Unsplit launches only: the plan's runs, partials and tickets
// are for groups of four.  Every query then reads the rows for itself, each XCD into an L2 of its own, which pays while the rows
// of all workgroups stay there: 24 MiB, a little more for single queries that four would share and for pairs of short runs
// (and for bf16 pairs where the rows of workgroups of four do not stay either).
// Runs of more than 320 raw rows go to 8 or 16 waves: pairs there, in fp32 only of d = 64 and up to 160.
// Four / two / one query a workgroup, us, 287 or 319 rows: d = 128 8 sequences x 4 queries 8.8 / 7.0 / 5.6, 32 x 4 8.8 / 7.1 / 5.6, 40 x
// 4 8.9 / 6.7 / 7.1, 64 x 4 8.9 / 6.8 / 8.7, 96 x 4 8.9 / 7.4 / 16, 64 x 2 - / 7.0 / 5.6; d = 64 16 x 4 7.4 / - / 5.4, 32 x 4 7.4 / - / 5.1,
// 64 x 4 7.5 / 5.9 / -, 64 x 2 - / 6.2 / 5.1; fp32, d = 128, 160 rows 32 x 4 7.6 / - / 5.4, 96 x 4 x 250 8.8 / 10.6 / -.  With kept
// summaries: 287 + 256 rows, d = 128 16 x 4 14.2 / - / 9.3, 48 x 2 - / 11.0 / 11.8, 96 x 4 17.1 / 16.2 / -; 319 + 512 32 x 2 - / 15.6 /
// 17.0, 48 x 2 - / 16.2 / 21.0, 16 x 4 19.6 / 15.6 / 14.8, 48 x 4 19.8 / 22.8 / -, 96 x 4 26.9 /
// 24.1 / -, d = 64 64 x 2 - / 14.0 / 16.1, 48 x 8 16.9 / 21.6 / -; fp32, d = 128, 32 + 256 64 x 2 - / 9.0 / 11.8, 96 x 4 x 340 13.5 / 16.3 / -.
// The choice may look at the kept capacity, which differs between the indexed and the compact form, up to 320 raw rows: there
// all have 4 waves and add in the same order (fold4, fold8, fold16), so that the bits are those of any other choice.
int decode_queries(const AttnArgs &a, size_t elem)
{
    const int64_t R = (int64_t)a.G * a.Tq, one = a.S * R, two = a.S * ((R + 1) / 2), units = a.S * ((R + 3) / 4);
    const int64_t unit = (int64_t)a.rows_all * a.d * 2 * elem, cus = a.compute_units;
    const int most = R >= 4 ? 4 : R >= 2 ? 2 : 1;
    if (a.nsplit > 1) return most;
    if (a.rows_per_split <= 320) {
        if (one <= cus / 2 && one * unit <= (int64_t)(R >= 4 ? 26 : 24) << 20) return 1;
        const bool fit = two * unit <= (int64_t)(a.rows_all <= 352 ? 32 : 24) << 20, neither = elem == 2 && units * unit > 28ll << 20;
        return two <= cus * 3 / 4 && (fit || neither) ? std::min(most, 2) : most;
    }
    return two <= (elem == 2 ? cus * 3 / 4 : a.d == 64 ? cus * 5 / 8 : 0) ? std::min(most, 2) : most;
}

template <typename T, int D>
static hipError_t launch_decode_t(const AttnArgs &a, hipStream_t st)
{
    const int nq = decode_queries(a, sizeof(T));
    return nq == 4 ? launch_decode_q<T, D, 4>(a, st) : nq == 2 ? launch_decode_q<T, D, 2>(a, st) : launch_decode_q<T, D, 1>(a, st);
}

hipError_t launch_attn_decode(const AttnArgs &a, int dtype, hipStream_t st)
{
    // Four queries or more that share bf16 rows, at least one unit (a group of four) per compute unit, unsplit: on the matrix
    // cores, but for short runs of raw rows, where the several workgroups per compute unit here hide each other's starts,
    // and for many units of middling length (this kernel and that one, rows that the memory-side cache holds where they
    // fit it: d = 128, one group of 4, 1024 units x 352 rows 34.6 and 32.0 us, 2048 x 96 25.4 and 27.7 us; two or three groups,
    // 2048 units x 364 67.2 and 67.7 us, 3072 x 364 91 and 94 us, 960 x 364 36 and 32 us, 3072 x 790 207 and 158 us; d = 64, 256 x
    // 352 10.7 and 6.9 us, 512 x 220 and 164 summaries 14.7 and 15.4 us, 2048 x 352 35.1 and 36.4 us, x 1000 89 and 85
    // us).  With fewer queries the vector unit has time to spare (one query: 1024 x 352 28.3 and 31.5 us).
    const int64_t R = (int64_t)a.G * a.Tq, units = a.S * ((R + 3) / 4), cus = a.compute_units;
    const int rows = a.T - a.win0;
    const bool long_enough = a.d == 128 ? rows >= 192 && (R == 4 || units <= 4 * cus || rows >= 600)
                                        : rows >= 320 && (units <= 4 * cus || rows >= 800);
    if (dtype == KVEV_BF16 && R >= 4 && a.nsplit == 1 && units >= cus && long_enough)
        return launch_attn_decode_mfma(a, st);
    if (dtype == KVEV_F32) return a.d == 64 ? launch_decode_t<float, 64>(a, st) : launch_decode_t<float, 128>(a, st);
    return a.d == 64 ? launch_decode_t<bf16_t, 64>(a, st) : launch_decode_t<bf16_t, 128>(a, st);
}

}  // namespace kvev
