// Multi-query attention (a new frame of Tq query tokens per sequence), bf16
// storage: Eq. 1 of the paper over the kept summaries + raw window (or the whole
// cache for the dense baseline), on the matrix cores.
//
// With Tq queries sharing every key/value row the op does 4*Tq flop per 2 bytes
// of cache read, which puts it near the machine's ridge: the cache must still be
// read only once per sequence, and the contractions must run on MFMA.
//
// Two kernels share the layout of the work.  attn_mq_kernel (v_mfma_f32_16x16x32_bf16, described here) serves launches
// of few or short frames; attn_mq32_kernel (v_mfma_f32_32x32x16_bf16, described where it stands) those that fill the
// chip.
//
// A workgroup owns 16*QS queries per wave (4 waves) of one sequence and walks the
// rows in tiles of 64.  A tile's K and V rows are copied once, coalesced, into
// LDS (a kept summary is reached through its chunk index); the copy of tile t+1
// is in flight in registers while tile t is computed.  Both products are taken
// transposed, so that the softmax weights never change lanes between the MFMAs:
//   S^T = K Q^T   A = 16 key rows from LDS, B = 16 queries (registers, loaded once);
//                 C puts query l%16 in the lane and 4 keys in its registers;
//   O^T = V^T P^T B = those same registers, rounded to bf16; A = V^T, read from the
//                 row-major LDS tile with the transposing LDS load of gfx950
//                 (ds_read_b64_tr_b16): 16 lanes that each point at 4 consecutive
//                 d of one key receive, per lane, one d of 4 keys.  Two such loads
//                 give a lane its 8 keys in the order the C layout holds them (the
//                 contraction index may be permuted freely as long as A and B agree).
// Online softmax state (m, l) is per query = per lane, shared by 4 lanes through
// two exchanges; the running output is rescaled only when some maximum moved.
// Query tiles of one sequence sit in neighbouring workgroups of the same XCD, so
// the second one finds the cache rows in that XCD's L2.
#include "common.hpp"
#include "kernels.hpp"
#include <utility>

namespace kvev {

constexpr float kNegBigMq = -1.0e30f;

// The two kernels below are this body under two register budgets: launches of at most one workgroup per compute unit are
// latency chains, and the scheduler spends registers on them that would cost a full chip its occupancy (32 sequences x 197
// queries x 312 rows: 11.6 us with the budget of a full chip, 10.1 us with that of two waves per SIMD; 2048 x 256 queries
// the other way round: 307 and 358 us).
template <int D, int QS>
__device__ __forceinline__ void attn_mq_body(const AttnArgs &a, int qtiles, int nblocks)
{
    constexpr int BN = 64, RP = D + 8, KS = D / 32, DT = D / 16, BM = 64 * QS, NT = 256;
    // V rows are padded by 32 bytes: the transposing load has 16 lanes read 8 bytes each from 4 consecutive
    // rows, and a row pitch of 8 banks (mod 64) puts those 16 pieces in 16 different bank pairs; the 16-byte
    // row reads of K want the 16-byte padding instead
    constexpr int RPV = D + 16;
    constexpr int CPT = BN * (D / 8) / NT;          // 16-byte chunks per thread per tile, for K and for V
    __shared__ __align__(16) bf16_t s_k[BN * RP];    // row-major, padded rows
    __shared__ __align__(16) bf16_t s_v[BN * RPV];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    // XCD-aware order: consecutive hardware workgroup ids go round-robin over the 8
    // XCDs; give each XCD a contiguous run of logical ids
    int b = blockIdx.x;
    if (nblocks % 8 == 0) b = (b % 8) * (nblocks / 8) + b / 8;
    const int s = b / qtiles, qt = b % qtiles;

    const bf16_t *K = static_cast<const bf16_t *>(a.K), *V = static_cast<const bf16_t *>(a.V);
    const bf16_t *Kbar = static_cast<const bf16_t *>(a.Kbar), *Vbar = static_cast<const bf16_t *>(a.Vbar);
    int cnt = 0;
    if (a.gated) cnt = min(max(a.count[s], 0), a.k_cap);
    const int nrows = cnt + (a.T - a.win0);
    const int32_t *idx = a.idx ? a.idx + (size_t)s * a.k_cap : nullptr;   // null: compact store, row j is entry j
    const size_t seq_raw = (size_t)s * a.T_cap, seq_sum = (size_t)s * a.N_cap;

    // staging role of this thread: column chunk dc of rows sr, sr + 256/(D/8), ...
    const int dc = tid % (D / 8), sr = tid / (D / 8);
    constexpr int RSTEP = NT / (D / 8);
    u32x4_t kreg[CPT], vreg[CPT];
    // branch-free so that the copies stay in registers while the tile before is computed
#define KVEV_MQ_FETCH(J0)                                                                              \
    _Pragma("unroll") for (int i = 0; i < CPT; ++i)                                                    \
    {                                                                                                  \
        const int j = min((J0) + sr + RSTEP * i, nrows - 1);                                           \
        const bool sm = j < cnt;                                                                       \
        const int c_ = sm ? min(max(idx ? idx[j] : j, 0), a.N_cap - 1) : 0;                            \
        int r_ = a.win0 + (j - cnt) + a.ring_first;                                                    \
        r_ = r_ >= a.T_cap ? r_ - a.T_cap : r_;                                                        \
        const size_t off = (sm ? (seq_sum + c_) : (seq_raw + r_)) * D + dc * 8;                        \
        kreg[i] = *reinterpret_cast<const u32x4_t *>((sm ? Kbar : K) + off);                             \
        vreg[i] = *reinterpret_cast<const u32x4_t *>((sm ? Vbar : V) + off);                             \
    }

    // Tiles that hold raw rows only (all of them for the dense baseline, all but the first one or two
    // otherwise) are fetched through buffer descriptors: one lane offset for all loads, the tile and row
    // step in a scalar register; rows past the end read as zeros (they are masked in the softmax).
    const size_t raw_rows = (size_t)(a.T - a.win0);
    const bool fast = raw_rows * D * sizeof(bf16_t) < ((size_t)1 << 32) && a.ring_first == 0;   // (a ring wraps: no linear tile addresses)
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(K + (seq_raw + a.win0) * D, (uint32_t)(raw_rows * D * sizeof(bf16_t)));
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(V + (seq_raw + a.win0) * D, (uint32_t)(raw_rows * D * sizeof(bf16_t)));
    const uint32_t voff = (uint32_t)((sr * D + dc * 8) * sizeof(bf16_t));
#define KVEV_MQ_FETCH_RAW(J0)                                                                          \
    _Pragma("unroll") for (int i = 0; i < CPT; ++i)                                                    \
    {                                                                                                  \
        const uint32_t soff = (uint32_t)(((J0) - cnt + RSTEP * i) * D * (int)sizeof(bf16_t));          \
        kreg[i] = buffer_load16<u32x4_t>(rk, voff, soff);                                              \
        vreg[i] = buffer_load16<u32x4_t>(rv, voff, soff);                                              \
    }
#define KVEV_MQ_FETCH_ANY(J0)                                                                          \
    if (fast && (J0) >= cnt) { KVEV_MQ_FETCH_RAW(J0) } else { KVEV_MQ_FETCH(J0) }

    // queries of this wave: sub-tile u holds query qt*BM + wave*16*QS + u*16 + n
    // (queries that share the sequence: the Tq queries of each of the G heads of its group, r = g*Tq + tq)
    bf16x8_t qf[QS][KS];
    int qrow[QS], lim[QS];
    size_t orow[QS];
    const int R = a.G * a.Tq;
#pragma unroll
    for (int u = 0; u < QS; ++u) {
        qrow[u] = qt * BM + (wave * QS + u) * 16 + n;
        const int rc = min(qrow[u], R - 1);
        const int gq = rc / a.Tq, tq = rc - gq * a.Tq;
        orow[u] = ((size_t)(s / a.Hkv) * ((size_t)a.Hkv * a.G) + (size_t)(s % a.Hkv) * a.G + gq) * a.Tq + tq;
        // causal frame: the queries are the last Tq cached tokens; rows after a query's own token are hidden
        lim[u] = a.causal ? nrows - (a.Tq - 1 - tq) : nrows;
        const bf16_t *Qp = static_cast<const bf16_t *>(a.Q) + orow[u] * D + g * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[u][ks] = *reinterpret_cast<const bf16x8_t *>(Qp + ks * 32);
    }

    float m[QS], lsum[QS];
    f32x4_t o[QS][DT];
#pragma unroll
    for (int u = 0; u < QS; ++u) {
        m[u] = kNegBigMq;
        lsum[u] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[u][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    const float c = a.scale_log2e;

    if (nrows > 0) { KVEV_MQ_FETCH_ANY(0) }
    for (int j0 = 0; j0 < nrows; j0 += BN) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            *reinterpret_cast<u32x4_t *>(s_k + (size_t)(sr + RSTEP * i) * RP + dc * 8) = kreg[i];
            *reinterpret_cast<u32x4_t *>(s_v + (size_t)(sr + RSTEP * i) * RPV + dc * 8) = vreg[i];
        }
        __syncthreads();
        if (j0 + BN < nrows) { KVEV_MQ_FETCH_ANY(j0 + BN) }   // next tile's copy rides under this tile's math
        const bool full = j0 + BN <= nrows - (a.causal ? a.Tq - 1 : 0);    // no row of the tile is hidden from any query

        // ---- S^T = K Q^T: every K fragment read from LDS serves all QS query sub-tiles of the wave ----
        f32x4_t st[QS][4];
#pragma unroll
        for (int u = 0; u < QS; ++u)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) st[u][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const bf16x8_t kf = *reinterpret_cast<const bf16x8_t *>(s_k + (size_t)(kt * 16 + n) * RP + ks * 32 + g * 8);
#pragma unroll
                for (int u = 0; u < QS; ++u)
                    st[u][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[u][ks], st[u][kt], 0, 0, 0);
            }
        // ---- online softmax for this lane's queries (raw scores; scale folded into exp2) ----
        bf16x8_t pb[QS][2];
#pragma unroll
        for (int u = 0; u < QS; ++u) {
            if (!full) {
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (j0 + kt * 16 + 4 * g + r >= lim[u]) st[u][kt][r] = kNegBigMq;
            }
            float mx = kNegBigMq;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, st[u][kt][r]);
            mx = rows_max(mx);
            const float m_new = fmaxf(m[u], mx);
            if (__any(m_new > m[u])) {
                const float alpha = __builtin_amdgcn_exp2f((m[u] - m_new) * c);
                lsum[u] *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[u][dt][r] *= alpha;
                m[u] = m_new;
            }
            const float mc = -m_new * c;
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                float p[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(fmaf(st[u][2 * h2 + (e >> 2)][e & 3], c, mc));   // masked: exp2(-huge) = 0
                    lsum[u] += p[e];
                }
                pb[u][h2] = __builtin_bit_cast(bf16x8_t, make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]),
                                                                     pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7])));
            }
        }
        // ---- O^T += V^T P^T: every V^T fragment serves all QS sub-tiles ----------------
        // transposing load: source lane i of a 16-lane block points at key 4g + i/4,
        // d = 16 dt + 4 (i%4) .. +3; destination lane i receives d = 16 dt + i of keys
        // 4g .. 4g+3.  The second load does the same 16 keys further (registers e >= 4).
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const bf16_t *src = s_v + (size_t)(h2 * 32 + 4 * g + (n >> 2)) * RPV + dt * 16 + 4 * (n & 3);
                const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)src);
                const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(src + 16 * RPV));
                const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int u = 0; u < QS; ++u)
                    o[u][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pb[u][h2], o[u][dt], 0, 0, 0);
            }
        __syncthreads();
    }

#pragma unroll
    for (int u = 0; u < QS; ++u) {
        const float l = rows_sum(lsum[u]);
        if (qrow[u] < R) {
            const float inv = l > 0.f ? 1.0f / l : 0.f;
            bf16_t *Op = static_cast<bf16_t *>(a.O) + orow[u] * D + 4 * g;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                uint2 w;
                w.x = pack_bf16x2(o[u][dt][0] * inv, o[u][dt][1] * inv);
                w.y = pack_bf16x2(o[u][dt][2] * inv, o[u][dt][3] * inv);
                *reinterpret_cast<uint2 *>(Op + dt * 16) = w;
            }
        }
    }
}

template <int D, int QS>
__global__ __launch_bounds__(256, 2) void attn_mq_kernel(AttnArgs a, int qtiles, int nblocks)
{
    attn_mq_body<D, QS>(a, qtiles, nblocks);
}
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_mq_small_kernel(AttnArgs a, int qtiles, int nblocks)
{
    attn_mq_body<D, 1>(a, qtiles, nblocks);
}

#undef KVEV_MQ_FETCH
#undef KVEV_MQ_FETCH_RAW
#undef KVEV_MQ_FETCH_ANY

// ---- launches that fill the chip ------------------------------------------------------------------------------------
// The same products with 32 queries per wave on v_mfma_f32_32x32x16_bf16 (C: query lane % 32, 16 of 32 keys in a lane's
// registers).  What bounds it: power on long rows (32768 rows: the chip clocks it at 1.65 GHz, matrix cores 52 %,
// vector unit 51 % busy, 19 % of it together; a bf16 product of 8192^3 reaches 1.27 PFLOP/s here), on short ones the
// ends of an item (640 rows: 35, 46 and 14 % at 2.0 GHz; 51 % of the HBM peak).  What is different from the kernel above:
//   * a 32 x 32 x 16 instruction takes half the LDS fragments per flop, and vector instructions run beside it that do not
//     beside a 16 x 16 x 32 one (two waves per SIMD, 128 matrix clocks against 16 fma + 4 exp2 per wave: 140 clocks
//     together, 202 with the smaller one);
//   * fragments are asked for RING steps ahead of their use, and the softmax weights of a step are made between the
//     products of the step before;
//   * rows are copied straight into LDS (no registers, no LDS stores by the waves), NB - 1 tiles ahead, one barrier per
//     tile;
//   * workgroups stay: one (8 waves, 256 queries) or two (4 waves, 128 queries) per compute unit walk the items, and the
//     copies run on into the next item's tiles; its queries are asked for before the last product of this one's;
//   * results leave through LDS in whole lines (with 32 bytes of 32 rows per store instruction: 3 us more at the first shape).
// Measured in turn on changing inputs, kernel above (8 or 4 waves) and this one: 2048 sequences x 256 queries x 640 rows,
// d = 128: 283 and 242 us; 512 x 256 x 8192: 644 and 629 us (873 TFLOP/s); 1024 causal x 300 x 476: 213 and 145 us; 512 x 160 x
// 364: 48.0 and 42.2 us; d = 64, 4096 x 256 x 768: 385 and 350 us.  Tried and dropped: weights against a maximum that may lag
// by a factor 2^8, which spares the rescaling (235 us at the first shape, but the largest weight is then rounded like the
// others: 4 % more error); the queries through the slots of the tile stream (240 us); a barrier for every second tile
// (no difference); query loads a tile earlier, in registers of their own (no difference).
template <int D, int NWV, int NB> struct Mq32 {
    static constexpr int BN = 64, KS = D / 16, DT = D / 32, BM = 32 * NWV, CPR = D / 8;     // CPR: 16-byte pieces of a row
    static constexpr int TB = BN * D * 2;                   // bytes of a tile of K or of V
    static constexpr int RPI = 512 / D;                     // rows of one 1 KiB copy instruction
    static constexpr int PER = TB / 1024 / NWV;             // copy instructions per wave and tile, for K and for V
    static constexpr int STAGE = 4096;                      // of a wave's results on their way out: 32 rows of 128 bytes
    static constexpr int lds = NB * 2 * TB + NWV * STAGE;
    static_assert(TB % (1024 * NWV) == 0 && (RPI * NWV) % 16 == 0, "a wave's copies of a tile lie a multiple of 16 rows apart");
    // Rows lie unpadded in LDS (the copies write runs of 1 KiB); piece c of a row is put at c ^ swz(row) instead, so that
    // the 16-byte reads of K (16 lanes: one piece of 16 rows) and the transposing reads of V (32 lanes: four pieces of
    // four rows) touch every bank once.
    static __device__ __forceinline__ int swz_k(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
    static __device__ __forceinline__ int swz_v(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};


template <int D, int NWV, int NB, bool STREAM>
__global__ __launch_bounds__(64 * NWV, NWV == 4 ? 2 : 1) void attn_mq32_kernel(AttnArgs a, int qtiles, int items)
{
    using M = Mq32<D, NWV, NB>;
    constexpr int BN = M::BN, KS = M::KS, DT = M::DT, PER = M::PER, TB = M::TB, RPI = M::RPI, RB = D * 2, RING = 6;
    extern __shared__ __align__(1024) unsigned char smem_mq[];
    lds_byte_t *lds = (lds_byte_t *)smem_mq;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;

    // This workgroup's items (query tile qt of sequence s).  Workgroups go round-robin over the 8 XCDs; an XCD takes a
    // contiguous run of items, in proportion to its workgroups, so that the query tiles of a sequence meet in its L2.
    const int xcd = blockIdx.x & 7, step = ((int)gridDim.x + 7 - xcd) >> 3;          // (step: workgroups of this XCD)
    const int before = xcd * ((int)gridDim.x >> 3) + min(xcd, (int)gridDim.x & 7);   // workgroups of the XCDs before it
    const int it_first = (int)((int64_t)items * before / gridDim.x) + (int)(blockIdx.x >> 3);
    const int it_end = (int)((int64_t)items * (before + step) / gridDim.x);

    const unsigned char *K = static_cast<const unsigned char *>(a.K), *V = static_cast<const unsigned char *>(a.V);
    const unsigned char *Kbar = static_cast<const unsigned char *>(a.Kbar), *Vbar = static_cast<const unsigned char *>(a.Vbar);
    auto kept_of = [&](int s) { return a.gated ? min(max(((const_int_t *)(uintptr_t)a.count)[s], 0), a.k_cap) : 0; };

    // ---- the copies: one stream of tiles over all items of the workgroup, NB - 1 tiles ahead of the products ----
    int f_it = it_first, f_s = 0, f_j0 = 0, f_cnt = 0, f_nrows = 0;       // next tile to copy
    int f_slot = 0, ahead = 0;                                            // its slot; tiles copied and not yet waited for
    auto open_item = [&]() {                                              // on to the next item that has rows
        for (; f_it < it_end; f_it += step) {
            f_s = f_it / qtiles;
            f_cnt = kept_of(f_s);
            f_nrows = f_cnt + (a.T - a.win0);
            f_j0 = 0;
            if (f_nrows > 0) break;
        }
    };
    const int lr = lane / M::CPR, pc = lane % M::CPR;
    const int ck = (pc ^ M::swz_k(RPI * wave + lr)) * 16, cv = (pc ^ M::swz_v(RPI * wave + lr)) * 16;
    auto copy_tile = [&]() {
        if (f_it >= it_end) return;
        const size_t seq_raw = (size_t)f_s * a.T_cap, seq_sum = (size_t)f_s * a.N_cap;
        auto raw_row = [&](int j) __attribute__((always_inline)) {
            int r = a.win0 + (j - f_cnt) + a.ring_first;
            r = r >= a.T_cap ? r - a.T_cap : r;
            return (seq_raw + r) * RB;
        };
        auto copy = [&](int q, const unsigned char *kp, const unsigned char *vp) __attribute__((always_inline)) {
            const uint32_t dst = (uint32_t)(uintptr_t)lds + f_slot * 2 * TB + q * 1024;
            copy_to_lds<STREAM>(kp + ck, dst);
            copy_to_lds<STREAM>(vp + cv, dst + TB);
        };
        if (f_j0 >= f_cnt && f_j0 + BN <= f_nrows) {                      // raw rows only
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const size_t off = raw_row(f_j0 + RPI * (wave + NWV * i) + lr);
                copy(wave + NWV * i, K + off, V + off);
            }
        } else {
            const_int_t *idx = (const_int_t *)(uintptr_t)(a.idx ? a.idx + (size_t)f_s * a.k_cap : nullptr);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int q = wave + NWV * i, jb = f_j0 + RPI * q, j = jb + lr;
                const unsigned char *kp = kZeroRow, *vp = kZeroRow;       // (rows past the end: masked in the softmax)
                if (j >= f_cnt && j < f_nrows) {
                    const size_t off = raw_row(j);
                    kp = K + off;
                    vp = V + off;
                }
                if (jb < f_cnt) {                                         // some of these rows are summaries
                    int c = j;                                            // (null list: compact store, row j is entry j)
                    if (a.idx) {
                        c = 0;
#pragma unroll
                        for (int e = 0; e < RPI; ++e) {
                            const int ce = idx[min(jb + e, f_cnt - 1)];
                            c = lr == e ? ce : c;
                        }
                    }
                    const size_t off = (seq_sum + min(max(c, 0), a.N_cap - 1)) * RB;
                    if (j < f_cnt) { kp = Kbar + off; vp = Vbar + off; }
                }
                copy(q, kp, vp);
            }
        }
        f_slot = f_slot + 1 == NB ? 0 : f_slot + 1;
        ++ahead;
        f_j0 += BN;
        if (f_j0 >= f_nrows) { f_it += step; open_item(); }
    };
    // the oldest tile of this wave's copies has landed (loads return in order: those of younger tiles may be in flight)
    auto wait_tile = [&]() {
        if (NB >= 4 && ahead >= 3) wait_vmem<4 * PER>();
        else if (NB >= 3 && ahead >= 2) wait_vmem<2 * PER>();
        else wait_vmem<0>();
        --ahead;
    };
    open_item();
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) copy_tile();

    const int R = a.G * a.Tq;
    const float c = a.scale_log2e;
    // K fragments: row 32 kb + n, piece 2 ks + h; V fragments by transposing loads (see the header), key 16 s + 8 p + 4 h + i / 4,
    // d = 32 dt + 16 (lane / 16 % 2) + 4 (i % 4) of lane i of 16
    const int k_rd = n * RB + ((h ^ M::swz_k(n)) << 4);                   // ^ (ks << 5)
    const int i16 = lane & 15, v_row = 4 * h + (i16 >> 2);
    const int v_rd = TB + v_row * RB + (((2 * ((lane >> 4) & 1) + ((i16 >> 1) & 1)) ^ M::swz_v(v_row)) << 4) + 8 * (i16 & 1);   // ^ (dt << 6)

    // this lane's query of an item (of those that share the sequence: of each of the G heads of its group the Tq tokens; rows
    // s R .. s R + R - 1 of Q and O)
    int qrow, orow;                       // (at most 2^26 rows)
    auto locate = [&](int it) {
        const int s = it / qtiles;
        qrow = (it - s * qtiles) * M::BM + wave * 32 + n;
        orow = s * R + min(qrow, R - 1);
    };
    bf16x8_t qf[KS];
    auto load_q = [&]() {
        const bf16_t *Qp = static_cast<const bf16_t *>(a.Q) + (size_t)orow * D + h * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8_t *>(Qp + ks * 16);
    };
    // (the queries are waited for where this stands, not at their first use behind copies of later tiles)
    auto wait_q = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
    };
    if (it_first < it_end) {
        locate(it_first);
        load_q();
        wait_q();
    }

    int slot = 0;
    for (int it = it_first; it < it_end; it += step) {
        const int cnt = kept_of(it / qtiles), nrows = cnt + (a.T - a.win0);
        // causal frame: the queries are the last Tq cached tokens; rows after a query's own token are hidden
        const int lim = a.causal ? nrows - (a.Tq - 1 - min(qrow, R - 1) % a.Tq) : nrows;
        const int o_row = qrow < R ? orow : -1;
        float m = kNegBigMq, lsum = 0.f;
        f32x16_t o[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;

        const bool busy = (it % qtiles) * M::BM + wave * 32 < R;      // this wave has queries of the item
        auto next_q = [&]() __attribute__((always_inline)) {
            if (it + step < it_end) {
                locate(it + step);
                load_q();
            }
        };
        auto tile_step = [&](int j0, auto lastc) __attribute__((always_inline)) {
            constexpr bool last = decltype(lastc)::value;      // of the item: the next item's queries are asked for
            wait_tile();
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
            __builtin_amdgcn_s_barrier();            // the tile is there for all waves, and nobody reads the one before
            asm volatile("" : : : "memory");
            copy_tile();
            const lds_byte_t *tile = lds + slot * 2 * TB;
            slot = slot + 1 == NB ? 0 : slot + 1;
            const bool full = j0 + BN <= nrows - (a.causal ? a.Tq - 1 : 0);    // no row of the tile is hidden from any query

            if (!busy) {
                if constexpr (last) next_q();
                return;
            }
            // ---- S^T = K Q^T; fragments come from LDS RING steps ahead ----
            f32x16_t st[2];
            bf16x8_t ring[RING];
            auto read_k = [&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                ring[i % RING] = *(const __attribute__((address_space(3))) bf16x8_t *)(tile + (k_rd ^ ((i / 2) << 5)) + (i % 2) * 32 * RB);
            };
            auto read_v = [&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, sx = i / DT, dt = i % DT;
                const lds_byte_t *src = tile + (v_rd ^ (dt << 6)) + 16 * sx * RB;
                const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)src);
                const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(src + 8 * RB));
                ring[i % RING] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            static_for<RING>(read_k);
            __builtin_amdgcn_sched_barrier(0);
            static_for<2 * KS>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, ks = i / 2, kb = i % 2;
                const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                st[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i % RING], qf[ks], ks == 0 ? zero : st[kb], 0, 0, 0);
                if constexpr (i + RING < 2 * KS) read_k(std::integral_constant<int, i + RING>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            static_for<RING>(read_v);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (last) next_q();
            __builtin_amdgcn_sched_barrier(0);
            // ---- online softmax of this lane's query over its half of the keys: register r of block kb is key
            //      32 kb + 8 (r / 4) + 4 h + r % 4 (raw scores; the scale is folded into exp2) ----
            if (!full) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (j0 + 32 * kb + 8 * (r >> 2) + 4 * h + (r & 3) >= lim) st[kb][r] = kNegBigMq;
            }
            float mx = max3(st[0][0], st[0][1], st[1][0]), my = max3(st[0][2], st[0][3], st[1][1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2) {
                mx = max3(mx, st[1][r], st[1][r + 1]);
                if (r > 2) my = max3(my, st[0][r], st[0][r + 1]);
            }
            mx = fmaxf(mx, my);
            my = mx;
            swap32(mx, my);
            mx = max3(m, mx, my);
            if (__ballot(mx > m)) {
                const float alpha = __builtin_amdgcn_exp2f((m - mx) * c);
                m = mx;
                lsum *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
            }
            // ---- O^T += V^T P^T: step sx takes keys 16 sx .. 16 sx + 15 in the order in which the score registers hold
            //      them; the weights of the next step are made under the products of this one ----
            const float mc = -m * c;
            uint32_t pw[2][4];
            float p_even = 0.f;
            auto weights = [&](auto sxc, auto ec) __attribute__((always_inline)) {          // of keys 2 e, 2 e + 1 of step sx
                constexpr int sx = decltype(sxc)::value, e = decltype(ec)::value;
                const float p0 = __builtin_amdgcn_exp2f(fmaf(st[sx >> 1][8 * (sx & 1) + 2 * e], c, mc));          // masked: exp2(-huge) = 0
                const float p1 = __builtin_amdgcn_exp2f(fmaf(st[sx >> 1][8 * (sx & 1) + 2 * e + 1], c, mc));
                lsum += p0;
                p_even += p1;
                pw[sx & 1][e] = pack_bf16x2(p0, p1);
            };
            static_for<4>([&](auto ec) __attribute__((always_inline)) { weights(std::integral_constant<int, 0>{}, ec); });
            static_for<4 * DT>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, sx = i / DT, dt = i % DT;
                const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, make_uint4(pw[sx & 1][0], pw[sx & 1][1], pw[sx & 1][2], pw[sx & 1][3]));
                o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i % RING], pb, o[dt], 0, 0, 0);
                if constexpr (i + RING < 4 * DT) read_v(std::integral_constant<int, i + RING>{});
                if constexpr (sx < 3)
                    static_for<4 / DT>([&](auto kc) __attribute__((always_inline)) {
                        weights(std::integral_constant<int, (sx + 1) & 3>{}, std::integral_constant<int, dt * (4 / DT) + decltype(kc)::value>{});
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
            lsum += p_even;
        };
        if (nrows > 0) {
            int j0 = 0;
            for (; j0 + BN < nrows; j0 += BN) tile_step(j0, std::false_type{});
            tile_step(j0, std::true_type{});
        } else {
            next_q();
        }
        wait_q();

        float lo = lsum;
        swap32(lsum, lo);
        const float l = lsum + lo, inv = l > 0.f ? 1.0f / l : 0.f;
        // Out through LDS, so that a store instruction writes whole lines (8 rows x 128 bytes) instead of 32 bytes of 32 rows.
        lds_byte_t *stage = lds + NB * 2 * TB + wave * M::STAGE;
        const int st_row = lane >> 3, st_piece = lane & 7;
#pragma unroll
        for (int half = 0; half < D / 64; ++half) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // registers 8 g + 0..3 and 8 g + 4..7 are d = 32 dt + 16 g + 4 h + 0..3 and + 8: after the exchanges a lane holds 8 in a row
                const int dt = 2 * half + (k >> 1), g = k & 1;
                uint32_t w0[2], w1[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    w0[e] = pack_bf16x2(o[dt][8 * g + 2 * e] * inv, o[dt][8 * g + 2 * e + 1] * inv);
                    w1[e] = pack_bf16x2(o[dt][8 * g + 4 + 2 * e] * inv, o[dt][8 * g + 4 + 2 * e + 1] * inv);
                    const auto x = __builtin_amdgcn_permlane32_swap(w0[e], w1[e], false, false);
                    w0[e] = x[0];
                    w1[e] = x[1];
                }
                *(__attribute__((address_space(3))) u32x4_t *)(stage + n * 128 + (((2 * k + h) ^ ((n >> 1) & 7)) << 4)) = u32x4_t{w0[0], w0[1], w1[0], w1[1]};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 8 * i + st_row, out = __shfl(o_row, row);
                const u32x4_t w = *(__attribute__((address_space(3))) u32x4_t *)(stage + row * 128 + ((st_piece ^ ((row >> 1) & 7)) << 4));
                if (out >= 0) {
                    *reinterpret_cast<u32x4_t *>(static_cast<bf16_t *>(a.O) + (size_t)out * D + half * 64 + st_piece * 8) = w;
                    hold_store_data(w);
                }
            }
        }
    }
}

template <int D, int NWV, int NB, bool STREAM>
static hipError_t launch_mq32_t(const AttnArgs &a, hipStream_t st)
{
    using M = Mq32<D, NWV, NB>;
    const int qtiles = (a.G * a.Tq + M::BM - 1) / M::BM;
    const int64_t items = (int64_t)a.S * qtiles, fit = (int64_t)a.compute_units * (NWV == 4 ? 2 : 1);
    static std::atomic<uint64_t> done{0};
    const hipError_t e = allow_lds(attn_mq32_kernel<D, NWV, NB, STREAM>, M::lds, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attn_mq32_kernel<D, NWV, NB, STREAM>), dim3((unsigned)(items < fit ? items : fit)), dim3(64 * NWV), M::lds, st, a, qtiles, (int)items);
    return hipGetLastError();
}
template <int D, int NWV, int NB>
static hipError_t launch_mq32(const AttnArgs &a, hipStream_t st)
{
    // rows that a single query tile reads, and that no cache can hold until the next call, carry the non-temporal hint
    return a.stream && a.G * a.Tq <= 32 * NWV ? launch_mq32_t<D, NWV, NB, true>(a, st) : launch_mq32_t<D, NWV, NB, false>(a, st);
}

template <int D, int QS>
static hipError_t launch_mq_t(const AttnArgs &a, hipStream_t st)
{
    const int qtiles = (a.G * a.Tq + 64 * QS - 1) / (64 * QS);
    const size_t blocks = (size_t)a.S * qtiles;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((attn_mq_kernel<D, QS>), dim3((unsigned)blocks), dim3(256), 0, st, a, qtiles, (int)blocks);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_mq_d(const AttnArgs &a, hipStream_t st)
{
    const int64_t R = (int64_t)a.G * a.Tq, cus = a.compute_units;
    const int rows = a.T - a.win0;
    // Launches that leave compute units idle with 128 or 256 queries per workgroup take smaller query tiles: 64 queries
    // while those are at most one workgroup per compute unit (64 sequences x 256 queries x 2048 rows: 41 us, 54 us with
    // 128 queries, 72 us with 256).
    const int64_t tiles64 = a.S * ((R + 63) / 64), tiles128 = a.S * ((R + 127) / 128), tiles256 = a.S * ((R + 255) / 256);
    if (tiles64 > 0 && tiles64 <= cus) {
        hipLaunchKernelGGL((attn_mq_small_kernel<D>), dim3((unsigned)tiles64), dim3(256), 0, st, a, (int)((R + 63) / 64), (int)tiles64);
        return hipGetLastError();
    }
    // Up to 64 queries: the 64-query tiles, whose several workgroups per compute unit hide each other's waits, unless the
    // launch reads more than the caches hold over many sequences: then the deeper copies win (d = 128, 64 queries, old and
    // new: 1020 sequences x 1000 rows 109 and 97 us, 2040 x 350 90 and 79 us; 600 x 1000 66 and 67 us; d = 64 1020 x 1000
    // 47 and 51 us).  Counted by the raw rows alone, as every choice here: the compact and the indexed form over the same rows
    // have other capacities for the summaries and must sum in the same order (a.stream counts those too).
    if (R <= 64) {
        if (D == 128 && (size_t)a.S * rows * D * 2 * sizeof(bf16_t) > kCacheBytes && a.S >= 3 * cus) return launch_mq32<D, 4, D == 128 ? 2 : 4>(a, st);
        return launch_mq_t<D, 1>(a, st);
    }
    // Up to 128 queries: at d = 64 the workgroups of attn_mq_kernel are small enough to sit three to a compute unit (1020 x
    // 128 x 350: 27.6 and 29.2 us); at d = 128 they are only worth it for a few short rows (400 x 80 x 100: 10.9 and 11.4
    // us, x 350: 22.5 and 20.3 us; 600 x 80 x 100: 19.1 and 16.9 us).
    if (R <= 128) {
        if (D == 64 || (a.S <= 2 * cus && rows < 192)) return launch_mq_t<D, 2>(a, st);
        return launch_mq32<D, 4, D == 128 ? 2 : 4>(a, st);
    }
    // More: 8 waves on 256 queries stage a tile once for all of them; 4 waves on 128 leave less of a ragged frame's last
    // tile, and of the launch's last round, unused.  Times in units of one 256-query item on a compute unit of its own: two
    // 128-query items beside each other take 1.12, one alone 0.65 (512 x 256 x 8192: 596 and 670 us; 300 x 160 x 1000: 66
    // and 55 us; 100 x 300 x 1000: 35 and 38 us).
    const double t256 = (double)((tiles256 + cus - 1) / cus);
    const int64_t rest = tiles128 % (2 * cus);
    const double t128 = 1.12 * (double)(tiles128 / (2 * cus)) + (rest == 0 ? 0.0 : rest <= cus ? 0.65 : 1.12);
    if (t128 < t256) return launch_mq32<D, 4, D == 128 ? 2 : 4>(a, st);
    return launch_mq32<D, 8, 4>(a, st);
}

hipError_t launch_attn_mq(const AttnArgs &a, hipStream_t st)
{
    return a.d == 64 ? launch_mq_d<64>(a, st) : launch_mq_d<128>(a, st);
}

}  // namespace kvev
