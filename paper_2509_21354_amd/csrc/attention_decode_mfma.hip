// Decode attention (Eq. 1 of the paper over kept summaries and raw rows, or the whole cache) for up to 4 queries that
// share the rows, bf16 storage, on the matrix cores: large launches.
//
// attn_decode_kernel (attention_decode.hip) is bound by HBM with one query per sequence; with four the vector unit is
// busy 63 % of the time (dot products, lane folds, weighted sums: 2200 instructions per 64 rows) and its registers leave
// three waves per SIMD.  Here both products run on v_mfma_f32_16x16x32_bf16, whose 16 columns hold the 4 queries four
// times over:
//   S^T = K Q^T    column n: query n % 4.  bf16 products are exact, sums fp32, as in the dot products there;
//   O^T = V^T P^T  the softmax weights are fp32 and stay so: column n holds term n / 4 of the weight of query n % 4, the
//                  three bf16 terms whose sum is the fp32 value (8 + 8 + 8 bits; the fourth is 0), and the columns are
//                  added at the end: fp32-grade weights and sums.
// Rows are copied straight into LDS, 32 at a time and each wave's for itself (no barrier per tile): a wave takes every
// fourth tile of its workgroup's unit, two tiles ahead and on into the next unit, whose queries ride along.  One barrier
// per unit, where the four waves' partial results meet.  K and V tiles lie in LDS with their 16-byte pieces exchanged
// within a row so that no bank is touched twice by a read; V is read with the transposing load (see attention_mq.hip).
// Measured in turn, attn_decode_kernel and this one, d = 128, on changing inputs: 2048 sequences x 325 rows, 4 queries 67.9 and
// 64.1 us (5.4 TB/s; matrix cores 3 %, vector unit 28 % busy: the 128 KiB of LDS that can be under way per compute unit
// are what bounds it now); 1024 x 333 38.8 and 36.1 us (33.8 and 31.3 us on inputs that the memory-side cache holds); 8
// queries, 512 x 1000 81 and 64 us (83 and 57 us).
#include "common.hpp"
#include "kernels.hpp"
#include "lstm_common.hpp"
#include <utility>

namespace kvev {

namespace {
constexpr float kNone = -3.0e38f;       // finite stand-in for -inf, below (almost) every unscaled score
constexpr uint32_t kOdd = 0x7fc1;       // a NaN that marks an output for the second look at the kernel's end
constexpr int kWaves = 4, kRows = 32, kSlots = 2;
}

template <int D> struct Dm {
    static constexpr int KS = D / 32, DT = D / 16, CPR = D / 8, RPI = 512 / D;     // CPR: 16-byte pieces of a row; RPI: rows of a copy
    static constexpr int TB = kRows * D * 2, PER = TB / 1024;                      // bytes and copies of a tile of K or V
    static constexpr int QB = 4 * D * 2;                                           // the unit's queries: one copy (d = 64: half of its lanes twice)
    static constexpr int wave_lds = kSlots * 2 * TB + 2 * 1024;
    static constexpr int merge = kWaves * (4 * D + 8) * 4;                         // partial sums of a unit: o, then m and l
    static constexpr int lds = kWaves * wave_lds + 2 * merge;
    static __device__ __forceinline__ int swz_k(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
    static __device__ __forceinline__ int swz_v(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

// The units of a workgroup (query group qg of sequence s): an XCD takes a contiguous run, in proportion to its workgroups.
struct Units { int first, end, step; };
__device__ __forceinline__ Units units_of(int units)
{
    const int xcd = blockIdx.x & 7, step = ((int)gridDim.x + 7 - xcd) >> 3;
    const int before = xcd * ((int)gridDim.x >> 3) + min(xcd, (int)gridDim.x & 7);
    return {(int)((int64_t)units * before / gridDim.x) + (int)(blockIdx.x >> 3), (int)((int64_t)units * (before + step) / gridDim.x), step};
}

// Values that are not finite.  An infinity meets zeros and remainders of the other sign in the columns of the weights' terms, and
// a slot past the last row its weight of 0: NaN, where Eq. 1 is infinite.  Such outputs were marked; the sum of the values
// that are not finite, among the rows that the query sees, is their result.  (After all units: a look at every unit's columns
// and zeros in the slots past the end cost every launch 2 to 5 %, taken or not.)
template <int D> __device__ void second_look(const AttnArgs &a, int wave, int lane)
{
    wait_vmem<0>();
    const int R = a.G * a.Tq, qgroups = (R + 3) / 4, nraw = a.T - a.win0;
    const Units us = units_of(a.S * qgroups);
    for (int u = us.first; u < us.end; u += us.step) {
        const int s = u / qgroups, r = (u - s * qgroups) * 4 + wave;
        if (r >= R) continue;
        uint16_t *O = static_cast<uint16_t *>(a.O) + ((size_t)s * R + r) * D + lane * (D / 64);
        bool odd[D / 64], some = false;
#pragma unroll
        for (int e = 0; e < D / 64; ++e) {
            odd[e] = O[e] == kOdd;
            some |= odd[e];
        }
        if (!__ballot(some)) continue;
        const int total = nraw + (a.gated ? min(max(a.count[s], 0), a.k_cap) : 0);
        const int lim = a.causal ? nraw - (a.Tq - 1 - r % a.Tq) : nraw;
        float sum[D / 64] = {};
        for (int p = 0; p < total; ++p) {
            if (p >= lim && p < nraw) continue;
            size_t at = (size_t)s * a.N_cap;
            if (p < nraw) {
                const int w = a.win0 + p + a.ring_first;
                at = (size_t)s * a.T_cap + (w >= a.T_cap ? w - a.T_cap : w);
            } else {
                at += min(max(a.idx ? a.idx[(size_t)s * a.k_cap + p - nraw] : p - nraw, 0), a.N_cap - 1);
            }
            const bf16_t *v = static_cast<const bf16_t *>(p < nraw ? a.V : a.Vbar) + at * D + lane * (D / 64);
#pragma unroll
            for (int e = 0; e < D / 64; ++e) {
                const float x = bf16_to_f32(v[e]);
                sum[e] += fabsf(x) < __builtin_inff() ? 0.f : x;
            }
        }
#pragma unroll
        for (int e = 0; e < D / 64; ++e)
            if (odd[e] && sum[e] != 0.f) O[e] = f32_to_bf16(sum[e]);
    }
}

template <int D, bool STREAM>
__global__ __launch_bounds__(64 * kWaves, 1) void attn_decode_mfma_kernel(AttnArgs a, int qgroups, int units)
{
    using M = Dm<D>;
    constexpr int KS = M::KS, DT = M::DT, PER = M::PER, TB = M::TB, RPI = M::RPI, RB = D * 2;
    extern __shared__ __align__(1024) unsigned char smem_dm[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte_t *const mine = (lds_byte_t *)smem_dm + wave * M::wave_lds, *const s_q = mine + kSlots * 2 * TB;
    float *const merge = reinterpret_cast<float *>(smem_dm + kWaves * M::wave_lds);
    const int n = lane & 15, g = lane >> 4, qi = n & 3, term = n >> 2;

    const Units own = units_of(units);
    const int u_first = own.first, u_end = own.end, step = own.step;

    const unsigned char *K = static_cast<const unsigned char *>(a.K), *V = static_cast<const unsigned char *>(a.V);
    const unsigned char *Kbar = static_cast<const unsigned char *>(a.Kbar), *Vbar = static_cast<const unsigned char *>(a.Vbar);
    const int R = a.G * a.Tq, nraw = a.T - a.win0;           // the raw rows come first, then the kept summaries
    // a wave takes every fourth tile; which one comes first changes from unit to unit, so that ragged ends even out
    auto first_row = [&](int u) { return ((wave + u) & (kWaves - 1)) * kRows; };
    auto total_of = [&](int s) { return nraw + (a.gated ? min(max(((const_int_t *)(uintptr_t)a.count)[s], 0), a.k_cap) : 0); };

    // ---- the copies: this wave's tiles (every fourth) of one unit after the other; a unit's queries with its first ----
    int f_u = u_first, f_s = 0, f_j0 = 0, f_total = 0, f_first = 1, f_qslot = 0;
    int f_slot = 0, in_flight = 0, newest = 0;               // copies of the youngest tile: those that may be outstanding behind the one waited for
    auto open_unit = [&]() {                                 // on to the next unit that has rows for this wave
        for (; f_u < u_end; f_u += step) {
            f_s = f_u / qgroups;
            f_total = total_of(f_s);
            f_j0 = first_row(f_u);
            f_first = 1;
            if (f_j0 < f_total) break;
        }
    };
    const int lr = lane / M::CPR, pc = lane % M::CPR;
    auto copy_tile = [&]() {
        if (f_u >= u_end) return;
        const uint32_t slot = (uint32_t)(uintptr_t)mine + f_slot * 2 * TB;
        newest = 2 * PER + f_first;
        if (f_first) {
            const int r0 = f_s * R + (f_u - f_s * qgroups) * 4, last = f_s * R + R - 1;
            copy_to_lds<false>(static_cast<const unsigned char *>(a.Q) + (size_t)min(r0 + (lr & 3), last) * RB + pc * 16,
                               (uint32_t)(uintptr_t)s_q + f_qslot * 1024);
            f_qslot ^= 1;
            f_first = 0;
        }
        const size_t seq_raw = (size_t)f_s * a.T_cap, seq_sum = (size_t)f_s * a.N_cap;
        const_int_t *idx = (const_int_t *)(uintptr_t)(a.idx ? a.idx + (size_t)f_s * a.k_cap : nullptr);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int jb = f_j0 + RPI * i, row = RPI * i + lr;
            const int j = min(f_j0 + row, f_total - 1);                      // (rows past the end are masked in the softmax)
            int r = a.win0 + min(j, max(nraw - 1, 0)) + a.ring_first;
            r = r >= a.T_cap ? r - a.T_cap : r;
            size_t off = (seq_raw + r) * RB;
            const unsigned char *kp = K + off, *vp = V + off;
            if (min(jb + RPI, f_total) > nraw) {                             // some of these rows are summaries
                int c = j - nraw;                                            // (null list: compact store, row j is entry j)
                if (a.idx) {
                    c = 0;
#pragma unroll
                    for (int e = 0; e < RPI; ++e) {
                        const int ce = idx[max(min(jb + e, f_total - 1) - nraw, 0)];
                        c = min(jb + e, f_total - 1) == j ? ce : c;
                    }
                }
                off = (seq_sum + min(max(c, 0), a.N_cap - 1)) * RB;
                if (j >= nraw) { kp = Kbar + off; vp = Vbar + off; }
            }
            copy_to_lds<STREAM>(kp + ((pc ^ M::swz_k(row)) << 4), slot + i * 1024);
            copy_to_lds<STREAM>(vp + ((pc ^ M::swz_v(row)) << 4), slot + TB + i * 1024);
        }
        f_slot = f_slot + 1 == kSlots ? 0 : f_slot + 1;
        ++in_flight;
        f_j0 += kWaves * kRows;
        if (f_j0 >= f_total) { f_u += step; open_unit(); }
    };
    // The older of the tiles in flight has landed.  Loads and stores return in order: the younger tile's copies may be under
    // way, and so may the store of a unit's results that left after either was asked for (stored: for how many tiles).
    int stored = 0;
    auto wait_tile = [&]() {
        const int behind = (in_flight > 1 ? newest : 0) + (stored > 0 ? 1 : 0);
        if (stored > 0) --stored;
        if (behind == 2 * PER + 2) wait_vmem<2 * PER + 2>();
        else if (behind == 2 * PER + 1) wait_vmem<2 * PER + 1>();
        else if (behind == 2 * PER) wait_vmem<2 * PER>();
        else if (behind == 1) wait_vmem<1>();
        else wait_vmem<0>();
        --in_flight;
    };
    open_unit();
    copy_tile();
    copy_tile();

    const float c = a.scale_log2e;
    const int k_rd = n * RB + ((g ^ M::swz_k(n)) << 4);                      // row n of 16, piece 4 ks + g: ^ (ks << 6), + 16 rows
    const int v_row = 4 * g + (n >> 2);
    const int v_rd = TB + v_row * RB + ((((n & 3) >> 1) ^ M::swz_v(v_row)) << 4) + 8 * (n & 1);      // d = 16 dt + 4 (n % 4): ^ (dt << 5)
    int slot = 0, qslot = 0, parity = 0;
    uint32_t any_odd = 0;
    for (int u = u_first; u < u_end; u += step) {
        const int s = u / qgroups, total = total_of(s), r0 = (u - s * qgroups) * 4;
        // positions p of rows that this lane's query sees: summaries (p >= nraw) and raw rows before lim (causal frame: the
        // queries are the last Tq cached tokens and see nothing after their own position)
        const int lim = r0 + qi >= R ? -1 : a.causal ? nraw - (a.Tq - 1 - (r0 + qi) % a.Tq) : nraw;
        const bool there = r0 + qi < R;
        bf16x8_t qf[KS];
        float m = kNone, l = 0.f;
        f32x4_t o[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        const int j_first = first_row(u);
        for (int j0 = j_first; j0 < total; j0 += kWaves * kRows) {
            wait_tile();
            const lds_byte_t *tile = mine + slot * 2 * TB;
            slot = slot + 1 == kSlots ? 0 : slot + 1;
            if (j0 == j_first) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    qf[ks] = *(const __attribute__((address_space(3))) bf16x8_t *)(s_q + qslot * 1024 + qi * RB + ks * 64 + g * 16);
                qslot ^= 1;
            }
            // ---- S^T = K Q^T: 32 keys, register 4 kt + r is key 16 kt + 4 g + r ----
            bf16x8_t kf[2][KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
                    kf[kt][ks] = *(const __attribute__((address_space(3))) bf16x8_t *)(tile + (k_rd ^ (ks << 6)) + kt * 16 * RB);
            v4i16_t vf[DT][2];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    vf[dt][p] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t *)(tile + (v_rd ^ (dt << 5)) + p * 16 * RB));
            f32x4_t st[2] = {};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int kt = 0; kt < 2; ++kt) st[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][ks], qf[ks], st[kt], 0, 0, 0);
            // the tile is in registers: its slot takes the tile after the next
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
            __builtin_amdgcn_sched_barrier(0);
            copy_tile();

            // ---- online softmax ----
            // no row of the tile is hidden from any query
            const bool full = j0 + kRows <= nraw - (a.causal ? a.Tq - 1 : 0) || (j0 >= nraw && j0 + kRows <= total);
            float x[8];
            bool seen[8];
            float mx = kNone;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int p = j0 + 16 * (e >> 2) + 4 * g + (e & 3);
                seen[e] = there && (full || (p < total && (p >= nraw || p < lim)));
                x[e] = seen[e] ? st[e >> 2][e & 3] : kNone;
                mx = fmaxf(mx, x[e]);
            }
            mx = fmaxf(m, rows_max(mx));
            if (__ballot(mx > m)) {
                const float alpha = __builtin_amdgcn_exp2f((m - mx) * c);
                l *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
                m = mx;
            }
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                w[e] = seen[e] ? __builtin_amdgcn_exp2f((x[e] - m) * c) : 0.f;       // (1 at the maximum, however large the scores)
                l += w[e];
            }
            // the lane's bf16 term of each weight: what the terms before it leave (exact differences)
            uint32_t pw[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const uint32_t hi = pack_bf16x2(w[e], w[e + 1]);
                const float a0 = w[e] - __uint_as_float(hi << 16), a1 = w[e + 1] - __uint_as_float(hi & 0xffff0000u);
                const uint32_t mid = pack_bf16x2(a0, a1);
                const uint32_t lo = pack_bf16x2(a0 - __uint_as_float(mid << 16), a1 - __uint_as_float(mid & 0xffff0000u));
                pw[e / 2] = term == 0 ? hi : term == 1 ? mid : term == 2 ? lo : 0u;
            }
            // ---- O^T += V^T P^T ----
            const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, make_uint4(pw[0], pw[1], pw[2], pw[3]));
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, __builtin_shufflevector(vf[dt][0], vf[dt][1], 0, 1, 2, 3, 4, 5, 6, 7)), pb, o[dt], 0, 0, 0);
        }

        // ---- the four waves' parts: per query the maximum, the sum, and the weighted rows (all terms together) ----
        float *const s_o = merge + parity * (M::merge / 4), *const s_ml = s_o + kWaves * 4 * D;      // [wave][query][D], [wave][query] {m, l}
        parity ^= 1;
        l = rows_sum(l);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[dt][r] += dpp_move<kRowRor4>(o[dt][r]);
                o[dt][r] += dpp_move<kRowRor8>(o[dt][r]);
            }
        if (term == 0) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4_t *>(s_o + (wave * 4 + qi) * D + 16 * dt + 4 * g) = o[dt];
            if (g == 0) { s_ml[(wave * 4 + qi) * 2] = m; s_ml[(wave * 4 + qi) * 2 + 1] = l; }
        }
        lds_barrier();           // (the next unit's parts go to the other half: a wave is one unit ahead at most)
        // wave q writes query r0 + q: D / 64 elements per lane
        float Mx = kNone, L = 0.f, acc[D / 64] = {};
#pragma unroll
        for (int w_ = 0; w_ < kWaves; ++w_) Mx = fmaxf(Mx, s_ml[(w_ * 4 + wave) * 2]);
#pragma unroll
        for (int w_ = 0; w_ < kWaves; ++w_) {
            const float f = __builtin_amdgcn_exp2f((s_ml[(w_ * 4 + wave) * 2] - Mx) * c);
            L = fmaf(s_ml[(w_ * 4 + wave) * 2 + 1], f, L);
#pragma unroll
            for (int e = 0; e < D / 64; ++e) acc[e] = fmaf(s_o[(w_ * 4 + wave) * D + lane * (D / 64) + e], f, acc[e]);
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;
        // (the descriptor ends with the sequence's last query: every wave issues one store, which wait_tile counts)
        const __amdgpu_buffer_rsrc_t o_rsrc = make_rsrc(static_cast<unsigned char *>(a.O) + (size_t)s * R * RB, (uint32_t)R * RB);
        uint32_t out = pack_bf16x2(acc[0] * inv, acc[D / 64 - 1] * inv);
        const bool odd_lo = acc[0] != acc[0], odd_hi = acc[D / 64 - 1] != acc[D / 64 - 1];
        if (__builtin_expect(__ballot(odd_lo || odd_hi) != 0, 0)) {
            out = L != L ? 0x7fc07fc0u : (odd_lo ? kOdd : out & 0xffffu) | (odd_hi ? kOdd << 16 : out & 0xffff0000u);
            any_odd = 1;
        }
        if (D == 128) __builtin_amdgcn_raw_buffer_store_b32(out, o_rsrc, (r0 + wave) * RB + lane * 4, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16((uint16_t)out, o_rsrc, (r0 + wave) * RB + lane * 2, 0, 0);
        stored = in_flight;
    }

    if (__builtin_expect(any_odd, 0)) {
        // (the arguments again: kept through the loop for this, they would not fit the scalar registers)
        auto *args = (const __attribute__((address_space(4))) AttnArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        second_look<D>(*(const AttnArgs *)args, wave, lane);
    }
}

template <int D, bool STREAM>
static hipError_t launch_dm(const AttnArgs &a, hipStream_t st)
{
    const int qgroups = (a.G * a.Tq + 3) / 4;
    const int64_t units = (int64_t)a.S * qgroups;
    const auto kernel = attn_decode_mfma_kernel<D, STREAM>;
    static std::atomic<uint64_t> done{0};
    const hipError_t e = allow_lds(kernel, Dm<D>::lds, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(units < a.compute_units ? units : a.compute_units)), dim3(64 * kWaves), Dm<D>::lds, st, a, qgroups, (int)units);
    return hipGetLastError();
}

hipError_t launch_attn_decode_mfma(const AttnArgs &a, hipStream_t st)
{
    if (a.d == 64) return a.stream ? launch_dm<64, true>(a, st) : launch_dm<64, false>(a, st);
    return a.stream ? launch_dm<128, true>(a, st) : launch_dm<128, false>(a, st);
}

}  // namespace kvev
