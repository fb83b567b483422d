// Recurrent gate, Eq. 3 of the paper, bf16 storage, d_g = 64 and 128: the sequential half.
//
// What bounds it is the chain of one step: read h, multiply, the cell, publish h, barrier.  W_hh (32 or 128 KiB as fp16)
// fits the registers of one workgroup with a wave per 16 units, so a group of sequences never leaves its compute unit and a
// step costs one barrier:
//   * 8 sequences per workgroup.  The 16 columns of a matrix instruction hold the two fp16 terms of h for the 8 sequences
//     side by side (column n: sequence n mod 8, hi for n < 8, lo for n >= 8), so one instruction per weight fragment gives
//     both products; the two lanes that hold the same sums after the fold share the four units between them.  Per sequence
//     the matrix work and the nonlinearities are those of 16 sequences with two instructions per fragment, and a launch of
//     few sequences has half of either on its chain;
//   * the input projections are requested kDepth steps before they are used, into registers;
//   * the utility logit of a step is summed in the next one, beside its products: each wave takes the shares of one
//     (d_g = 128) or two (d_g = 64) sequences from LDS, keeps the logits of 64 or 32 steps in its lanes and stores them in
//     one run; so a step's barrier waits for no store.
// Two buffers of h and of the shares by step parity: what a step reads, the next one leaves alone.
// Measured (whole gate call, weights prepared) against 16 sequences per workgroup with the weights in LDS and the
// projections asked for in the step that uses them (1.7 ... 2 us a step): d_g = 128, 7 layers x 8 sequences x 100 steps
// 170 -> 93 us, 464 sequences x 241 steps 448 -> 268 us; d_g = 64, 192 x 11 23.6 -> 15.1 us.  8192 x 128 983 -> 912 us (d_g = 64)
// and 1342 -> 1213 us (128), bound by the projections' way through memory.
// Registers are bounded to 128, so that two workgroups of d_g = 128 or four of d_g = 64 run beside each other per unit.
#include "common.hpp"
#include "kernels.hpp"
#include "lstm_common.hpp"

namespace kvev {

template <int DG> struct NarrowGeo {
    static constexpr int KS = DG / 32, NW = DG / 16, THREADS = NW * 64, HP = DG + 8;
    static constexpr int DEPTH = DG == 64 ? 4 : 2;        // steps that the projections are ahead (2 or 4: the end of the step loop)
    static constexpr int RUN = NW * 8;                    // shares of a sequence's logit, and steps kept per store
    static constexpr int UPITCH = RUN + 8;                // (8 sequences land in different banks)
    static_assert(NW * Geo<DG>::KS * 4 * 64 == Geo<DG>::NW * Geo<DG>::ITEMS * 4 * 64, "the packed order walks 16 units at a time");
};

template <int DG>
__global__ __launch_bounds__(NarrowGeo<DG>::THREADS, 4) void lstm_rec_narrow_kernel(LstmArgs a, int t0, int nb)
{
    using N = NarrowGeo<DG>;
    constexpr int KS = N::KS, NW = N::NW, HP = N::HP, DEPTH = N::DEPTH, RUN = N::RUN;
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    __shared__ __align__(16) f16_t s_h[2][16 * HP];
    __shared__ float s_up[2][8 * N::UPITCH];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g4 = lane >> 4, sn = n & 7, half = n >> 3;
    const int gpl = (a.BH + 7) / 8;
    const int gid = xcd_order(blockIdx.x, gridDim.x);
    const int l = gid / gpl, grp = gid % gpl;
    const bool live = grp * 8 + sn < a.BH;
    const size_t s = (size_t)l * a.BH + min(grp * 8 + sn, a.BH - 1);
    const int unit0 = wave * 16 + 4 * g4 + 2 * half;      // this lane's two cells: units unit0, unit0 + 1 of sequence s

    const bf16_t *w_s = static_cast<const bf16_t *>(a.w_s) + (size_t)l * DG;
    auto scalar = [](float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); };
    const float b_s = scalar(bf16_to_f32(static_cast<const bf16_t *>(a.b_s)[l]));
    const float inv_scale = scalar(ldexpf(1.f, -whh_scale_exp(whh_layer_max(a.whh_max_bits, l))));

    const uint32_t lane16 = lane * 16;
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(a.whh_packed + ((size_t)l * NW + wave) * KS * 4 * 64, KS * 4096);
    f16x8_t w[KS][4];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int q = 0; q < 4; ++q) w[ks][q] = buffer_load16<f16x8_t>(w_rsrc, lane16 + q * 1024, ks * 4096);

    // projections: written in fragments of 16 sequences, this lane reads its two units of its sequence (past the block: the last step again)
    const int gid16 = l * ((a.BH + 15) / 16) + grp / 2;
    const unsigned char *xbase = reinterpret_cast<const unsigned char *>(a.xproj + xp_block<DG>(gid16, a.tb, 0, wave / 2, wave % 2, 0) * 256);
    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(xbase, (uint32_t)nb * NW * 4096 - (uint32_t)wave * 4096);
    const uint32_t xoff = (uint32_t)((g4 * 16 + (grp & 1) * 8 + sn) * 16 + half * 8);
    float xin[DEPTH][4][2];
    auto fetch_x = [&](int tt, float (&x)[4][2]) __attribute__((always_inline)) {
        const uint32_t at = (uint32_t)min(tt, nb - 1) * NW * 4096;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(x_rsrc, (int)xoff, (int)(at + q * 1024), 0);
            x[q][0] = __uint_as_float(v[0]);
            x[q][1] = __uint_as_float(v[1]);
        }
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) fetch_x(i, xin[i]);

    float c_reg[2], h_reg[2], ws_reg[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {   // (chunk 0 starts the recurrence from a zero state, whatever the buffers hold)
        c_reg[r] = live && t0 > 0 ? a.c[s * DG + unit0 + r] : 0.f;
        h_reg[r] = live && t0 > 0 ? a.h[s * DG + unit0 + r] : 0.f;
        ws_reg[r] = bf16_to_f32(w_s[unit0 + r]);
    }
    auto publish_h = [&](int buf) __attribute__((always_inline)) {      // two fp16 terms (hi + lo = h to 22 bits)
        const f16x2_t hi = {(f16_t)h_reg[0], (f16_t)h_reg[1]};
        const f16x2_t lo = {(f16_t)(h_reg[0] - (float)hi[0]), (f16_t)(h_reg[1] - (float)hi[1])};
        *reinterpret_cast<f16x2_t *>(&s_h[buf][sn * HP + unit0]) = hi;
        *reinterpret_cast<f16x2_t *>(&s_h[buf][(sn + 8) * HP + unit0]) = lo;
    };

    // the logits: lane `pos` of its part of the wave keeps step base + pos of sequence us
    const int us = wave * (64 / RUN) + lane / RUN, pos = lane % RUN;
    float logits = 0.f;
    auto share = [&](int buf) __attribute__((always_inline)) { return s_up[buf][us * N::UPITCH + pos]; };
    auto logit_of = [&](float u, int step) __attribute__((always_inline)) {
        u += dpp_move<kQuadXor1>(u);
        u += dpp_move<kQuadXor2>(u);
        u += dpp_move<kRowRor8>(u);          // (before the turn by 4: so all lanes add in the same order, and whichever
        u += dpp_move<kRowRor4>(u);          // keeps the step has the same bits)
        if constexpr (RUN == 64) {
            u = rows_sum(u);
        } else {
            float x = u, y = u;
            swap16(x, y);
            u = x + y;
        }
        logits = pos == step % RUN ? u + b_s : logits;
    };
    auto store_logits = [&](int base, int last) __attribute__((always_inline)) {
        int useq = grp * 8 + us;
        asm volatile("" : "+v"(useq));       // (the address is made here, not held in registers through the steps)
        if (useq < a.BH && base + pos <= last) {
            const size_t at = ((size_t)l * a.BH + useq) * a.N_cap + t0 + base + pos;
            a.util[at] = logits;
            a.gate[at] = sigmoid_hw(logits);
        }
    };

    auto store_state = [&]() __attribute__((always_inline)) {
        int seq = grp * 8 + sn;
        asm volatile("" : "+v"(seq));
        if (seq < a.BH) {
            const size_t at = ((size_t)l * a.BH + seq) * DG + unit0;
            *reinterpret_cast<float2 *>(a.h + at) = make_float2(h_reg[0], h_reg[1]);
            *reinterpret_cast<float2 *>(a.c + at) = make_float2(c_reg[0], c_reg[1]);
        }
    };

    auto step = [&](int tt, auto slot) __attribute__((always_inline)) {
        constexpr int i = decltype(slot)::value, cur = i & 1, nxt = cur ^ 1;
        f16x8_t hb[2];
        auto read_h = [&](int ks) __attribute__((always_inline)) { hb[ks & 1] = *reinterpret_cast<const f16x8_t *>(&s_h[cur][n * HP + g4 * 8 + ks * 32]); };
        read_h(0);
        const float up = share(nxt);
        f32x4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) read_h(ks + 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[ks][q], hb[ks & 1], acc[q], 0, 0, 0);
            if (ks == KS - 2) logit_of(up, tt - 1);              // (step -1 is kept by no lane)
            if (KS > 2) __builtin_amdgcn_sched_barrier(0);       // (two operands of h in registers, not all of them)
        }
        if (tt > 0 && tt % RUN == 0) store_logits(tt - RUN, tt - 1);
        // own two rows from this column and from the one that holds the other term
        float pre[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float sum = (half ? acc[q][2 + r] : acc[q][r]) + dpp_move<kRowRor8>(half ? acc[q][r] : acc[q][2 + r]);
                pre[q][r] = fmaf(sum, inv_scale, xin[i][q][r]);
            }
        float upart = 0.f;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float ig = sigmoid_hw(pre[0][r]), fg = sigmoid_hw(pre[1][r]), gg = tanh_hw(pre[2][r]), og = sigmoid_hw(pre[3][r]);
            c_reg[r] = fmaf(fg, c_reg[r], ig * gg);
            float hn = og * tanh_hw(c_reg[r]);
            asm volatile("" : "+v"(hn));     // opaque to the optimiser: hn is the rounded product from here on
            h_reg[r] = hn;
            upart = fmaf(ws_reg[r], hn, upart);
        }
        publish_h(nxt);
        if (tt == nb - 1) store_state();
        s_up[cur][sn * N::UPITCH + wave * 8 + g4 * 2 + half] = upart;
        fetch_x(tt + DEPTH, xin[i]);
        lds_barrier();
    };

    publish_h(0);
    lds_barrier();
    using std::integral_constant;
    int tt = 0;
#pragma nounroll
    for (; tt + DEPTH <= nb; tt += DEPTH)    // (no way out but the end: the counted waits for the projections rely on it)
        static_for<DEPTH>([&](auto ic) __attribute__((always_inline)) { step(tt + decltype(ic)::value, ic); });
    if (tt < nb) {
        step(tt++, integral_constant<int, 0>{});
        if constexpr (DEPTH == 4) {
            if (tt < nb) step(tt++, integral_constant<int, 1>{});
            if (tt < nb) step(tt, integral_constant<int, 2>{});
        }
    }
    logit_of(share((nb - 1) & 1), nb - 1);
    store_logits((nb - 1) / RUN * RUN, nb - 1);
}

hipError_t launch_lstm_narrow(const LstmArgs &a, int t0, int nb, hipStream_t st)
{
    const dim3 grid((unsigned)(a.L * ((a.BH + 7) / 8)));
    if (a.d_g == 64) hipLaunchKernelGGL((lstm_rec_narrow_kernel<64>), grid, dim3(NarrowGeo<64>::THREADS), 0, st, a, t0, nb);
    else hipLaunchKernelGGL((lstm_rec_narrow_kernel<128>), grid, dim3(NarrowGeo<128>::THREADS), 0, st, a, t0, nb);
    return hipGetLastError();
}

}  // namespace kvev
