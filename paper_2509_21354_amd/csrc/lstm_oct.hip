// Recurrent gate, Eq. 3 of the paper, bf16 storage, d_g = 256 and 512: the sequential half for launches of few sequences,
// 4 or 8 sequences on four or 8 on two compute units (256), 4, 8 or 16 on eight (512).
//
// What bounds such a launch is the chain of one step, and the chip is mostly idle.  As in lstm_rec_pair_kernel
// (lstm_mfma.hip) the workgroups of a group share the hidden units, keep their rows of W_hh in registers and exchange
// the new h every step.  What is different, all of it to shorten the step:
//   * 8 sequences per group instead of 16.  The 16 columns of a matrix instruction hold the two fp16 terms of h for the
//     8 sequences side by side (column n: sequence n mod 8, hi for n < 8, lo for n >= 8), so one instruction per weight
//     fragment gives both products; they are added across the columns afterwards, and the two lanes that then hold the
//     same sums share the four units between them.  Half the matrix work, half the nonlinearities and half the exchange
//     per group, on compute units that were idle;
//   * P = 4 workgroups of 4 waves where the launch leaves room for them, else 2 of 8 (d_g = 512: 8 of 4): a wave owns 16
//     units either way (smaller launches yet take groups of 4 sequences: lstm_rec_few_kernel, below);
//   * 8 bytes per lane carry 4 units of one column: |h| <= 1 leaves bit 14 of an fp16 term free (of hi and of lo), and the
//     first term of every aligned 8-byte word, which is written and read as one, carries a flag there that flips from one
//     use of a slot to the next.  Two slots by step parity, cleared before the launch: a slot is rewritten two steps
//     later, by a workgroup that has seen its partners' h of the step between, whose waves had all read this one: they
//     publish behind a barrier that follows the reads.  Stores write through and loads look past the caches of one XCD
//     (device scope): the members sit on different ones.  A reader has itself taken the use before from the same
//     addresses, and such loads do not go back at a location, so it meets the use that it waits for or the one before,
//     and one bit tells them apart (the first use is told from zeros);
//   * the input projections of the next step are requested in this one, into registers of their own.
// A step: products over the own units | take the partners' h, stage in LDS | barrier | products over the partners' units |
// cell, publish, own h to LDS | barrier.  Bounded waits, status word and the layout of weights and projections: as the
// paired kernel.
// Measured (the whole gate call, weights prepared): 32 sequences x 128 steps 304 us on pairs per 16 sequences, 233 us in groups of 8 (P =
// 4; 175 to 205 in groups of 4; about 0.95 us of a step are its own work, the rest is the exchange), 248 us with 16 bytes per
// lane, a stamp of the step beside every two units, in the flag's place; 512 x 64 183, 145 and 156 us; 1024 x 64 (P = 2) 245, 218
// and 219 us.
// Members on one XCD that exchange by plain stores through its L2 took 185 us at the first shape, but publications of that
// kind were lost under cache pressure (seen in lstm_quad.hip; cause not shown), so all stores write through.
// d_g = 512: W_hh is 2 MiB as fp16, and what bounds the forms on two or four compute units is its stream out of L2 in every
// step (8 to 14 us).  On eight a wave's rows are 64 KiB, 256 registers per lane: they fit beside the rest because a workgroup of
// 4 waves has 512 registers per lane, and matrix instructions take them from the accumulation half.  Where 8 * groups of 8 are
// more than the compute units, a workgroup takes two groups in turn (SUB = 2): the h of one travels while the other is
// computed, so nothing is waited for, and each needs one barrier instead of two.  Measured (whole gate call, weights
// prepared): 32 sequences x 128 steps 1049 -> 325 us (291 in groups of 4), 144 (16 a layer) x 130 1364 -> 414, 256 x 64 564 -> 208,
// 512 x 64 570 -> 361, 512 (16 a layer) x 64 910 -> 392, 32 x 8 85 -> 45 us.  At d_g = 256 two groups in turn on two workgroups are slower
// than lstm_rec_pair_kernel (2048 x 128 769 against 690 us: vector work, not the exchange, bounds it there).
#include "common.hpp"
#include "kernels.hpp"
#include "lstm_common.hpp"
#include <utility>

namespace kvev {

namespace {
// exchange slots of 8 sequences: [parity][member][column 16][own units], an fp16 term per unit
template <int DG> constexpr uint32_t slots8() { return 2 * DG * 16 * 2; }
static_assert(2 * slots8<256>() <= kLstmPairExchBytes256, "two groups of 8 fit the scratch planned for one of 16");
static_assert(slots8<512>() == kLstmOctExchBytes512, "the scratch planner's figure");
}

// P workgroups per group, each with DG / P hidden units: a wave per 16 of them; SUB times 8 sequences in turn
template <int DG, int P, int SUB>
__global__ __launch_bounds__(4 * DG / P) void lstm_rec_oct_kernel(LstmArgs a, int t0, int nb)
{
    using G = Geo<DG>;
    constexpr int kKS = DG / 32, kNW = DG / 16 / P, kKH = kKS / P, kKP = kKS - kKH;      // k-steps; waves; k-steps over own units, over the partners'
    constexpr int kOwn = DG / P, kOP = kOwn + 8, kPP = DG - kOwn + 8;       // own units; row pitches in LDS
    constexpr uint32_t kSlot = 16 * kOwn * sizeof(f16_t), kGroupSlots = slots8<DG>();     // one member's h of one step: [column 16][own units]
    constexpr int kLR = kOwn / 4, kRows = 64 / kLR;                  // receiving: lanes per row, rows per wave
    constexpr int kPin = DG == 512 ? 15 : 0;                         // k-steps whose weights are kept in accumulation registers
    __shared__ __align__(16) f16_t s_h[SUB][16 * kOP];       // own units of h, row = column of the operand
    __shared__ __align__(16) f16_t s_p[SUB][16 * kPP];       // the partners' units
    __shared__ float s_up[SUB][2][kNW][8], s_up2[SUB][16];             // shares of the utility logit: own units (by step parity), partners' by column
    __shared__ int s_fail;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g4 = lane >> 4, sn = n & 7, hn2 = n >> 3;
    // The members of a group are neighbours in launch order: where one runs, the others run or are next.
    const int gpl = (a.BH + 8 * SUB - 1) / (8 * SUB);
    const int member = blockIdx.x % P, gid = blockIdx.x / P;
    const int l = gid / gpl, grp = gid % gpl;
    bool live[SUB];
    size_t s[SUB];
#pragma unroll
    for (int g = 0; g < SUB; ++g) {
        live[g] = (grp * SUB + g) * 8 + sn < a.BH;
        s[g] = (size_t)l * a.BH + min((grp * SUB + g) * 8 + sn, a.BH - 1);
    }
    // the partners follow cyclically: k-step i < kKP of theirs belongs to member + 1 + i / kKH (mod P)
    auto par_of = [&](int i) __attribute__((always_inline)) { return (member + 1 + i / kKH) % P; };
    const int tile = member * kNW + wave;                    // unit tile (16 units) of this wave
    const int unit0 = tile * 16 + 4 * g4 + 2 * hn2;          // this lane's two cells: units unit0, unit0 + 1 of sequence s[g]

    const bf16_t *w_s = static_cast<const bf16_t *>(a.w_s) + (size_t)l * DG;
    const float b_s = bf16_to_f32(static_cast<const bf16_t *>(a.b_s)[l]);
    const float inv_scale = ldexpf(1.f, -whh_scale_exp(whh_layer_max(a.whh_max_bits, l)));
    if (tid == 0) s_fail = 0;

    // ---- all weights of the wave: kKS k-steps x 4 gates, own units first ----
    const uint32_t lane16 = lane * 16;
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(
        reinterpret_cast<const unsigned char *>(a.whh_packed + (((size_t)l * G::NW + tile / G::UT) * G::ITEMS + (tile % G::UT) * kKS) * 4 * 64),
        kKS * 4096);
    f16x8_t w[kKS][4];
#pragma unroll
    for (int i = 0; i < kKS; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[i][q] = buffer_load16<f16x8_t>(w_rsrc, lane16 + q * 1024, (uint32_t)((i < kKH ? member * kKH + i : par_of(i - kKH) * kKH + (i - kKH) % kKH) * 4096));
            if (i < kPin) asm volatile("" : "+a"(w[i][q]));      // (left to itself the compiler moves them to vector registers before every use)
        }

    // ---- the input projections: written in fragments of 16 sequences, this lane reads its two units of its sequence ----
    const int gpl16 = (a.BH + 15) / 16;
    __amdgpu_buffer_rsrc_t x_rsrc[(SUB + 1) / 2];
    uint32_t xoff[SUB];
#pragma unroll
    for (int g = 0; g < SUB; ++g) {
        const int g8 = grp * SUB + g;
        if (g % 2 == 0)
            x_rsrc[g / 2] = make_rsrc(reinterpret_cast<const f32x4_t *>(a.xproj) +
                                          xp_block<DG>(l * gpl16 + min(g8 / 2, gpl16 - 1), a.tb, 0, tile / G::UT, tile % G::UT, 0) * 64,
                                      (uint32_t)nb * G::NW * G::UT * 4096 - (uint32_t)tile * 4096);
        xoff[g] = (uint32_t)((g4 * 16 + (g8 & 1) * 8 + sn) * 16 + hn2 * 8);
    }
    // (two sets by step parity: a set in flight across the step boundary is not copied, which would wait for it)
    float xin[SUB][2][4][2];
    auto fetch_x = [&](int g, int tt, float (&x)[4][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(x_rsrc[g / 2], (int)(xoff[g] + q * 1024), (int)((uint32_t)tt * G::NW * G::UT * 4096), 2);
            x[q][0] = __uint_as_float(v[0]);
            x[q][1] = __uint_as_float(v[1]);
        }
    };
#pragma unroll
    for (int g = 0; g < SUB; ++g) fetch_x(g, 0, xin[g][0]);

    const __amdgpu_buffer_rsrc_t e_rsrc = make_rsrc(a.exch + (size_t)gid * SUB * kGroupSlots, SUB * kGroupSlots);
    // a look at the partners' slots of parity `par`: this wave takes rows wave * kRows .. of each, 8 bytes per lane
    const int rrow = wave * kRows + lane / kLR, rcol = lane % kLR;       // column of the operand; 4 units from 4 rcol on
    auto ask = [&](int g, int par, u32x2_t (&v)[P - 1]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < P - 1; ++p)
            v[p] = __builtin_amdgcn_raw_buffer_load_b64(e_rsrc, lane * 8, (int)(g * kGroupSlots + (par * P + (member + 1 + p) % P) * kSlot + wave * 512), 16);
    };

    // h of step t0 - 1, split into two fp16 terms: (hi, lo) pairs of two neighbouring units
    auto split2 = [](float h0, float h1, uint32_t &hi, uint32_t &lo) __attribute__((always_inline)) {
        typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
        const f16x2_t h = {(f16_t)h0, (f16_t)h1};
        const f16x2_t r = {(f16_t)(h0 - (float)h[0]), (f16_t)(h1 - (float)h[1])};
        hi = __builtin_bit_cast(uint32_t, h);
        lo = __builtin_bit_cast(uint32_t, r);
    };
    // the lanes of a sequence trade pairs: lane n < 8 leaves with hi of units 4 g4 .. + 3, lane n + 8 with lo of them
    auto gather = [&](uint32_t hi, uint32_t lo) __attribute__((always_inline)) {
        const uint32_t other = __float_as_uint(dpp_move<kRowRor8>(__uint_as_float(hn2 ? hi : lo)));
        return hn2 ? u32x2_t{other, lo} : u32x2_t{hi, other};
    };
    f16_t *const h_wr = s_h[0] + (size_t)n * kOP + wave * 16 + 4 * g4;          // + g * 16 * kOP
    const f16_t *const h_rd = s_h[0] + (size_t)n * kOP + g4 * 8, *const p_rd = s_p[0] + (size_t)n * kPP + g4 * 8;     // + g * 16 * pitch + j * 32
    f16_t *const p_wr = s_p[0] + (size_t)rrow * kPP + 4 * rcol;         // + g * 16 * kPP + p * kOwn

    float c_reg[SUB][2], ws_own[2];
#pragma unroll
    for (int gp = 0; gp < SUB * P; ++gp) {       // own units, then the partners'
        const int g = gp / P, p = gp % P;
        float hv[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int u = (member + p) % P * kOwn + unit0 - member * kOwn + r;
            // (chunk 0 starts the recurrence from a zero state, whatever the buffers hold)
            hv[r] = live[g] && t0 > 0 ? a.h[s[g] * DG + u] : 0.f;
            if (p == 0) {
                c_reg[g][r] = live[g] && t0 > 0 ? a.c[s[g] * DG + u] : 0.f;
                ws_own[r] = bf16_to_f32(w_s[u]);
            }
        }
        uint32_t hi, lo;
        split2(hv[0], hv[1], hi, lo);
        f16_t *dst = p == 0 ? h_wr + g * 16 * kOP : s_p[g] + (size_t)n * kPP + (p - 1) * kOwn + wave * 16 + 4 * g4;
        *reinterpret_cast<u32x2_t *>(dst) = gather(hi, lo);
    }
    float ws_par[P - 1][4];          // of the units that this lane receives
#pragma unroll
    for (int p = 0; p < P - 1; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) ws_par[p][e] = bf16_to_f32(w_s[(member + 1 + p) % P * kOwn + 4 * rcol + e]);
    __syncthreads();

    // the logit of a step from the shares of all members, by wave 0 of member 0 where it would otherwise wait
    auto write_util = [&](int g, int step) __attribute__((always_inline)) {
        float u = s_up2[g][sn] + s_up2[g][sn + 8];       // products with hi and with lo
#pragma unroll
        for (int w_ = 0; w_ < kNW; ++w_) u += s_up[g][step & 1][w_][sn];
        u += b_s;
        if (live[g] && lane < 8) {
            a.util[s[g] * a.N_cap + t0 + step] = u;
            a.gate[s[g] * a.N_cap + t0 + step] = sigmoid_hw(u);
        }
    };
    // the flag of the publication of step tt (within the launch)
    constexpr uint32_t kFlag = 0x4000u;
    auto flag_of = [](int tt) { return (tt >> 1) & 1 ? 0u : kFlag; };
    // The partners' h of step tt - 1 into LDS, from a look asked for earlier; more looks follow if it is not there yet.
    // Member 0 also sums up this wave's rows for the utility.
    auto receive = [&](int g, int tt, u32x2_t (&v)[P - 1]) __attribute__((always_inline)) {
        typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
        const int par = (tt - 1) & 1;
        const uint32_t flag = flag_of(tt - 1);
        auto complete = [&]() __attribute__((always_inline)) {
            uint32_t off = 0;
#pragma unroll
            for (int p = 0; p < P - 1; ++p) off |= v[p][0] ^ flag;
            return __all((off & kFlag) == 0) != 0;
        };
        bool got = complete();
        for (int spin = 0; !got && spin < a.pair_spin_limit; ++spin) {
            asm volatile("" ::: "memory");
            if ((spin & 255) == 255 && s_fail) break;
            ask(g, par, v);
            got = complete();
        }
        if (!got) s_fail = 1;
        float u = 0.f;
#pragma unroll
        for (int p = 0; p < P - 1; ++p) {
            uint32_t x = v[p][0] & ~kFlag;
            // a NaN without its flag bit reads as a magnitude above 1 (exponent 15, a mantissa), which no |h| <= 1 has
            if ((x & 0x7fffu) > 0x3c00u) x |= kFlag;
            const u32x2_t o = {x, v[p][1]};
            *reinterpret_cast<u32x2_t *>(p_wr + g * 16 * kPP + p * kOwn) = o;
            const f16x4_t h4 = __builtin_bit_cast(f16x4_t, o);
#pragma unroll
            for (int e = 0; e < 4; ++e) u = fmaf(ws_par[p][e], (float)h4[e], u);
        }
        return u;
    };
    // ... whose sums over a row's lanes are not waited for by the products
    auto share = [&](int g, float u) __attribute__((always_inline)) {
        u += dpp_move<kQuadXor1>(u);
        u += dpp_move<kQuadXor2>(u);
        u += dpp_move<kRowRor4>(u);
        u += dpp_move<kRowRor8>(u);
        if (kLR == 32) {
            float w_ = u;
            swap16(u, w_);
            u += w_;
        }
        if (rcol == 0) s_up2[g][rrow] = u;
    };

    bool failed = false;
    u32x2_t look[P - 1];
    // one step of 8 sequences; false: a wait in it expired in some wave of the workgroup
    auto step = [&](auto g_tag, int tt, auto cur_tag) __attribute__((always_inline)) {
        constexpr int g = decltype(g_tag)::value, cur = decltype(cur_tag)::value, nxt = cur ^ 1;
        f32x4_t acc[4];
        auto products = [&](const f16_t *rd, auto first_tag, auto count_tag) __attribute__((always_inline)) {
            constexpr int first = decltype(first_tag)::value, count = decltype(count_tag)::value;
            f16x8_t hb[count];
#pragma unroll
            for (int j = 0; j < count; ++j) hb[j] = *reinterpret_cast<const f16x8_t *>(rd + j * 32);
#pragma unroll
            for (int j = 0; j < count; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                    acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[first + j][q], hb[j], first + j == 0 ? zero : acc[q], 0, 0, 0);
                }
        };
        products(h_rd + g * 16 * kOP, std::integral_constant<int, 0>{}, std::integral_constant<int, kKH>{});
        if (SUB == 1 && tt > 0) ask(g, nxt, look);      // (earlier it finds the slots not yet written)
        __builtin_amdgcn_sched_barrier(0);
        if (tt > 1 && member == 0 && wave == 0) write_util(g, tt - 2);
        float ushare = 0.f;
        if (tt > 0) ushare = receive(g, tt, look);
        lds_barrier();
        if (s_fail) return false;
        products(p_rd + g * 16 * kPP, std::integral_constant<int, kKH>{}, std::integral_constant<int, kKP>{});
        if (tt > 0 && member == 0) share(g, ushare);

        // ---- hi + lo products of this lane's two units, the cell, the new h ----
        float z[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float keep = hn2 ? acc[q][2 + r] : acc[q][r], send = hn2 ? acc[q][r] : acc[q][2 + r];
                z[q][r] = fmaf(keep + dpp_move<kRowRor8>(send), inv_scale, xin[g][cur][q][r]);
            }
        fetch_x(g, min(tt + 1, nb - 1), xin[g][nxt]);
        float hv[2], upart = 0.f;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float ig = sigmoid_hw(z[0][r]), fg = sigmoid_hw(z[1][r]), gg = tanh_hw(z[2][r]), og = sigmoid_hw(z[3][r]);
            const float cn = fmaf(fg, c_reg[g][r], ig * gg);
            c_reg[g][r] = cn;
            float hn = og * tanh_hw(cn);
            asm volatile("" : "+v"(hn));     // opaque to the optimiser: hn is the rounded product from here on
            hv[r] = hn;
            upart = fmaf(ws_own[r], hn, upart);
        }
        uint32_t hi, lo;
        split2(hv[0], hv[1], hi, lo);
        const u32x2_t mine = gather(hi, lo);
        // to the partner first (the long way), then to this workgroup's own waves
        if (member != a.pair_mute) {
            const u32x2_t out = {(mine[0] & ~kFlag) | flag_of(tt), mine[1]};
            __builtin_amdgcn_raw_buffer_store_b64(out, e_rsrc, n * kOwn * 2 + wave * 32 + g4 * 8, (int)(g * kGroupSlots + (cur * P + member) * kSlot), 16);
        }
        // (the h that the next 8 sequences wait for is a turn old: it is there by now, unlike this one)
        if (SUB > 1 && (g + 1 < SUB ? tt > 0 : tt + 1 < nb)) ask((g + 1) % SUB, g + 1 < SUB ? nxt : cur, look);
        *reinterpret_cast<u32x2_t *>(h_wr + g * 16 * kOP) = mine;
        upart = rows_sum(upart);
        upart += dpp_move<kRowRor8>(upart);
        if (lane < 8) s_up[g][cur][wave][lane] = upart;
        if (tt == nb - 1) *reinterpret_cast<u32x2_t *>(h_wr + g * 16 * kOP) = u32x2_t{__float_as_uint(hv[0]), __float_as_uint(hv[1])};     // nobody reads it as an operand: see the end
        // (with more sequences in turn the barriers of the others come before these are read or replaced)
        if (SUB == 1) lds_barrier();
        return true;
    };
    auto turn = [&](int tt, auto cur_tag) __attribute__((always_inline)) {
        static_for<SUB>([&](auto g_tag) { if (!failed) failed = !step(g_tag, tt, cur_tag); });
    };
    for (int tt = 0; tt < nb && !failed; tt += 2) {
        turn(tt, std::integral_constant<int, 0>{});
        if (tt + 1 < nb && !failed) turn(tt + 1, std::integral_constant<int, 1>{});
    }
    if (!failed) {      // the last step's logit needs the partners' last h
        if (SUB > 1) lds_barrier();
        if (nb > 1 && member == 0 && wave == 0) {
#pragma unroll
            for (int g = 0; g < SUB; ++g) write_util(g, nb - 2);
        }
        lds_barrier();
#pragma unroll
        for (int g = 0; g < SUB; ++g) {
            ask(g, (nb - 1) & 1, look);
            share(g, receive(g, nb, look));
        }
        lds_barrier();
        failed = s_fail != 0;
        if (!failed && member == 0 && wave == 0) {
#pragma unroll
            for (int g = 0; g < SUB; ++g) write_util(g, nb - 1);
        }
    }
    // The state leaves the kernel as fp32, and not before this point: a member reads the partners' units of a.h when it
    // starts, and only their publications, received above, say that they have all done so (a launch of one step receives
    // nothing before its last one).
#pragma unroll
    for (int g = 0; g < SUB; ++g) {
        if (!failed && live[g]) {
            const u32x2_t hb = *reinterpret_cast<const u32x2_t *>(h_wr + g * 16 * kOP);      // (as the last step left it in LDS)
            *reinterpret_cast<float2 *>(a.h + s[g] * DG + unit0) = make_float2(__uint_as_float(hb[0]), __uint_as_float(hb[1]));
        }
        if (live[g]) {
#pragma unroll
            for (int r = 0; r < 2; ++r) a.c[s[g] * DG + unit0 + r] = failed ? __builtin_nanf("") : c_reg[g][r];
        }
        if (failed && tid < 8 && live[g]) {
            for (int t = 0; t < nb; ++t) {
                a.util[s[g] * a.N_cap + t0 + t] = __builtin_nanf("");
                a.gate[s[g] * a.N_cap + t0 + t] = __builtin_nanf("");
            }
        }
    }
    if (failed && tid == 0) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // sticky: the caller's to clear
}

// The same for launches so small that groups of 4 sequences fit the chip, P workgroups of 4 waves each.  The 16 columns of a
// matrix instruction hold their hi and lo terms twice over, and the four lanes that then hold the same sums take one of the four
// units each: half the nonlinearities and half the exchange.  A unit travels as a 4-byte word {hi, lo} whose hi carries the
// flag (a NaN keeps its lo term), so a lane takes four units of a sequence in 16 bytes, and a wave takes the slots of its own
// partners (one, at d_g = 512 two) instead of a part of everybody's.
// Measured (whole gate call, weights prepared; groups of 8 and groups of 4 on one machine): d_g = 256 32 sequences x 128 steps 226 ->
// 187 us, 64 x 64 127 -> 105, 256 x 64 132 -> 130; d_g = 512 32 x 128 319 -> 291, 128 x 64 208 -> 176.  (From machine to machine the same code
// takes 187 to 215 and 114 to 130 us at the first and third shape.)  At d_g = 256 a wave asks again 512 clocks after its first look and
// takes that answer, which is there when the first one would have had to be repeated: 187 -> 174 and 211 -> 205, 130 -> 126 and 114 -> 111
// us (with the later look alone 184 .. 187; sleeps of 4, 6 and 8 x 64 clocks 211, 208, 205).  Two looks that are both examined: 203; a look at four
// times the bytes per wave, straight into operand registers (no LDS, one barrier less): 283 against 226 with groups of 8.
template <int DG, int P>
__global__ __launch_bounds__(256) void lstm_rec_few_kernel(LstmArgs a, int t0, int nb)
{
    using G = Geo<DG>;
    constexpr int kKS = DG / 32, kNW = 4, kKH = kKS / P, kKP = kKS - kKH;       // k-steps; waves; k-steps over own units, over the partners'
    constexpr int NS = 4, kOwn = DG / P, kOP = kOwn + 8, kPP = DG - kOwn + 8;      // sequences; own units; row pitches in LDS
    constexpr int kMine = (P - 1 + kNW - 1) / kNW;                                 // partners of a wave, at most
    constexpr uint32_t kSlot = NS * kOwn * 4, kGroup = 2 * P * kSlot, kFlag = 0x4000u;      // [parity][member][unit / 4][sequence][unit % 4]
    constexpr int kPin = DG == 512 ? 15 : 0;                                    // k-steps whose weights are kept in accumulation registers
    static_assert(kOwn == 64, "a wave per 16 units, 16 lanes of 4 units per slot");
    static_assert(16 / NS * kGroup <= (DG == 256 ? kLstmPairExchBytes256 : 2 * kLstmOctExchBytes512), "the scratch planned for 16 sequences");
    __shared__ __align__(16) f16_t s_h[2 * NS * kOP], s_p[2 * NS * kPP];       // own units and the partners', row = plane * NS + sequence
    __shared__ float s_up[2][kNW][NS], s_up2[kNW][NS];                         // shares of the utility logit: own units (by step parity), partners'
    __shared__ int s_fail;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g4 = lane >> 4, sn = n % NS, j = n / NS;
    const int gpl = (a.BH + NS - 1) / NS;
    const int member = blockIdx.x % P, gid = blockIdx.x / P;
    const int l = gid / gpl, grp = gid % gpl;
    const bool live = grp * NS + sn < a.BH;
    const size_t s = (size_t)l * a.BH + min(grp * NS + sn, a.BH - 1);
    auto par_of = [&](int i) __attribute__((always_inline)) { return (member + 1 + i / kKH) % P; };
    const int tile = member * kNW + wave, own = wave * 16 + 4 * g4 + j, unit = member * kOwn + own;    // this lane's cell

    const bf16_t *w_s = static_cast<const bf16_t *>(a.w_s) + (size_t)l * DG;
    const float b_s = bf16_to_f32(static_cast<const bf16_t *>(a.b_s)[l]);
    const float inv_scale = ldexpf(1.f, -whh_scale_exp(whh_layer_max(a.whh_max_bits, l)));
    if (tid == 0) s_fail = 0;

    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(
        reinterpret_cast<const unsigned char *>(a.whh_packed + (((size_t)l * G::NW + tile / G::UT) * G::ITEMS + (tile % G::UT) * kKS) * 4 * 64),
        kKS * 4096);
    f16x8_t w[kKS][4];          // own units' k-steps, then the partners'
#pragma unroll
    for (int i = 0; i < kKS; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[i][q] = buffer_load16<f16x8_t>(w_rsrc, lane * 16 + q * 1024, (uint32_t)((i < kKH ? member * kKH + i : par_of(i - kKH) * kKH + (i - kKH) % kKH) * 4096));
            if (i < kPin) asm volatile("" : "+a"(w[i][q]));      // (left to itself the compiler moves them to vector registers before every use)
        }

    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(
        reinterpret_cast<const f32x4_t *>(a.xproj) + xp_block<DG>(l * ((a.BH + 15) / 16) + grp / (16 / NS), a.tb, 0, tile / G::UT, tile % G::UT, 0) * 64,
        (uint32_t)nb * G::NW * G::UT * 4096 - (uint32_t)tile * 4096);
    const uint32_t xoff = (uint32_t)((g4 * 16 + grp % (16 / NS) * NS + sn) * 16 + j * 4);
    // (two sets by step parity: a set in flight across the step boundary is not copied, which would wait for it)
    float xin[2][4];
    auto fetch_x = [&](int tt, float (&x)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            x[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x_rsrc, (int)(xoff + q * 1024), (int)((uint32_t)tt * G::NW * G::UT * 4096), 2));
    };
    fetch_x(0, xin[0]);

    const __amdgpu_buffer_rsrc_t e_rsrc = make_rsrc(a.exch + (size_t)gid * kGroup, kGroup);
    // the m-th partner that this wave takes the slot of, 0 .. P - 2, if there is one
    auto partner_of = [&](int m) __attribute__((always_inline)) { return wave + m * kNW; };
    // a look at their slots of parity `par`: sequence lane % 4, units 4 (lane / 4) .. + 3
    auto ask = [&](int par, u32x4_t (&v)[kMine]) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < kMine; ++m)
            if (const int p = partner_of(m); p < P - 1)
                v[m] = __builtin_amdgcn_raw_buffer_load_b128(e_rsrc, lane * 16, (int)((par * P + (member + 1 + p) % P) * kSlot), 16);
    };
    auto split = [](float h, f16_t &hi, f16_t &lo) __attribute__((always_inline)) {
        hi = (f16_t)h;
        lo = (f16_t)(h - (float)hi);
    };
    f16_t *const h_wr = s_h + (size_t)sn * kOP + own;                                     // + NS kOP: the lo terms
    const f16_t *const h_rd = s_h + (size_t)(n % (2 * NS)) * kOP + g4 * 8, *const p_rd = s_p + (size_t)(n % (2 * NS)) * kPP + g4 * 8;    // + i * 32
    f16_t *const p_wr = s_p + (size_t)(lane & 3) * kPP + (lane >> 2) * 4;      // + partner * kOwn, + NS kPP: the lo terms

    float c_reg = 0.f, h_last = 0.f;
    const float ws_own = bf16_to_f32(w_s[unit]);
#pragma unroll
    for (int p = 0; p < P; ++p) {        // own units, then the partners'
        const int u = (member + p) % P * kOwn + own;
        // (chunk 0 starts the recurrence from a zero state, whatever the buffers hold)
        const float h0 = live && t0 > 0 ? a.h[s * DG + u] : 0.f;
        if (p == 0) c_reg = live && t0 > 0 ? a.c[s * DG + u] : 0.f;
        f16_t hi, lo;
        split(h0, hi, lo);
        f16_t *dst = p == 0 ? h_wr : s_p + (size_t)sn * kPP + (p - 1) * kOwn + own;
        dst[0] = hi;
        dst[NS * (p == 0 ? kOP : kPP)] = lo;
    }
    float ws_par[kMine][4];              // of the units that this lane receives
#pragma unroll
    for (int m = 0; m < kMine; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) ws_par[m][e] = bf16_to_f32(w_s[(member + 1 + min(partner_of(m), P - 2)) % P * kOwn + (lane >> 2) * 4 + e]);
    __syncthreads();

    // the logit of a step from the shares of all members, by the last wave of member 0 (it receives least)
    auto write_util = [&](int step) __attribute__((always_inline)) {
        float u = b_s;
#pragma unroll
        for (int w_ = 0; w_ < kNW; ++w_)
            if (w_ < P - 1) u += s_up2[w_][sn];
#pragma unroll
        for (int w_ = 0; w_ < kNW; ++w_) u += s_up[step & 1][w_][sn];
        if (live && lane < NS) {
            a.util[s * a.N_cap + t0 + step] = u;
            a.gate[s * a.N_cap + t0 + step] = sigmoid_hw(u);
        }
    };
    auto flag_of = [](int tt) { return (tt >> 1) & 1 ? 0u : kFlag; };      // of the publication of step tt
    // The partners' h of step tt - 1 into LDS, from a look asked for earlier; more looks follow if it is not there yet.
    auto receive = [&](int tt, u32x4_t (&v)[kMine]) __attribute__((always_inline)) {
        typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
        const uint32_t flag = flag_of(tt - 1);
        auto complete = [&]() __attribute__((always_inline)) {
            uint32_t off = 0;
#pragma unroll
            for (int m = 0; m < kMine; ++m)
                if (partner_of(m) < P - 1) off |= (v[m][0] ^ flag) | (v[m][1] ^ flag) | (v[m][2] ^ flag) | (v[m][3] ^ flag);
            return __all((off & kFlag) == 0) != 0;
        };
        bool got = complete();
        for (int spin = 0; !got && spin < a.pair_spin_limit; ++spin) {
            asm volatile("" ::: "memory");
            if ((spin & 255) == 255 && s_fail) break;
            ask((tt - 1) & 1, v);
            got = complete();
        }
        if (!got) s_fail = 1;
        float u = 0.f;
#pragma unroll
        for (int m = 0; m < kMine; ++m)
            if (const int p = partner_of(m); p < P - 1) {
                const u32x2_t hi = {__builtin_amdgcn_perm(v[m][1], v[m][0], 0x05040100u) & ~(kFlag | kFlag << 16),
                                    __builtin_amdgcn_perm(v[m][3], v[m][2], 0x05040100u) & ~(kFlag | kFlag << 16)};
                const u32x2_t lo = {__builtin_amdgcn_perm(v[m][1], v[m][0], 0x07060302u), __builtin_amdgcn_perm(v[m][3], v[m][2], 0x07060302u)};
                *reinterpret_cast<u32x2_t *>(p_wr + p * kOwn) = hi;
                *reinterpret_cast<u32x2_t *>(p_wr + p * kOwn + NS * kPP) = lo;
                const f16x4_t hi4 = __builtin_bit_cast(f16x4_t, hi), lo4 = __builtin_bit_cast(f16x4_t, lo);
#pragma unroll
                for (int e = 0; e < 4; ++e) u = fmaf(ws_par[m][e], (float)lo4[e], fmaf(ws_par[m][e], (float)hi4[e], u));
            }
        return u;
    };
    // sums over the lanes of a sequence
    auto lanes_sum = [](float u) __attribute__((always_inline)) {
        u += dpp_move<kRowRor4>(u);
        u += dpp_move<kRowRor8>(u);
        return rows_sum(u);
    };
    // ... of what was received, which the products do not wait for
    auto put_share = [&](float u) __attribute__((always_inline)) {
        u = lanes_sum(u);
        if (wave < P - 1 && lane < NS) s_up2[wave][lane] = u;
    };

    bool failed = false;
    u32x4_t look[kMine];
    // one step; false: a wait in it expired in some wave of the workgroup
    auto step = [&](int tt, auto cur_tag) __attribute__((always_inline)) {
        constexpr int cur = decltype(cur_tag)::value, nxt = cur ^ 1;
        f32x4_t acc[4];
        auto products = [&](const f16_t *rd, auto first_tag, auto count_tag) __attribute__((always_inline)) {
            constexpr int first = decltype(first_tag)::value, count = decltype(count_tag)::value;
            f16x8_t hb[count];
#pragma unroll
            for (int i = 0; i < count; ++i) hb[i] = *reinterpret_cast<const f16x8_t *>(rd + i * 32);
#pragma unroll
            for (int i = 0; i < count; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                    acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[first + i][q], hb[i], first + i == 0 ? zero : acc[q], 0, 0, 0);
                }
        };
        products(h_rd, std::integral_constant<int, 0>{}, std::integral_constant<int, kKH>{});
        u32x4_t early[kMine];
        if (tt > 0) ask(nxt, DG == 256 ? early : look);
        if (DG == 256) {         // asked again, later, and that answer is taken: see above
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_sleep(8);
            if (tt > 0) ask(nxt, look);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (tt > 1 && member == 0 && wave == kNW - 1) write_util(tt - 2);
        float share = 0.f;
        if (tt > 0) {
            share = receive(tt, look);
            if (DG == 256) {     // (the first answer is thrown away, but asked for: without a use the request would be the compiler's to drop)
#pragma unroll
                for (int m = 0; m < kMine; ++m) asm volatile("" ::"v"(early[m]));
            }
        }
        lds_barrier();
        if (s_fail) return false;
        products(p_rd, std::integral_constant<int, kKH>{}, std::integral_constant<int, kKP>{});
        if (tt > 0 && member == 0) put_share(share);

        // ---- hi + lo products of this lane's unit, the cell, the new h ----
        float z[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = acc[q][r] + dpp_move<kRowRor4>(acc[q][r]);
            const float y0 = j & 1 ? y[1] : y[0], y1 = j & 1 ? y[3] : y[2];
            z[q] = fmaf(j & 2 ? y1 : y0, inv_scale, xin[cur][q]);
        }
        fetch_x(min(tt + 1, nb - 1), xin[nxt]);
        const float ig = sigmoid_hw(z[0]), fg = sigmoid_hw(z[1]), gg = tanh_hw(z[2]), og = sigmoid_hw(z[3]);
        c_reg = fmaf(fg, c_reg, ig * gg);
        h_last = og * tanh_hw(c_reg);
        asm volatile("" : "+v"(h_last));     // opaque to the optimiser: the rounded product from here on
        f16_t hi, lo;
        split(h_last, hi, lo);
        // to the partners first (the long way), then to this workgroup's own waves
        if (member != a.pair_mute) {
            const uint32_t word = __builtin_bit_cast(uint16_t, hi) | (uint32_t)__builtin_bit_cast(uint16_t, lo) << 16;
            __builtin_amdgcn_raw_buffer_store_b32((word & ~kFlag) | flag_of(tt), e_rsrc, ((wave * 4 + g4) * NS + sn) * 16 + j * 4,
                                                  (int)((cur * P + member) * kSlot), 16);
        }
        h_wr[0] = hi;
        h_wr[NS * kOP] = lo;
        const float upart = lanes_sum(ws_own * h_last);
        if (lane < NS) s_up[cur][wave][lane] = upart;
        lds_barrier();
        return true;
    };
    for (int tt = 0; tt < nb && !failed; tt += 2) {
        failed = !step(tt, std::integral_constant<int, 0>{});
        if (tt + 1 < nb && !failed) failed = !step(tt + 1, std::integral_constant<int, 1>{});
    }
    if (!failed) {      // the last step's logit needs the partners' last h
        if (nb > 1 && member == 0 && wave == kNW - 1) write_util(nb - 2);
        lds_barrier();
        ask((nb - 1) & 1, look);
        put_share(receive(nb, look));
        lds_barrier();
        failed = s_fail != 0;
        if (!failed && member == 0 && wave == kNW - 1) write_util(nb - 1);
    }
    // (not before this point: see lstm_rec_oct_kernel)
    if (live) {
        if (!failed) a.h[s * DG + unit] = h_last;
        a.c[s * DG + unit] = failed ? __builtin_nanf("") : c_reg;
    }
    if (failed && tid == 0) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // sticky: the caller's to clear
    if (failed && tid < NS && live) {
        for (int t = 0; t < nb; ++t) {
            a.util[s * a.N_cap + t0 + t] = __builtin_nanf("");
            a.gate[s * a.N_cap + t0 + t] = __builtin_nanf("");
        }
    }
}

template <int DG, int P, int SUB>
static void launch_oct(const LstmArgs &a, int t0, int nb, hipStream_t st)
{
    hipLaunchKernelGGL((lstm_rec_oct_kernel<DG, P, SUB>), dim3(P * a.L * ((a.BH + 8 * SUB - 1) / (8 * SUB))), dim3(4 * DG / P), 0, st, a, t0, nb);
}

template <int DG, int P>
static void launch_few(const LstmArgs &a, int t0, int nb, hipStream_t st)
{
    hipLaunchKernelGGL((lstm_rec_few_kernel<DG, P>), dim3(P * a.L * ((a.BH + 3) / 4)), dim3(256), 0, st, a, t0, nb);
}

// The smallest groups that the compute units hold at once, P workgroups each.
hipError_t launch_lstm_oct(const LstmArgs &a, int t0, int nb, hipStream_t st)
{
    const int fours = a.L * ((a.BH + 3) / 4), eights = a.L * ((a.BH + 7) / 8);
    if (a.d_g == 512) {
        if (8 * fours <= a.compute_units) launch_few<512, 8>(a, t0, nb, st);
        else if (8 * eights <= a.compute_units) launch_oct<512, 8, 1>(a, t0, nb, st);
        else launch_oct<512, 8, 2>(a, t0, nb, st);
    } else if (4 * fours <= a.compute_units) launch_few<256, 4>(a, t0, nb, st);
    else if (4 * eights <= a.compute_units) launch_oct<256, 4, 1>(a, t0, nb, st);
    else launch_oct<256, 2, 1>(a, t0, nb, st);
    return hipGetLastError();
}

}  // namespace kvev
