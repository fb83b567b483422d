// Host-visible launch interface between the C-ABI layer (api.hip) and the
// kernel files.  Everything here is plain data; shapes were validated by the
// caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace kvev {

#define KVEV_ATTN_MAX_SPLIT 256   // decode attention: most splits of one query's rows
constexpr size_t kCacheBytes = (size_t)256 << 20;     // what the memory-side cache holds

struct AttnArgs {
    const void *Q, *K, *V, *Kbar, *Vbar;
    const int32_t *idx, *count;
    void *O;
    float *part;          // split partials [S*Tq][nsplit][d+2] (o, m, l), or null when nsplit == 1
    int32_t *tickets;     // one arrival counter per (key-value sequence, query group), zero between calls; null when nsplit == 1
    int S, Tq, d;          // S: key-value sequences (L*B*H_kv)
    int G, Hkv;           // query heads per key-value head; key-value heads per (layer, batch row)
    int causal;           // 1: the Tq queries are the last Tq cached tokens and see nothing after themselves
    int T, T_cap, N_cap, k_cap;
    int win0;             // first raw token attended (0 for the dense baseline)
    int ring_first;       // compact form: the window buffer is a ring, its token t sits in row (ring_first + t) mod T_cap; else 0
    int gated;            // 1: kept summaries precede the raw rows
    int nsplit, rows_per_split;
    int rows_all;         // raw rows and kept summaries that a sequence can have
    int compute_units;    // of the device the launch goes to
    int stream;           // 1: the launch reads more than the memory-side cache holds: single-query loads carry the non-temporal hint
    float scale_log2e;    // log2(e) / sqrt(d)
};

struct PoolArgs {
    const void *K, *V;
    void *Kbar, *Vbar;
    const void *W1K, *b1K, *W2K, *b2K, *W1V, *b1V, *W2V, *b2V;   // per layer
    int L, BH, d, T_cap, C, N_cap, d_sum;
    int c0, c1;
    int mode;
    int compute_units;    // of the device the launch goes to
    int flush_shift;      // the persistent form writes its summaries once per 2^flush_shift ticks of the 100 MHz real-time counter
    void *wpack;          // workspace for the MLP weights in MFMA fragment order (pool_pack_bytes), or null: read as given
};

// The MLP weights of both sides re-laid per layer for the matrix cores: W1 and W2 as 1 KiB fragments (one 16-byte piece
// per lane, in the order the kernel walks them), then the biases as fp32.
constexpr size_t pool_pack_layer_bytes(int d, int d_sum) { return (size_t)8 * d_sum * d + (size_t)8 * (d_sum + d); }
inline size_t pool_pack_bytes(int L, int d, int d_sum) { return (size_t)L * pool_pack_layer_bytes(d, d_sum); }

struct LstmArgs {
    const void *Kbar, *Vbar;
    const void *W_ih, *W_hh, *b_ih, *b_hh, *w_s, *b_s;           // per layer
    float *h, *c, *util, *gate;
    float *xproj;         // workspace: fp32 input projections of a block of steps (fragment layout)
    const __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 *whh_packed;   // workspace: W_hh in fragment order (16-byte pieces; fp16 inside)
    uint32_t *whh_max_bits;   // workspace: 32 partial maxima of |W_hh| per layer as bit patterns (their maximum fixes the power-of-two scale)
    const __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 *wih_packed;   // workspace: W_ih in fragment order
    unsigned char *exch;  // workspace: exchange slots of the split recurrence (lstm_split_exch_bytes), or null
    size_t exch_bytes;    // 0: one workgroup per sequence group
    int split;            // workgroups that share a sequence group in the recurrence: 0 (one), 2, 4 or 8 (lstm_split)
    int quad_groups;      // split == 4: groups of 32 sequences per launch at most (compute units / 4)
    int pair_spin_limit;  // polls a wave of the paired recurrence spends on one wait before it gives up
    int pair_mute;        // member (0, 1) whose publications are withheld, -1: none (failure-path tests only)
    int32_t *status;      // workspace: word that a launch sets to 1 when a bounded wait expired (never cleared by the library)
    int prepared;         // 1: the packed weights are already in place (kvev_lstm_prepare), 0: this call packs them first
    int L, BH, d, N_cap, d_g;
    int compute_units;    // of the device the launch goes to
    int c0, c1;
    int tb;               // steps per workspace block
    int fused;            // 1: the single-kernel form (d_g = 256, 32 sequences per workgroup, no projections in scratch)
};

// How the gate spreads a group of sequences over workgroups that exchange h every step (0: one workgroup per 16
// sequences, no exchange).  Pairs: 16 sequences on two workgroups when the launch has at most one workgroup per compute
// unit (at d_g = 512 a single workgroup is bound by the weight stream out of L2 and a pair halves it; at d_g = 256 a
// pair keeps all of W_hh in registers).  Quadruples: at d_g = 512 with more than 16 sequences per layer, 32 sequences
// on four workgroups (a quarter of the stream each, and every fragment serves two blocks of sequences); a launch
// takes at most one workgroup per compute unit, larger calls are cut into several launches.  So all workgroups of a
// launch can be resident together on an idle device (bounded waits in the kernels cover the rest).
// Eight (lstm_oct.hip): at d_g = 512 while eight workgroups per 16 sequences fit the chip, which keeps all of W_hh in
// registers; up to there it is the faster one whatever the sequences per layer (512 x 64 steps 361 against 570 us, 16 a layer 392
// against 910; 1024 in two launches 730 against 579, so it ends there).  Caches of fewer than kLstmOctMinChunks chunks keep the
// others, which need no scratch for projections (8 KiB per sequence and step): 512 sequences x 8 steps take 77 us on four
// workgroups and 69 on eight, a difference that such a cache pays only once or twice.
// Its launches begin with all of W_hh from memory, so the form depends on the steps that the scratch holds as well; not on the
// steps of a call, so that a run cut into calls keeps its bits.  (What that costs: calls of 1 and 4 steps of 512 sequences
// take 23 and 46 us, four workgroups 18 and 44; one step of 15 layers of 17 sequences 33 and 22, of 256 in one layer 18.6 and
// 17.9; with 128 sequences and fewer it is the faster one.  A caller of such steps passes less scratch.)
// lstm_oct_min_block: the fewest steps per launch with which it is no slower than the kernel on four workgroups.  48 steps, four
// workgroups against eight with scratch for 4, 6, 8, 10 and 12 steps, us: d = 64, 512 sequences 377, eight 601 477 415 386 354;
// 15 layers of 17 433, 628 517 458 424 380; 8 layers of 32 376, 410 324 280; 256 in one 364, 363 304 291; d = 128, 512 434, 606
// 500 430 405 369, 8 layers of 32 430, 442 345.  Where pairs are the other form (at most 16 sequences a layer) it wins with any.
constexpr size_t kLstmPairExchBytes256 = 65536;     // scratch per group of 16 sequences and 256 hidden units
constexpr int kLstmOctMinChunks = 16;
constexpr size_t kLstmOctExchBytes512 = 32768;      // scratch per 8 sequences at d_g = 512 on eight workgroups
constexpr size_t kLstmQuadExchBytes = 131072;       // scratch per group of 32 sequences
inline int lstm_split(int d_g, int L, int BH, int N_cap, int compute_units, bool quad_allowed)
{
    const long long g16 = (long long)L * ((BH + 15) / 16);
    if (d_g == 512 && quad_allowed && N_cap >= kLstmOctMinChunks && 8 * g16 <= compute_units) return 8;
    if (d_g == 512 && quad_allowed && BH > 16 && compute_units >= 4) return 4;     // (more groups than fit at once: several launches)
    if ((d_g == 256 || d_g == 512) && 2 * g16 <= compute_units) return 2;
    return 0;
}
inline int lstm_oct_min_block(int L, int BH, int compute_units)
{
    return BH <= 16 ? 1 : 8ll * L * ((BH + 7) / 8) <= compute_units ? 6 : 12;
}
// At d_g = 256, launches that fit the chip with two workgroups per 8 sequences take lstm_rec_oct_kernel (four per 8 or per 4 where
// that fits too): 1024 sequences x 64 steps 224 us against 245 us on pairs per 16; above, the pairs remain.
inline bool lstm_takes_oct(int L, int BH, int compute_units) { return 2ll * L * ((BH + 7) / 8) <= compute_units; }
inline size_t lstm_split_exch_bytes(int split, int d_g, int L, int BH, int quad_groups)
{
    if (split == 4) {       // the slots of one launch (quad_groups groups at most), used again by the next
        const long long g32 = (long long)L * ((BH + 31) / 32);
        return (size_t)(g32 < quad_groups ? g32 : quad_groups) * kLstmQuadExchBytes;
    }
    if (split == 8) return (size_t)L * ((BH + 15) / 16) * 2 * kLstmOctExchBytes512;
    if (split == 2) return (size_t)L * ((BH + 15) / 16) * (d_g / 256) * kLstmPairExchBytes256;
    return 0;
}

struct SelectArgs {
    const float *util, *gate;
    int32_t *idx, *count;
    int S, N_cap, n_cand, k, k_cap, mode;
    float tau;
};

struct RetainArgs {
    const void *Kn, *Vn;          // new summaries [S, n_new_cap, d]
    const float *un;              // their scores [S, n_new_cap]
    void *Kc, *Vc;                // compact store [S, k_cap, d]
    int32_t *ids;                 // chunk ids of the store rows [S, k_cap], ascending
    float *uc;                    // their scores [S, k_cap]
    int32_t *count;               // [S]
    int S, row_bytes, k, k_cap, n_new_cap, first_chunk, n_new;
};

// Dynamic LDS beyond 64 KiB for a kernel, asked for once per device (a bit of `done` per device id): the attribute costs 0.06 to
// 0.25 us of host time per call (a decode call: 6).
template <class F> hipError_t allow_lds(F *kernel, int bytes, std::atomic<uint64_t> &done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (uint64_t)1 << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

hipError_t launch_attn_decode(const AttnArgs &a, int dtype, hipStream_t st);
int decode_queries(const AttnArgs &a, size_t elem);                       // its queries per workgroup: 1, 2 or 4 (elem: bytes of an element)
hipError_t launch_attn_decode_mfma(const AttnArgs &a, hipStream_t st);  // bf16, up to 4 queries per unit, unsplit: large launches
hipError_t launch_attn_mq(const AttnArgs &a, hipStream_t st);           // bf16 MFMA, many queries
hipError_t launch_select(const SelectArgs &a, hipStream_t st);
hipError_t launch_retain(const RetainArgs &a, hipStream_t st);
hipError_t launch_pool_generic(const PoolArgs &a, int dtype, hipStream_t st);
hipError_t launch_pool_mfma(const PoolArgs &a, hipStream_t st);          // bf16
// 16 waves on one tile at a time; workgroups that stay, with the MLP weights as given or re-laid in fragment order before
enum class PoolForm { one_tile, persistent, persistent_packed };
PoolForm pool_mfma_form(const PoolArgs &a);
hipError_t launch_pool_token_mfma(const PoolArgs &a, hipStream_t st);    // bf16, the MLP on every token
size_t pool_token_mfma_lds(int d, int d_sum);                            // its LDS need in bytes
hipError_t launch_lstm_generic(const LstmArgs &a, int dtype, hipStream_t st);
// its forms: up to 64 units, one sequence per workgroup with projections a block ahead; one or four sequences per workgroup (W_hh
// in registers up to 128 units, else read every step); one, bf16 rows of up to 192 units in registers as pairs
enum class LstmForm { chain, one, four, kept };
LstmForm lstm_generic_form(const LstmArgs &a, int dtype);
hipError_t launch_lstm_mfma(const LstmArgs &a, hipStream_t st);          // bf16
hipError_t launch_lstm_prepare(const LstmArgs &a, hipStream_t st);       // bf16: the packed weights alone
hipError_t launch_stream_probe(const void *src, size_t tiles, int tile_bytes, void *dst, int write_bytes, int hints, hipStream_t st);   // calibration
hipError_t launch_lstm_quad(const LstmArgs &a, hipStream_t st);          // bf16, d_g = 512: projection and recurrence of 32 sequences on four workgroups (weights already packed)
hipError_t launch_lstm_narrow(const LstmArgs &a, int t0, int nb, hipStream_t st);   // bf16, d_g = 64, 128: the recurrence, 8 sequences per workgroup
hipError_t launch_lstm_oct(const LstmArgs &a, int t0, int nb, hipStream_t st);   // bf16: the recurrence on two or four workgroups per 8 sequences or four per 4 (d_g = 256), on eight per 4, 8 or 16 (512)
hipError_t launch_lstm_fused(const LstmArgs &a, hipStream_t st);         // bf16, d_g = 256: the recurrence with the input projection inside (weights already packed)

}  // namespace kvev
