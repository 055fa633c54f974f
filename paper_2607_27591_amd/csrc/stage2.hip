// Stage 2 of the sparse decode step (Sec. 4.1 Stage 2) and the dense FFN
// (Sec. 2.1), which runs the same kernel over every channel.
//
// stage2_kernel, one workgroup per equal slice of the kept channels:
//  prologue  (sparse only) every workgroup finds the channel threshold of the
//            top-k_ff proxy scores itself, and the ascending global position
//            of every kept channel, so it can take exactly its slice of the
//            kept list (balanced to +-1 channel) without another launch.  When
//            a batch takes several launches, the first writes the kept list
//            to the workspace and the later ones read their slice from it.
//  gate/up   the slice's channels are cut into (channel, part of d) units
//            spread over the 16 waves; each unit streams two contiguous rows
//            with 16-byte loads and dot2 instructions (fp32 accumulation);
//            s_j = act(g_j) u_j is kept in LDS in fp32.
//  down      every thread owns 8 output columns and accumulates
//            s_j W_down[j, c..c+8] over the slice; the workgroup writes one
//            partial y.
// With INT4 base weights (WQ = 4) the two streaming loops read codes and
// per-group scales instead of 16-bit rows and dequantise on the fly.
// stage2_mfma_kernel and stage2_down_kernel (below) take batches of more than
// 8 rows of 16-bit weights.
// reduce_kernel sums the partial y of all workgroups in workgroup order and
// rounds y once.  No floating-point atomics: results are deterministic.
#include "common.hpp"
#include "kernels.hpp"
#include "topk.hpp"

namespace prox {

constexpr int kMaxSlice = (kMaxDFF + kStage2MaxWGs - 1) / kStage2MaxWGs;   // channels per WG
constexpr int kMaxParts = 8;

// d is cut into Q parts for the gate/up units: each part >= 2048 columns of
// 16-bit weights (up to four 16-byte loads per lane and matrix); with INT4
// codes, a power of two of equal parts of at most 4096 columns, so a part is
// one round of two 16-byte loads per lane and matrix.
__host__ __device__ inline int gateup_parts(int d, int nbt, int wq) {
    if (nbt > 2) return 1;
    if (wq == 4) {
        int q = 1;
        while (q * 4096 < d && q < kMaxParts) q *= 2;
        return q;
    }
    const int q = d / 2048;
    return q < 1 ? 1 : (q > kMaxParts ? kMaxParts : q);
}

__host__ __device__ inline bool x_in_lds(int d, int nbt) { return (size_t)nbt * d <= 32768; }

// Thread groups sharing the down projection's channels (> 1 only when d/8 <
// the block size), summed through LDS.
__host__ __device__ inline int stage2_down_groups(int d, int nbt) {
    const int ncg = d / 8;
    return (ncg >= kBlock || nbt > 4) ? 1 : kBlock / ncg;
}

// Dynamic LDS ahead of s: x (when staged; with INT4 weights as permuted
// pairs plus two sums per 32 inputs) or the down reduction buffer.
__host__ __device__ inline size_t stage2_head_bytes(int d, int nbt, int wq) {
    const size_t xbytes = x_in_lds(d, nbt) ? (size_t)nbt * d * 2 + (wq == 4 ? (size_t)nbt * (d / 32) * 8 : 0)
                                           : 0;
    const size_t red = stage2_down_groups(d, nbt) > 1 ? (size_t)kBlock * (nbt < 2 ? nbt : 2) * 8 * 4 : 0;
    return xbytes > red ? xbytes : red;
}

struct Stage2Smem {
    int list[kMaxSlice];
    float gu[kMaxSlice * kMaxParts * 2 * 2];   // [t][q][b][2] for nbt <= 2
};

// LDS of the selection prologue, besides the histogram.
struct ChanSel {
    SelScratch ss;
    int cnt[kMaxBlockWaves], eq[kMaxBlockWaves];   // per-wave counts
};

// The selection prologue of both Stage 2 kernels: this workgroup's slice of the
// kept channels (their ids to list[0..n), n returned, the slice's first
// kept-list position to p0_out) and its share of the mask.
// Every workgroup ranks the scores itself (top-k or the threshold rule), or,
// for the later launches of a multi-launch batch, reads the first launch's list.
// Bound by VALU issue (16 waves on 4 SIMDs: an instruction per score and thread
// costs ~0.2 us at d_ff 28672) and by the latency of its barriers, while HBM
// idles: so a score is compared a few times and counted by ballots, and only
// the waves whose run of channels meets the slice look at single channels.
// 8192 x 28672, one row, from the kernel's start to the first weight load: 7.4
// us (loads back at 2.7, the bracket's pass 2.2, its scan 0.5, counts 0.7, slice
// and x 1.2), against 8.6 with three radix passes over every score and a
// (row, wave) table of ballots.
// The caller synchronises before reading list.
template <int C>
__device__ __forceinline__ int stage2_slice(const float *__restrict__ scores, int f, int k_ff,
                                            uint8_t *__restrict__ mask,
                                            float *__restrict__ scores_copy, Select sel_rule,
                                            ScoreBracket br, int32_t *__restrict__ klist,
                                            int klist_mode, uint32_t *hist, ChanSel &cs, int *list,
                                            int &p0_out) {
    const int tid = threadIdx.x;
    const int nwg = gridDim.x, w = blockIdx.x;
    const bool sparse = scores != nullptr;
    // Channels of this workgroup: an even share of the n_ch kept channels
    // (with the threshold rule n_ch is only known after the selection).
    int n_ch = sparse ? k_ff : f;
    int p0, p1;
    auto split = [&](int n, int parts) {   // n parts < 2^25
        p0 = (int)((uint32_t)(w * n) / (uint32_t)parts);
        p1 = (int)((uint32_t)((w + 1) * n) / (uint32_t)parts);
    };
    // With the threshold rule the split is that of a launch for this count (the
    // grid is sized for every channel; the workgroups past it get none), so the
    // partial sums are those of the top-k launch with k = n_ch.
    auto split_tau = [&]() {
        const int nwg_k = min(nwg, stage2_wgs(n_ch));
        if (w < nwg_k) split(n_ch, nwg_k);
        else p0 = p1 = n_ch;
    };

    if (sparse && klist_mode == kListRead) {
        // A launch for the same call already selected: its list gives the
        // same slice as ranking again would.
        n_ch = klist[f];
        if (sel_rule.tau_mode) split_tau();
        else split(n_ch, nwg);
        for (int t = tid; t < p1 - p0; t += kBlock) list[t] = klist[p0 + t];
        __syncthreads();
    } else if (sparse) {
        const int lane = lane_id(), wid = wave_id();
        const int first = wid * C * kWave + lane;   // channel of item 0
        // Scores are |s~| >= 0, so their IEEE bit patterns order like the
        // values.  Loads past f return 0 (bounds-checked buffer loads).
        uint32_t key[C];
        const auto rs = buffer_of(scores, (uint32_t)f * 4);
#pragma unroll
        for (int r = 0; r < C; ++r) key[r] = buffer_load32(rs, (first + r * kWave) * 4);
        uint32_t v = 0, top = 0x7FFFFFFFu;   // kept: v <= key <= top, when `plain`
        int need = 0, bucket = 0;
        if (sel_rule.tau_mode) {
            // score >= tau as bit patterns, for tau > 0 (top: no NaN).
            if (sel_rule.tau > 0.0f) v = __float_as_uint(sel_rule.tau);
            top = 0x7F800000u;
        } else {
            bool done = false;
            if (br.stats) {
                // Every wave works out the bracket alike, all loads in flight.
                constexpr int NS = C <= 16 ? 4 : 8;   // tiles per lane: T is 64 up to d_ff 24448
                uint2 e[NS];
                const auto bs = buffer_of(br.stats, (uint32_t)br.n * 8);
#pragma unroll
                for (int t = 0; t < NS; ++t) e[t] = buffer_load64(bs, (t * kWave + lane) * 8);
                if (tid < kBracketBins<C> / 4) reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
                split(n_ch, nwg);
                float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
                for (int t = 0; t < NS; ++t) {
                    s1 += (float)e[t].x;
                    s2 += (float)e[t].y;
                }
                const float inv = 1.0f / (float)br.n;
                s1 = wave_sum(s1) * inv;
                s2 = wave_sum(s2) * inv;
                const float gap = s1 - s2;   // >= 0
                const float hi = s1 - gap * (br.at - br.half), lo = s1 - gap * (br.at + br.half);
                __syncthreads();   // the zeroed histogram
                if (lo >= 1.0f && hi < 2147483000.0f)
                    done = kth_score_bracket<C>(key, k_ff, (uint32_t)lo, (uint32_t)hi + 1u, hist,
                                                cs.ss, cs.cnt, v, need, bucket);
            } else {
                split(n_ch, nwg);
            }
            if (!done) kth_score<C>(key, f, first, k_ff, hist, cs.ss, v, need, bucket);
        }
        // Selected: v <= key <= top, but for v = 0 (keys past f are 0 too) and for
        // a k-th key of which only `need` equal ones, in index order, are in.
        const bool tie = need < bucket, plain = v != 0 && !tie;
        const uint32_t span = top - v;
        auto over = [&](int r) {
            if (sel_rule.tau_mode) return first + r * kWave < f && __uint_as_float(key[r]) >= sel_rule.tau;
            return tie ? key[r] > v : first + r * kWave < f;
        };
        auto equal = [&](int r) { return key[r] == v && first + r * kWave < f; };
        int n_over = 0, n_equal = 0;
        if (plain) {
#pragma unroll
            for (int r = 0; r < C; ++r) n_over += __popcll(__ballot(key[r] - v <= span));
        } else {
#pragma unroll
            for (int r = 0; r < C; ++r) {
                n_over += __popcll(__ballot(over(r)));
                n_equal += tie ? __popcll(__ballot(equal(r))) : 0;
            }
        }
        if (lane == 0) {
            cs.cnt[wid] = n_over;
            cs.eq[wid] = n_equal;
        }
        __syncthreads();
        // Counts of the waves before this one, and in all.
        const int ca = wave_inclusive_scan(lane < kMaxBlockWaves ? cs.cnt[lane] : 0);
        int base = wid > 0 ? __builtin_amdgcn_readlane(ca, wid - 1) : 0, n_sel = n_over, eq_run = 0;
        if (tie) {
            const int ce = wave_inclusive_scan(lane < kMaxBlockWaves ? cs.eq[lane] : 0);
            eq_run = wid > 0 ? __builtin_amdgcn_readlane(ce, wid - 1) : 0;
            base += min(need, eq_run);
            n_sel += min(need, eq_run + n_equal) - min(need, eq_run);
        }
        if (sel_rule.tau_mode) {
            n_ch = __builtin_amdgcn_readlane(ca, kMaxBlockWaves - 1);
            split_tau();
            if (w == 0 && tid == 0 && sel_rule.count) *sel_rule.count = n_ch;
        }
        // The waves that hold a part of the slice write it to the list; of the
        // mask's (wave, row) entries, w, w + nwg, ... are this workgroup's.
        const bool in_slice = p0 < p1 && base < p1 && base + n_sel > p0;   // wave-uniform
        const int m0 = (int)((uint32_t)(w + nwg - (int)((uint32_t)(wid * C) % (uint32_t)nwg)) % (uint32_t)nwg);
        if (in_slice || m0 < C) {
            uint32_t lo = 0, hi = 0;   // lane r: the ballot of row r's selected channels
            if (plain) {
#pragma unroll
                for (int r = 0; r < C; ++r) {
                    const uint64_t m = __ballot(key[r] - v <= span);
                    lo = write_lane(lo, (uint32_t)m, r);
                    hi = write_lane(hi, (uint32_t)(m >> 32), r);
                }
            } else {
#pragma unroll
                for (int r = 0; r < C; ++r) {
                    uint64_t m = __ballot(over(r));
                    if (tie) {
                        const uint64_t e = __ballot(equal(r));
                        m |= __ballot(((e >> lane) & 1) && eq_run + (int)lanes_below(e) < need);
                        eq_run += __popcll(e);
                    }
                    lo = write_lane(lo, (uint32_t)m, r);
                    hi = write_lane(hi, (uint32_t)(m >> 32), r);
                }
            }
            auto ballot_of = [&](int r) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, r) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)lo, r);
            };
            if (in_slice) {
                const int cnt = __popc(lo) + __popc(hi);
                const int pos = base + wave_inclusive_scan(cnt) - cnt;
                uint64_t hit = __ballot(cnt > 0 && pos < p1 && pos + cnt > p0);
                while (hit) {
                    const int r = __builtin_ctzll(hit);
                    hit &= hit - 1;
                    const uint64_t m = ballot_of(r);
                    const int q = __builtin_amdgcn_readlane(pos, r) + (int)lanes_below(m);
                    if (((m >> lane) & 1) && q >= p0 && q < p1) {
                        const int j = min(first + r * kWave, f - 1);   // rows in bounds
                        list[q - p0] = j;
                        if (klist_mode == kListWrite) klist[q] = j;
                    }
                }
            }
            for (int r = m0; r < C; r += nwg) {
                const uint64_t m = ballot_of(r);
                const int j = first + r * kWave;
                if (j < f) {
                    mask[j] = (uint8_t)((m >> lane) & 1);
                    if (scores_copy) scores_copy[j] = scores[j];
                }
            }
        }
        if (klist_mode == kListWrite && w == 0 && tid == 0) klist[f] = n_ch;
    } else {
        split(n_ch, nwg);
        for (int t = tid; t < p1 - p0; t += kBlock) list[t] = p0 + t;
    }
    p0_out = p0;
    return p1 - p0;
}

// WQ: 16 for 16-bit weights, 4 for INT4 codes (wt.sg/su/sd: their scales).
template <int NB, int DT, int C, int WQ>
__global__ __launch_bounds__(kBlock) void stage2_kernel(
    const uint16_t *__restrict__ x, int nb, int d, int f, Stage2Weights wt,
    const float *__restrict__ scores,   // NULL: dense FFN over all f channels
    int k_ff, uint8_t *__restrict__ mask, float *__restrict__ scores_copy,
    float *__restrict__ ypart, int ypart_stride,   // partial y rows per workgroup
    Select sel_rule, ScoreBracket br, int act,      // act: gate activation
    int32_t *__restrict__ klist, int klist_mode) {  // kept-channel list, KeptList mode
    static_assert(WQ == 16 || WQ == 4, "16-bit or INT4 weights");
    const uint16_t *__restrict__ wg = static_cast<const uint16_t *>(wt.wg);
    const uint16_t *__restrict__ wu = static_cast<const uint16_t *>(wt.wu);
    const uint16_t *__restrict__ wd = static_cast<const uint16_t *>(wt.wd);
    const int tid = threadIdx.x, wid = tid / kWave, lane = lane_id();

    __shared__ ChanSel cs;
    __shared__ Stage2Smem sm;
    // The channel selection's histogram, then x [NB][d] or the down reduction
    // | s [slice][NB].
    extern __shared__ __align__(16) float dyn[];

    // x (when it goes to LDS) is loaded before the selection, so its load
    // latency hides behind the ranking, and stored once the selection's
    // histogram is dead; with 64 score rows per thread the registers are
    // short, and x is loaded after it.  Thread t holds uint4 number
    // k * kBlock + t of the [NB][d / 8] vectors (rows past nb: zeros).
    const bool xl = x_in_lds(d, NB);   // always true with INT4 weights (host-checked)
    const int nvec = d / 8;
    constexpr int XPT = NB * kMaxDModel / 8 / kBlock < 4 ? NB * kMaxDModel / 8 / kBlock : 4;
    static_assert(XPT * kBlock * 8 >= 32768 || XPT * kBlock * 8 >= NB * kMaxDModel,
                  "x vectors per thread cover every x that fits in LDS");
    constexpr bool kEarlyX = C <= 32;
    uint4 xr[XPT];
    auto load_x = [&]() {
        const auto rs = buffer_of(x, xl ? (uint32_t)(nb * d) * 2 : 0u);
#pragma unroll
        for (int k = 0; k < XPT; ++k) xr[k] = buffer_load128(rs, (k * kBlock + tid) * 16);
    };
    if constexpr (kEarlyX) load_x();

    int p0;
    const int n = stage2_slice<C>(scores, f, k_ff, mask, scores_copy, sel_rule, br, klist,
                                  klist_mode, reinterpret_cast<uint32_t *>(dyn), cs, sm.list, p0);
    (void)p0;
    if constexpr (!kEarlyX) load_x();

    uint16_t *xs = reinterpret_cast<uint16_t *>(dyn);
    float2 *xsum = reinterpret_cast<float2 *>(dyn + (size_t)NB * d / 2);   // INT4: [NB][d / 32]
    if constexpr (WQ == 4) {
        // x as pairs (x_{8m+k}, x_{8m+k+4}), k = 0..3, one uint4 per 8
        // inputs: nibble k of a code word and nibble k + 4 sit in the two
        // halves of the word at the same bit offsets, so one dot2 takes both.
        // Per 32 inputs, the sums of x over the even-k pairs (the low halves
        // of the input words) and the odd-k pairs (the high halves): 4 per
        // lane in order, then the four lanes of a 32-input run (consecutive
        // threads) as (s0 + s1) + (s2 + s3).
#pragma unroll
        for (int k = 0; k < XPT; ++k) {
            const int e = k * kBlock + tid;
            const uint4 v = xr[k];
            if (e < NB * nvec)
                reinterpret_cast<uint4 *>(xs)[e] = make_uint4(
                    __builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                    __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u));
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
            float se = 0.0f, so = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                se += lo_to_float<DT>(vw[q]);
                so += hi_to_float<DT>(vw[q]);
            }
            se += dpp_move<kDppXor1>(se);
            so += dpp_move<kDppXor1>(so);
            se += dpp_move<kDppXor2>(se);
            so += dpp_move<kDppXor2>(so);
            if (e < NB * nvec && (tid & 3) == 0) xsum[e / 4] = make_float2(se, so);
        }
    } else if (xl) {
#pragma unroll
        for (int k = 0; k < XPT; ++k) {
            const int e = k * kBlock + tid;
            if (e < NB * nvec) reinterpret_cast<uint4 *>(xs)[e] = xr[k];
        }
    }
    __syncthreads();

    // ---- gate/up: units (channel t, part q) over the 16 waves ----
    const int Q = gateup_parts(d, NB, WQ);
    float *s_sh = dyn + align_up(stage2_head_bytes(d, NB, WQ), 16) / 4;   // [slice][NB]
    if constexpr (WQ == 4) {
        // 16-byte code vectors (32 inputs, inside one group) per row.  Each
        // code word's nibbles go under the exponent of the magic constant M
        // in pairs (k, k + 4): the even-k pairs from the low nibble of a byte
        // (value M + n), the odd-k pairs from its high nibble, moved only to
        // the top of the 16-bit mantissa (M + 8n for bf16 after one shift,
        // M + 16n in place for fp16).  Per vector and batch row the dot2 sums
        // t_e, t_o then give sum x (n - 8) = (t_e - B_e X_e) + (t_o - B_o X_o) / s
        // with the even and odd x sums X_e, X_o, and the group scale
        // multiplies that into the row's total.
        constexpr uint32_t M = Int4Magic<DT>::pair;
        constexpr bool kBf = DT == kBF16;
        constexpr uint32_t kOddMask = kBf ? 0x00780078u : 0x00F000F0u;
        constexpr int kOddShift = kBf ? 1 : 0;
        constexpr float kBiasE = kBf ? 136.0f : 1032.0f;                   // M + 8
        constexpr float kBiasO = kBf ? 128.0f + 64.0f : 1024.0f + 128.0f;  // M + 8 s
        constexpr float kInvO = kBf ? 0.125f : 0.0625f;                     // 1 / s
        const int ng = d / wt.group;
        const int nv4 = d / 32;
        // Scale index of vector v: v / (group / 32) by a multiply (exact for
        // v < 2^16).
        const uint32_t smagic = 0xFFFFFFFFu / (uint32_t)(wt.group / 32) + 1u;
        const uint4 *xs4 = reinterpret_cast<const uint4 *>(xs);
        constexpr int U = 2;   // vectors per lane and matrix in one round
        // One round of a unit: the codes and group scales of U vectors of
        // both rows.
        struct Round {
            uint4 g[U], u[U];
            uint16_t sg[U], su[U];
        };
        // Q is a power of two here: unit = t Q + q by shifts.
        const int lq = __builtin_ctz((unsigned)Q);
        auto part = [&](int q, int &v_begin, int &v_end) {
            v_begin = (q * nv4) >> lq;
            v_end = ((q + 1) * nv4) >> lq;
        };
        // The loads are issued unconditionally (lanes past the part read its
        // last vector, whose data consume skips), so the compiler can wait
        // for exactly the loads of the round it consumes while the next
        // round's are in flight.
        auto issue = [&](int unit, int v0, Round &R) {
            const int t = unit >> lq, q = unit & (Q - 1);
            const int j = sm.list[t];
            const uint4 *rg = reinterpret_cast<const uint4 *>(static_cast<const uint8_t *>(wt.wg) + (size_t)j * (d / 2));
            const uint4 *ru = reinterpret_cast<const uint4 *>(static_cast<const uint8_t *>(wt.wu) + (size_t)j * (d / 2));
            const uint16_t *sgr = wt.sg + (size_t)j * ng, *sur = wt.su + (size_t)j * ng;
            int v_begin, v_end;
            part(q, v_begin, v_end);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int vv = min(v_begin + v0 + u * kWave, v_end - 1);
                R.g[u] = load_stream16(rg + vv);
                R.u[u] = load_stream16(ru + vv);
                const int si = (int)__umulhi((uint32_t)vv, smagic);
                R.sg[u] = sgr[si];
                R.su[u] = sur[si];
            }
        };
        // Branch-free as well: a lane past the part computes on the part's
        // last vector with scale 0.
        auto consume = [&](int unit, int v0, const Round &R, float (&ag)[NB], float (&au)[NB]) {
            int v_begin, v_end;
            part(unit & (Q - 1), v_begin, v_end);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = v_begin + v0 + u * kWave < v_end;
                const int vv = min(v_begin + v0 + u * kWave, v_end - 1);
                {
                    const float scg = in ? f16_bits_to_float(R.sg[u]) : 0.0f;
                    const float scu = in ? f16_bits_to_float(R.su[u]) : 0.0f;
                    const uint32_t cgw[4] = {R.g[u].x, R.g[u].y, R.g[u].z, R.g[u].w};
                    const uint32_t cuw[4] = {R.u[u].x, R.u[u].y, R.u[u].z, R.u[u].w};
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        float tge = 0.0f, tgo = 0.0f, tue = 0.0f, tuo = 0.0f;
#pragma unroll
                        for (int w4 = 0; w4 < 4; ++w4) {
                            const uint4 P = xs4[(size_t)b * nvec + vv * 4 + w4];
                            const uint32_t g8 = cgw[w4] >> 8, u8 = cuw[w4] >> 8;
                            tge = dot2<DT>(P.x, and_or(cgw[w4], 0x000F000Fu, M), tge);
                            tue = dot2<DT>(P.x, and_or(cuw[w4], 0x000F000Fu, M), tue);
                            tgo = dot2<DT>(P.y, and_or(cgw[w4] >> kOddShift, kOddMask, M), tgo);
                            tuo = dot2<DT>(P.y, and_or(cuw[w4] >> kOddShift, kOddMask, M), tuo);
                            tge = dot2<DT>(P.z, and_or(g8, 0x000F000Fu, M), tge);
                            tue = dot2<DT>(P.z, and_or(u8, 0x000F000Fu, M), tue);
                            tgo = dot2<DT>(P.w, and_or(g8 >> kOddShift, kOddMask, M), tgo);
                            tuo = dot2<DT>(P.w, and_or(u8 >> kOddShift, kOddMask, M), tuo);
                        }
                        const float2 xv = xsum[b * nv4 + vv];
                        const float ge = tge - kBiasE * xv.x, go = tgo - kBiasO * xv.y;
                        const float ue = tue - kBiasE * xv.x, uo = tuo - kBiasO * xv.y;
                        ag[b] = fmaf(scg, fmaf(go, kInvO, ge), ag[b]);
                        au[b] = fmaf(scu, fmaf(uo, kInvO, ue), au[b]);
                    }
                }
            }
        };
        auto finish = [&](int unit, float (&ag)[NB], float (&au)[NB]) {
            const int t = unit >> lq, q = unit & (Q - 1);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float gs = wave_sum(ag[b]);
                const float us = wave_sum(au[b]);
                if (lane == 0) {
                    if (Q == 1) {
                        s_sh[t * NB + b] = gate_act(gs, act) * us;
                    } else {
                        sm.gu[((t * Q + q) * 2 + b) * 2 + 0] = gs;
                        sm.gu[((t * Q + q) * 2 + b) * 2 + 1] = us;
                    }
                }
            }
        };
        const int nunits = n * Q;
        if constexpr (NB == 1) {
            // A unit is one round (a part holds at most U * kWave vectors).
            // The wave's next unit is loaded before this one is computed, so
            // its load latency hides behind this unit's dequant and dot
            // products; two register sets take turns.
            auto run = [&](int unit, const Round &cur, Round &nxt) {
                // The last unit of the wave loads itself again (unused).
                issue(min(unit + kMaxBlockWaves, nunits - 1), lane, nxt);
                float ag[NB], au[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) ag[b] = au[b] = 0.0f;
                consume(unit, lane, cur, ag, au);
                finish(unit, ag, au);
            };
            Round ra, rb;
            // Nothing loaded before the loop is left in flight, so the waits
            // inside it only ever count the loop's own loads.
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            // The loop leaves at either half, so its back edge is taken only
            // after both register sets were consumed in turn (unit and count
            // wave-uniform, so the branches are scalar).
            int unit = __builtin_amdgcn_readfirstlane(wid);
            const int nu = __builtin_amdgcn_readfirstlane(nunits);
            if (unit < nu) {
                issue(unit, lane, ra);
                while (true) {
                    run(unit, ra, rb);
                    unit += kMaxBlockWaves;
                    if (unit >= nu) break;
                    run(unit, rb, ra);
                    unit += kMaxBlockWaves;
                    if (unit >= nu) break;
                }
            }
        } else {
            for (int unit = wid; unit < nunits; unit += kMaxBlockWaves) {
                int v_begin, v_end;
                part(unit & (Q - 1), v_begin, v_end);
                float ag[NB], au[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) ag[b] = au[b] = 0.0f;
                for (int v0 = lane; v_begin + v0 < v_end; v0 += kWave * U) {
                    Round R;
                    issue(unit, v0, R);
                    consume(unit, v0, R, ag, au);
                }
                finish(unit, ag, au);
            }
        }
    } else {
    const int qv = nvec / Q;                                   // 16-byte vectors per part
    constexpr int U = 4;
    for (int unit = wid; unit < n * Q; unit += kMaxBlockWaves) {
        const int t = unit / Q, q = unit % Q;
        const int j = sm.list[t];
        const uint4 *rg = reinterpret_cast<const uint4 *>(wg + (size_t)j * d);
        const uint4 *ru = reinterpret_cast<const uint4 *>(wu + (size_t)j * d);
        const int v_begin = q * qv, v_end = (q == Q - 1) ? nvec : v_begin + qv;
        float ag[NB], au[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) ag[b] = au[b] = 0.0f;
        for (int v0 = v_begin + lane; v0 < v_end; v0 += kWave * U) {
            uint4 gv[U], uv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (v0 + u * kWave < v_end) {
                    gv[u] = load_stream16(rg + v0 + u * kWave);
                    uv[u] = load_stream16(ru + v0 + u * kWave);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int vv = v0 + u * kWave;
                if (vv < v_end) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        uint4 xv;
                        if (xl) xv = reinterpret_cast<const uint4 *>(xs)[b * nvec + vv];
                        else xv = b < nb ? reinterpret_cast<const uint4 *>(x + (size_t)b * d)[vv]
                                         : make_uint4(0, 0, 0, 0);
                        ag[b] = dot2<DT>(xv.x, gv[u].x, ag[b]);
                        ag[b] = dot2<DT>(xv.y, gv[u].y, ag[b]);
                        ag[b] = dot2<DT>(xv.z, gv[u].z, ag[b]);
                        ag[b] = dot2<DT>(xv.w, gv[u].w, ag[b]);
                        au[b] = dot2<DT>(xv.x, uv[u].x, au[b]);
                        au[b] = dot2<DT>(xv.y, uv[u].y, au[b]);
                        au[b] = dot2<DT>(xv.z, uv[u].z, au[b]);
                        au[b] = dot2<DT>(xv.w, uv[u].w, au[b]);
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float gs = wave_sum(ag[b]);
            const float us = wave_sum(au[b]);
            if (lane == 0) {
                if (Q == 1) {
                    s_sh[t * NB + b] = gate_act(gs, act) * us;
                } else {
                    sm.gu[((t * Q + q) * 2 + b) * 2 + 0] = gs;
                    sm.gu[((t * Q + q) * 2 + b) * 2 + 1] = us;
                }
            }
        }
    }
    }
    __syncthreads();
    if (Q > 1) {
        for (int e = tid; e < n * NB; e += kBlock) {
            const int t = e / NB, b = e % NB;
            float gs = 0.0f, us = 0.0f;
            for (int q = 0; q < Q; ++q) {
                gs += sm.gu[((t * Q + q) * 2 + b) * 2 + 0];
                us += sm.gu[((t * Q + q) * 2 + b) * 2 + 1];
            }
            s_sh[t * NB + b] = gate_act(gs, act) * us;
        }
        __syncthreads();
    }

    // ---- down: partial y over this slice ----
    // d/8 groups of 8 columns; with fewer groups than threads (and NB <= 4)
    // the channels are split over G thread groups, summed through LDS in
    // group order.
    const int ncg = d / 8;
    constexpr int UD = 8;
    if constexpr (WQ == 16 && NB == 8) {
        // Eight batch rows up to d = 4096: 4 columns per thread, so that every
        // thread takes part (split channel sums would need more registers than
        // eight rows leave).  Each column is still summed over the slice in
        // order by one thread, as below.
        if (ncg < kBlock && d / 4 <= kBlock) {
            const int c4 = tid;
            if (c4 < d / 4) {
                float acc[NB][4];
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
                for (int t0 = 0; t0 < n; t0 += UD) {
                    uint2 wv[UD];
#pragma unroll
                    for (int u = 0; u < UD; ++u) {
                        const int t = t0 + u;
                        if (t < n) wv[u] = load_stream8(wd + (size_t)sm.list[t] * d + c4 * 4);
                    }
#pragma unroll
                    for (int u = 0; u < UD; ++u) {
                        const int t = t0 + u;
                        if (t < n) {
                            const float wf[4] = {lo_to_float<DT>(wv[u].x), hi_to_float<DT>(wv[u].x),
                                                 lo_to_float<DT>(wv[u].y), hi_to_float<DT>(wv[u].y)};
#pragma unroll
                            for (int b = 0; b < NB; ++b) {
                                const float sv = s_sh[t * NB + b];
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[b][e] = fmaf(sv, wf[e], acc[b][e]);
                            }
                        }
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (b < nb)
                        *reinterpret_cast<float4 *>(ypart + ((size_t)blockIdx.x * ypart_stride + b) * d + c4 * 4) =
                            make_float4(acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
                }
            }
            return;
        }
    }
    const int G = stage2_down_groups(d, NB);
    const int stride = G > 1 ? ncg : kBlock;
    const int gi = tid / stride, cgt = tid % stride;
    // Reuses the x area: two batch rows at a time, [row][8][G][ncg], so that the
    // threads of a wave (adjacent column groups) store to adjacent words.
    float *dred = dyn;
    for (int cg0 = 0; cg0 < ncg; cg0 += stride) {
        const int cg = cg0 + cgt;
        const bool active = cg < ncg && gi < G;
        float acc[NB][8];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[b][e] = 0.0f;
        if constexpr (WQ == 4) {
            // 8 columns per thread: one 32-bit code word and the scale of
            // their group per channel row.  The word's nibbles go under the
            // exponent of 1024.0 in fp16 pairs (columns e, e + 4): even e
            // from the low nibble of a byte (1024 + n), odd e from its high
            // nibble in place (1024 + 16 n); mixed-precision FMAs take each
            // half straight into the fp32 sums.  With S = sum_j s_j sigma_j,
            // sum_j s_j sigma_j (n - 8) is acc - 1032 S (even e) or
            // (acc - 1152 S) / 16 (odd e).
            const int ng = d / wt.group;
            constexpr uint32_t M16 = Int4Magic<kF16>::pair;
            constexpr int UD4 = NB == 1 ? 8 : 4;   // rows per round: 4 bytes each
            const uint32_t smagic = 0xFFFFFFFFu / (uint32_t)(wt.group / 8) + 1u;
            const int si = (int)__umulhi((uint32_t)cg, smagic);   // cg * 8 / group
            float ssum[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) ssum[b] = 0.0f;
            // One round: UD4 rows of this thread group's channels, loaded
            // unconditionally (rows past n repeat the last one and get s = 0)
            // so the loop can keep the next round in flight while it
            // computes this one.
            struct DRound {
                uint32_t cw[UD4];
                uint16_t sb[UD4];
            };
            auto issue = [&](int t0, DRound &R) {
#pragma unroll
                for (int u = 0; u < UD4; ++u) {
                    const int j = sm.list[min(t0 + u * G, n - 1)];
                    R.cw[u] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(
                        static_cast<const uint8_t *>(wt.wd) + (size_t)j * (d / 2) + cg * 4));
                    R.sb[u] = wt.sd[(size_t)j * ng + si];
                }
            };
            auto consume = [&](int t0, const DRound &R) {
#pragma unroll
                for (int u = 0; u < UD4; ++u) {
                    const int t = t0 + u * G;
                    const float sc = t < n ? f16_bits_to_float(R.sb[u]) : 0.0f;
                    const int tc = min(t, n - 1);
                    const uint32_t w8 = R.cw[u] >> 8;
                    const uint32_t h[4] = {and_or(R.cw[u], 0x000F000Fu, M16),
                                           and_or(R.cw[u], 0x00F000F0u, M16),
                                           and_or(w8, 0x000F000Fu, M16),
                                           and_or(w8, 0x00F000F0u, M16)};
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float sv = s_sh[tc * NB + b] * sc;
                        ssum[b] += sv;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc[b][e] = fmaf(sv, lo_to_float<kF16>(h[e]), acc[b][e]);
                            acc[b][e + 4] = fmaf(sv, hi_to_float<kF16>(h[e]), acc[b][e + 4]);
                        }
                    }
                }
            };
            // The loop leaves at either half, so its back edge follows the
            // use of both register sets.
            auto rounds = [&](int t0) {
                const int step = G * UD4;
                DRound ra, rb;
                issue(t0, ra);
                while (true) {
                    issue(min(t0 + step, n - 1), rb);
                    consume(t0, ra);
                    t0 += step;
                    if (t0 >= n) break;
                    issue(min(t0 + step, n - 1), ra);
                    consume(t0, rb);
                    t0 += step;
                    if (t0 >= n) break;
                }
            };
            if (active && n > 0) {
                // Thread groups of whole waves (the usual case) take scalar
                // round starts, and the loop's branches are uniform.
                if (stride % kWave == 0) rounds(__builtin_amdgcn_readfirstlane(gi));
                else rounds(gi);
            }
            // acc[b][e] is column 8 cg + e: columns e < 4 from the low halves
            // of the fp16 pairs, e + 4 from the high halves; odd columns came
            // from high nibbles.
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc[b][e] = (e & 1) ? (acc[b][e] - 1152.0f * ssum[b]) * 0.0625f
                                        : acc[b][e] - 1032.0f * ssum[b];
        } else if (active) {
            for (int t0 = gi; t0 < n; t0 += G * UD) {
                uint4 wv[UD];
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    const int t = t0 + u * G;
                    if (t < n) wv[u] = load_stream16(wd + (size_t)sm.list[t] * d + cg * 8);
                }
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    const int t = t0 + u * G;
                    if (t < n) {
                        const uint32_t w4[4] = {wv[u].x, wv[u].y, wv[u].z, wv[u].w};
                        float wf[8];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            wf[2 * q] = lo_to_float<DT>(w4[q]);
                            wf[2 * q + 1] = hi_to_float<DT>(w4[q]);
                        }
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            const float sv = s_sh[t * NB + b];
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[b][e] = fmaf(sv, wf[e], acc[b][e]);
                        }
                    }
                }
            }
        }
        if (G > 1) {
            // G > 1 implies ncg < kBlock, so this body runs exactly once and
            // every thread reaches these barriers.  Every group stores its sums,
            // then every thread adds the groups' in order for some four columns two
            // barriers per two rows, not one per group (1024 x 3072, eight groups,
            // one row: the call 23.0 -> 22.3 us; 1152 x 12000 dense, seven groups,
            // four rows: 30.5 -> 26.5; two groups: no change).
            constexpr int RB = NB < 2 ? NB : 2;
            for (int b0 = 0; b0 < NB; b0 += RB) {
                __syncthreads();   // x, or the previous rows' sums, are no longer read
                if (active) {
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (b >= b0 && b < b0 + RB) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) dred[(((b - b0) * 8 + e) * G + gi) * ncg + cg] = acc[b][e];
                        }
                }
                __syncthreads();
                for (int o = tid; o < RB * ncg * 2; o += kBlock) {   // row, column group, half
                    const int h = o & 1, c = (o >> 1) % ncg, b = (o >> 1) / ncg;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float *src = dred + (size_t)((b * 8 + 4 * h + e) * G) * ncg + c;
                        v[e] = src[0];
                        for (int g2 = 1; g2 < G; ++g2) v[e] += src[(size_t)g2 * ncg];
                    }
                    if (b0 + b < nb)
                        *reinterpret_cast<float4 *>(ypart + ((size_t)blockIdx.x * ypart_stride + b0 + b) * d + c * 8 + 4 * h) =
                            make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        } else if (active) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (b < nb) {
                    float4 *dst = reinterpret_cast<float4 *>(ypart + ((size_t)blockIdx.x * ypart_stride + b) * d + cg * 8);
                    dst[0] = make_float4(acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
                    dst[1] = make_float4(acc[b][4], acc[b][5], acc[b][6], acc[b][7]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// stage2_mfma_kernel + stage2_down_kernel: Stage 2 for 9 to 64 batch rows of
// 16-bit weights, so every kept row of the three matrices is read once for all
// of them.  RT: tiles of 16 batch rows (1, 2 or 4).
//  prologue  the slice of kept channels, as in stage2_kernel.
//  gate/up   on the matrix cores: the slice is cut into tiles of 16 channels,
//            and wave w takes the w-th sixteenth of d for every tile, so the
//            waves stream equal bytes however few channels the slice holds.
//            Per 32 inputs a lane loads 16 contiguous bytes of one channel row
//            of each matrix (A) and of one batch row of x per row tile (B, from
//            L2), and two 16 x 16 x 16 MFMAs per matrix and row tile add the
//            products into the tile's [16 channels][16 rows] fp32 sums.  The 16
//            waves' sums of a tile are added through LDS in wave order; s =
//            act(g) u goes to the workspace at the channel's kept-list position.
//  down      a second launch, below.
// A launch per 16 rows read the weights four times for 64 rows: 4096 x 14336,
// 30% kept, gate/up 4 x 23 us, now 42 (x comes from L2, one step in flight);
// 16 rows are as before, 27 us.
// ---------------------------------------------------------------------------
constexpr int kS2mTiles = 2;   // channel tiles per pass through the gate/up loop
constexpr int kS2mRed = kS2mTiles * 2 * kMaxBlockWaves * kWave;   // float4 per pass and row tile

size_t stage2_mfma_lds_bytes() {
    return (size_t)kS2mRed * 16 > kSelHistF32Bytes ? (size_t)kS2mRed * 16 : kSelHistF32Bytes;
}

bool stage2_mfma_ok(int d, int wq) { return stage2_mfma_shape(d, wq); }

template <int DT, int C, int RT>
__global__ __launch_bounds__(kBlock) void stage2_mfma_kernel(
    const uint16_t *__restrict__ x, int nb, int d, int f, Stage2Weights wt,
    const float *__restrict__ scores, int k_ff, uint8_t *__restrict__ mask,
    float *__restrict__ scores_copy, float *__restrict__ sbuf, Select sel_rule, ScoreBracket br,
    int act, int32_t *__restrict__ klist) {
    constexpr int R = 16 * RT;
    const uint16_t *__restrict__ wg = static_cast<const uint16_t *>(wt.wg);
    const uint16_t *__restrict__ wu = static_cast<const uint16_t *>(wt.wu);
    const int tid = threadIdx.x, wid = tid / kWave, lane = lane_id();

    __shared__ ChanSel cs;
    __shared__ int list[kMaxSlice];
    // The channel selection's histogram, then red [tiles][2][waves][lanes] float4.
    extern __shared__ __align__(16) float dyn[];
    float4 *red = reinterpret_cast<float4 *>(dyn);

    int p0;
    const int n = stage2_slice<C>(scores, f, k_ff, mask, scores_copy, sel_rule, br, klist,
                                  scores ? kListWrite : kListNone, reinterpret_cast<uint32_t *>(dyn),
                                  cs, list, p0);
    __syncthreads();

    // ---- gate/up ----
    const int nsteps = d / 32;   // steps of 32 inputs
    const int k_lo = wid * nsteps / kMaxBlockWaves, k_hi = (wid + 1) * nsteps / kMaxBlockWaves;
    const int r = lane % 16, g4 = lane / 16;
    const auto xb = buffer_of(x, (uint32_t)(nb * d) * 2);   // rows past nb read 0
    const int ntiles = (n + 15) / 16;
    constexpr int U = RT == 1 ? 2 : 1;   // steps in flight per lane
    for (int t0 = 0; t0 < ntiles; t0 += kS2mTiles) {
        const uint16_t *rg[kS2mTiles], *ru[kS2mTiles];
        bool live[kS2mTiles];
        v4f ag[kS2mTiles][RT], au[kS2mTiles][RT];
#pragma unroll
        for (int tt = 0; tt < kS2mTiles; ++tt) {
            const int t = (t0 + tt) * 16 + r;
            live[tt] = t < n;
            const int j = live[tt] ? list[t] : 0;
            rg[tt] = wg + (size_t)j * d + 8 * g4;
            ru[tt] = wu + (size_t)j * d + 8 * g4;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) ag[tt][rt] = au[tt][rt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int k = k_lo; k < k_hi; k += U) {
            uint4 xv[U][RT], gv[kS2mTiles][U], uv[kS2mTiles][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kk = k + u;
                const bool in = kk < k_hi;
#pragma unroll
                for (int tt = 0; tt < kS2mTiles; ++tt) {
                    const bool ld = in && live[tt];
                    gv[tt][u] = ld ? load_stream16(rg[tt] + kk * 32) : make_uint4(0, 0, 0, 0);
                    uv[tt][u] = ld ? load_stream16(ru[tt] + kk * 32) : make_uint4(0, 0, 0, 0);
                }
                // Past k_hi the weights are 0 and x may be anything finite of its rows.
                const int xo = (r * d + min(kk, nsteps - 1) * 32 + 8 * g4) * 2;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) xv[u][rt] = buffer_load128(xb, xo + rt * 16 * d * 2);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // Inputs 8 g4 + 0..3 of the step in the first MFMA, 8 g4 + 4..7
                // in the second: A and B take the same inputs in the same slots.
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const uint2 xa = make_uint2(xv[u][rt].x, xv[u][rt].y);
                    const uint2 xc = make_uint2(xv[u][rt].z, xv[u][rt].w);
#pragma unroll
                    for (int tt = 0; tt < kS2mTiles; ++tt) {
                        ag[tt][rt] = mfma16<DT>(make_uint2(gv[tt][u].x, gv[tt][u].y), xa, ag[tt][rt]);
                        ag[tt][rt] = mfma16<DT>(make_uint2(gv[tt][u].z, gv[tt][u].w), xc, ag[tt][rt]);
                        au[tt][rt] = mfma16<DT>(make_uint2(uv[tt][u].x, uv[tt][u].y), xa, au[tt][rt]);
                        au[tt][rt] = mfma16<DT>(make_uint2(uv[tt][u].z, uv[tt][u].w), xc, au[tt][rt]);
                    }
                }
            }
        }
        // Lane l holds channel 4 (l / 16) + e, batch row l % 16 of each tile.
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
            for (int tt = 0; tt < kS2mTiles; ++tt) {
                const v4f g = ag[tt][rt], u = au[tt][rt];
                red[((tt * 2 + 0) * kMaxBlockWaves + wid) * kWave + lane] = make_float4(g[0], g[1], g[2], g[3]);
                red[((tt * 2 + 1) * kMaxBlockWaves + wid) * kWave + lane] = make_float4(u[0], u[1], u[2], u[3]);
            }
            __syncthreads();
            if (tid < kS2mTiles * kWave * 4) {
                const int tt = tid / (kWave * 4), ln = (tid / 4) % kWave, e = tid % 4;
                const float *rf = reinterpret_cast<const float *>(red);
                float gs = 0.0f, us = 0.0f;
                for (int w = 0; w < kMaxBlockWaves; ++w) {
                    gs += rf[(((tt * 2 + 0) * kMaxBlockWaves + w) * kWave + ln) * 4 + e];
                    us += rf[(((tt * 2 + 1) * kMaxBlockWaves + w) * kWave + ln) * 4 + e];
                }
                const int t = (t0 + tt) * 16 + 4 * (ln / 16) + e;
                if (t < n) sbuf[(size_t)(p0 + t) * R + rt * 16 + ln % 16] = gate_act(gs, act) * us;
            }
            __syncthreads();
        }
    }
}

// Down projection on the matrix cores: y[b][c] = sum_j s[b][j] W_down[j][c].  The
// kept list is cut into stage2_down_groups groups; a workgroup takes one group and
// 256 columns: four waves of 64 columns by four splits of the channels, in
// blocks of 16.  A lane loads 8 bytes (4 columns) of four channel rows, which
// paired by v_perm are the B operands of 16 x 16 x 16 MFMAs (4 rows of k per
// lane); s is the A operand, kept to fp32 precision: for bf16 weights as the sum
// of three bf16 (8 bits each: the 24 of fp32), three MFMAs; for fp16, whose range
// that would not fit, 16 x 16 x 4 fp32 MFMAs on the widened weights.  s is split
// on its way to LDS, kDownChunk channels at a time, in operand order.  The splits'
// sums meet in LDS in order.
// Against VALU FMAs (16 per weight, 64 groups of partial
// y): 4096 x 14336, 30% kept, 11 us instead of 18 at 16 rows, 23 instead of 4 x 17
// at 64 (4.2 and 16.8 MB of partial y instead of 16.8 and 67).
constexpr int kDownCols = 256;     // columns per workgroup
constexpr int kDownChunk = 320;    // channels staged at a time
constexpr int kDownSplit = 4;

template <int DT>
constexpr int kDownSBytes = DT == kBF16 ? 6 : 4;   // of one s in LDS

size_t stage2_down_lds_bytes(int dtype, int rt, int n_max, int groups) {
    const int m = (n_max + groups - 1) / groups;
    const size_t blocks = (size_t)((m < kDownChunk ? m : kDownChunk) + 15) / 16;
    const size_t s = blocks * 16 * rt * 16 * (dtype == kBF16 ? 6 : 4) + blocks * 16 * 4;
    const size_t red = (size_t)kBlock * 64;   // 16 sums per thread
    return s > red ? s : red;
}

// The next bf16 part of v, and what remains.  Cut off, not rounded: a finite v never
// becomes infinite, and three parts still hold the 24 bits.  Nothing remains of an
// infinity (Inf - Inf would be NaN).
__device__ __forceinline__ uint32_t bf16_part(float &v) {
    const uint32_t h = __float_as_uint(v) >> 16;
    const float t = bf16_lo(h);
    v = v == t ? 0.0f : v - t;
    return h;
}

template <int DT, int RT>
__global__ __launch_bounds__(kBlock) void stage2_down_kernel(
    int nb, int d, int f, const uint16_t *__restrict__ wd, const float *__restrict__ sbuf,
    const int32_t *__restrict__ klist, float *__restrict__ ypart, int ypart_stride) {
    constexpr int R = 16 * RT;
    extern __shared__ __align__(16) unsigned char dsm[];   // s in operand order | ids, then red
    const int tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    const int n_ch = klist ? klist[f] : f;
    const int grp = blockIdx.y, groups = gridDim.y;
    const int q0 = (int)((uint32_t)(grp * n_ch) / (uint32_t)groups);
    const int m = (int)((uint32_t)((grp + 1) * n_ch) / (uint32_t)groups) - q0;
    const int wc = wid % 4, sp = wid / 4;
    const int col = blockIdx.x * kDownCols + wc * 64 + (lane % 16) * 4;   // first of 4 columns
    const bool active = col < d;   // whole waves: d is a multiple of 128
    const int g = lane / 16;

    v4f acc[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[rt][c] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    for (int c0 = 0; c0 < m; c0 += kDownChunk) {
        const int mc = min(kDownChunk, m - c0);
        const int blocks = (mc + 15) / 16;
        int *ids = reinterpret_cast<int *>(dsm + (size_t)blocks * 16 * R * kDownSBytes<DT>);
        if (c0 > 0) __syncthreads();   // the previous chunk is used up
        // Pad channels repeat the last row, with s = 0.
        for (int t = tid; t < blocks * 16; t += kBlock) {
            const int q = q0 + c0 + min(t, mc - 1);
            ids[t] = klist ? klist[q] : q;
        }
        // Thread: batch row b, channels 4 t4 .. 4 t4 + 3 of the chunk.
        for (int e = tid; e < blocks * 4 * R; e += kBlock) {
            const int b = e % R, t4 = e / R;
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = t4 * 4 + q;
                v[q] = sbuf[(size_t)(q0 + c0 + min(t, mc - 1)) * R + b];
                if (t >= mc || b >= nb) v[q] = 0.0f;
            }
            // Operand slot: block t4 / 4, row tile b / 16, lane (t4 % 4) * 16 + b % 16.
            const int slot = ((t4 / 4) * RT + b / 16) * kWave + (t4 % 4) * 16 + b % 16;
            if constexpr (DT == kBF16) {
                uint2 *dst = reinterpret_cast<uint2 *>(dsm) + slot;
#pragma unroll
                for (int part = 0; part < 3; ++part) {
                    const uint32_t h0 = bf16_part(v[0]), h1 = bf16_part(v[1]);
                    const uint32_t h2 = bf16_part(v[2]), h3 = bf16_part(v[3]);
                    dst[(size_t)part * blocks * RT * kWave] = make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
                }
            } else {
                reinterpret_cast<float4 *>(dsm)[slot] = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
        __syncthreads();
        const int b_lo = sp * blocks / kDownSplit, b_hi = (sp + 1) * blocks / kDownSplit;
        constexpr int U = RT == 4 ? 3 : 5;   // blocks in flight
        if (active) {
            for (int k0 = b_lo; k0 < b_hi; k0 += U) {
                uint2 w[U][4];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int4 id = *reinterpret_cast<const int4 *>(ids + min(k0 + u, b_hi - 1) * 16 + 4 * g);
                    const int j[4] = {id.x, id.y, id.z, id.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[u][e] = load_stream8(wd + (size_t)j[e] * d + col);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (k0 + u >= b_hi) break;   // uniform
                    const int blk = k0 + u;
                    if constexpr (DT == kBF16) {
                        uint2 bop[4];   // column c: rows (0, 1) and (2, 3) side by side
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t sel = (c & 1) ? 0x07060302u : 0x05040100u;
                            const uint32_t a0 = c < 2 ? w[u][0].x : w[u][0].y, a1 = c < 2 ? w[u][1].x : w[u][1].y;
                            const uint32_t a2 = c < 2 ? w[u][2].x : w[u][2].y, a3 = c < 2 ? w[u][3].x : w[u][3].y;
                            bop[c] = make_uint2(__builtin_amdgcn_perm(a1, a0, sel), __builtin_amdgcn_perm(a3, a2, sel));
                        }
                        const uint2 *sl = reinterpret_cast<const uint2 *>(dsm) + (size_t)blk * RT * kWave + lane;
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                            for (int part = 0; part < 3; ++part) {
                                const uint2 a = sl[((size_t)part * blocks * RT + rt) * kWave];
#pragma unroll
                                for (int c = 0; c < 4; ++c) acc[rt][c] = mfma16<DT>(a, bop[c], acc[rt][c]);
                            }
                    } else {
                        const float4 *sl = reinterpret_cast<const float4 *>(dsm) + (size_t)blk * RT * kWave + lane;
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) {
                            const float4 a = sl[rt * kWave];
                            const float av[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float wf[4] = {lo_to_float<DT>(w[u][e].x), hi_to_float<DT>(w[u][e].x),
                                                     lo_to_float<DT>(w[u][e].y), hi_to_float<DT>(w[u][e].y)};
#pragma unroll
                                for (int c = 0; c < 4; ++c)
                                    acc[rt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], wf[c], acc[rt][c], 0, 0, 0);
                            }
                        }
                    }
                }
            }
        }
    }
    // The splits' sums in order.  Lane l of a wave holds rows 4 (l / 16) + e,
    // columns 4 (l % 16) + c; thread (e, wave, lane) of the output takes one row's
    // 4 columns.
    float4 *red = reinterpret_cast<float4 *>(dsm);   // [split][wave][c][lane]
    for (int rt = 0; rt < RT; ++rt) {
        __syncthreads();   // s, or the previous row tile, is used up
#pragma unroll
        for (int q = 0; q < RT; ++q)
            if (q == rt) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    red[((sp * 4 + wc) * 4 + c) * kWave + lane] =
                        make_float4(acc[q][c][0], acc[q][c][1], acc[q][c][2], acc[q][c][3]);
            }
        __syncthreads();
        const int e = wid / 4;   // the wave's output row within 4 (wave column group wc as before)
        float o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float t = 0.0f;
#pragma unroll
            for (int q = 0; q < kDownSplit; ++q)
                t += reinterpret_cast<const float *>(&red[((q * 4 + wc) * 4 + c) * kWave + lane])[e];
            o[c] = t;
        }
        const int b = rt * 16 + 4 * g + e;
        if (active && b < nb)
            *reinterpret_cast<float4 *>(ypart + ((size_t)grp * ypart_stride + b) * d + col) =
                make_float4(o[0], o[1], o[2], o[3]);
    }
}

// y[b][c] = sum over the Stage 2 workgroups of the partial y, rounded once.
// A 256-thread block covers kReduceCols columns; thread t takes column
// t % kReduceCols and every kReduceGroups-th workgroup from t / kReduceCols,
// with all its loads in flight at once, and the groups are added in a fixed
// order through LDS, so the result is deterministic.
constexpr int kReduceThreads = 256;
constexpr int kReduceCols = 32;
constexpr int kReduceGroups = kReduceThreads / kReduceCols;                 // 8
constexpr int kReducePerThread = (kStage2MaxWGs + kReduceGroups - 1) / kReduceGroups;   // 32
constexpr int kReduceSmall = kStage2DownMaxGroups / kReduceGroups;   // 2: for <= 16 partials

// UPT: partials per thread (kReducePerThread, or kReduceSmall when nwg <= 16,
// which adds the same terms in the same order).

template <int DT, int UPT>
__global__ __launch_bounds__(kReduceThreads) void reduce_kernel(const float *__restrict__ ypart, int nwg,
                                                                int nbt, int d, uint16_t *__restrict__ y) {
    __shared__ float red[kReduceGroups][kReduceCols];
    const int b = blockIdx.y, col = threadIdx.x % kReduceCols, g = threadIdx.x / kReduceCols;
    const int c = blockIdx.x * kReduceCols + col;
    const int cc = min(c, d - 1);
    float v[UPT];
#pragma unroll
    for (int u = 0; u < UPT; ++u) {   // clamped loads, masked below
        const int w = min(g + u * kReduceGroups, nwg - 1);
        v[u] = ypart[((size_t)w * nbt + b) * d + cc];
    }
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < UPT; ++u)
        if (g + u * kReduceGroups < nwg) acc += v[u];
    red[g][col] = acc;
    __syncthreads();
    if (g == 0 && c < d) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < kReduceGroups; ++q) s += red[q][col];
        y[(size_t)b * d + c] = float_to_half<DT>(s);
    }
}

template <int DT>
__global__ __launch_bounds__(1024) void add_rmsnorm_kernel(const uint16_t *__restrict__ x,
                                                           const uint16_t *__restrict__ y, int d,
                                                           float eps, uint16_t *out) {
    __shared__ float wsum[1024 / kWave];
    const int b = blockIdx.x;
    const uint16_t *xb = x + (size_t)b * d, *yb = y + (size_t)b * d;
    float ss = 0.0f;
    for (int i = threadIdx.x; i < d; i += 1024) {
        const float r = half_to_float<DT>(xb[i]) + half_to_float<DT>(yb[i]);
        ss = fmaf(r, r, ss);
    }
    ss = wave_sum(ss);
    if (lane_id() == 0) wsum[threadIdx.x / kWave] = ss;
    __syncthreads();
    float tot = 0.0f;
    for (int w = 0; w < 1024 / kWave; ++w) tot += wsum[w];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    __syncthreads();   // every thread has read its x, y before out (which may alias x) is written
    for (int i = threadIdx.x; i < d; i += 1024) {
        const float r = half_to_float<DT>(xb[i]) + half_to_float<DT>(yb[i]);
        out[(size_t)b * d + i] = float_to_half<DT>(r * inv);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// sparse: the channel selection's histogram shares the front of the space.
size_t stage2_lds_bytes(int d, int nbt, int wq, bool sparse) {
    const size_t b = align_up(stage2_head_bytes(d, nbt, wq), 16) + (size_t)kMaxSlice * nbt * 4;
    return sparse && b < kSelHistF32Bytes ? kSelHistF32Bytes : b;
}

int stage2_rows(int d, int wq) {
    if (wq != 4) return kStage2MaxNB;
    int r = kStage2MaxNB;   // a power of two, so the launch's row template is r
    while (r > 1 && !x_in_lds(d, r)) r /= 2;
    return r;
}

template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
    // Dynamic LDS above 64 KiB must be allowed per kernel (gfx950 has 160 KiB).
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int NB, int DT, int C, int WQ>
static hipError_t launch_stage2_t(const void *x, int nb, int d, int f, const Stage2Weights &wt,
                                  const float *scores, int k_ff, uint8_t *mask, float *scores_copy,
                                  float *ypart, int ystride, int nwg, Select sel_rule, ScoreBracket br, int act,
                                  int32_t *klist, int klist_mode, hipStream_t st) {
    if (WQ == 4 && !x_in_lds(d, NB)) return hipErrorInvalidValue;
    const size_t lds = stage2_lds_bytes(d, NB, WQ, scores != nullptr);
    hipError_t e = allow_lds(stage2_kernel<NB, DT, C, WQ>, lds);
    if (e != hipSuccess) return e;
    stage2_kernel<NB, DT, C, WQ><<<nwg, kBlock, lds, st>>>(
        static_cast<const uint16_t *>(x), nb, d, f, wt, scores, k_ff, mask, scores_copy, ypart,
        ystride, sel_rule, br, act, klist, klist_mode);
    return hipGetLastError();
}

template <int NB, int DT, int WQ>
static hipError_t launch_stage2_c(const void *x, int nb, int d, int f, const Stage2Weights &wt,
                                  const float *scores, int k_ff, uint8_t *mask, float *scores_copy,
                                  float *ypart, int ystride, int nwg, Select sel_rule, ScoreBracket br, int act,
                                  int32_t *klist, int klist_mode, hipStream_t st) {
    // C = score rows per thread of the channel top-k (the dense path has none).
#define S2C(C_) launch_stage2_t<NB, DT, C_, WQ>(x, nb, d, f, wt, scores, k_ff, mask, scores_copy, ypart, ystride, nwg, sel_rule, br, act, klist, klist_mode, st)
    // As few score rows per thread as d_ff needs (below 16 not for eight rows
    // of INT4 weights, whose registers are full).
    if constexpr (WQ == 16 || NB <= 4) {
        if (scores && f <= 4 * kBlock) return S2C(4);
        if (scores && f <= 8 * kBlock) return S2C(8);
        if (scores && f <= 12 * kBlock) return S2C(12);
    }
    if (!scores || f <= 16 * kBlock) return S2C(16);
    if (f <= 28 * kBlock) return S2C(28);
    if (f <= 32 * kBlock) return S2C(32);
    return S2C(64);
#undef S2C
}

hipError_t launch_stage2(int dtype, const void *x, int nb, int d, int f, const Stage2Weights &wt,
                         const float *scores, int k_ff, uint8_t *mask, float *scores_copy,
                         float *ypart, int ystride, int nwg, Select sel_rule, ScoreBracket br,
                         int act, int32_t *klist, int klist_mode, hipStream_t st) {
    if (nb < 1 || nb > stage2_rows(d, wt.wq)) return hipErrorInvalidValue;
    if (klist_mode != kListNone && (!scores || !klist)) return hipErrorInvalidValue;
#define S2(NB_, DT_, WQ_) return launch_stage2_c<NB_, DT_, WQ_>(x, nb, d, f, wt, scores, k_ff, mask, scores_copy, ypart, ystride, nwg, sel_rule, br, act, klist, klist_mode, st)
#define S2NB(DT_, WQ_)                   \
    switch (stage2_nb_t(nb)) {           \
        case 1: S2(1, DT_, WQ_);         \
        case 2: S2(2, DT_, WQ_);         \
        case 4: S2(4, DT_, WQ_);         \
        default: S2(8, DT_, WQ_);        \
    }
    if (wt.wq == 4) {
        if (dtype == kBF16) { S2NB(kBF16, 4) }
        S2NB(kF16, 4)
    }
    if (dtype == kBF16) { S2NB(kBF16, 16) }
    S2NB(kF16, 16)
#undef S2NB
#undef S2
}

template <int DT, int C, int RT>
static hipError_t launch_stage2m_t(const void *x, int nb, int d, int f, const Stage2Weights &wt,
                                   const float *scores, int k_ff, uint8_t *mask,
                                   float *scores_copy, float *sbuf, int nwg, Select sel_rule,
                                   ScoreBracket br, int act, int32_t *klist, hipStream_t st) {
    const size_t lds = stage2_mfma_lds_bytes();
    hipError_t e = allow_lds(stage2_mfma_kernel<DT, C, RT>, lds);
    if (e != hipSuccess) return e;
    stage2_mfma_kernel<DT, C, RT><<<nwg, kBlock, lds, st>>>(
        static_cast<const uint16_t *>(x), nb, d, f, wt, scores, k_ff, mask, scores_copy, sbuf,
        sel_rule, br, act, klist);
    return hipGetLastError();
}

template <int DT, int RT>
static hipError_t launch_stage2m_c(const void *x, int nb, int d, int f, const Stage2Weights &wt,
                                   const float *scores, int k_ff, uint8_t *mask,
                                   float *scores_copy, float *sbuf, int nwg, Select sel_rule,
                                   ScoreBracket br, int act, int32_t *klist, hipStream_t st) {
#define S2M(C_) launch_stage2m_t<DT, C_, RT>(x, nb, d, f, wt, scores, k_ff, mask, scores_copy, sbuf, nwg, sel_rule, br, act, klist, st)
    if (scores && f <= 4 * kBlock) return S2M(4);
    if (scores && f <= 8 * kBlock) return S2M(8);
    if (scores && f <= 12 * kBlock) return S2M(12);
    if (!scores || f <= 16 * kBlock) return S2M(16);
    if (f <= 28 * kBlock) return S2M(28);
    if (f <= 32 * kBlock) return S2M(32);
    return S2M(64);
#undef S2M
}

hipError_t launch_stage2_mfma(int dtype, const void *x, int nb, int d, int f,
                              const Stage2Weights &wt, const float *scores, int k_ff,
                              uint8_t *mask, float *scores_copy, float *sbuf, int nwg,
                              Select sel_rule, ScoreBracket br, int act, int32_t *klist,
                              hipStream_t st) {
    const int n_ch = scores && !sel_rule.tau_mode ? k_ff : f;   // the kept-list length
    if (nb < 1 || nb > kStage2MfmaMaxRows || !stage2_mfma_ok(d, wt.wq) || nwg < 1 ||
        nwg > kStage2MaxWGs || (long long)n_ch > (long long)kMaxSlice * nwg || !sbuf)
        return hipErrorInvalidValue;
    if (scores && !klist) return hipErrorInvalidValue;   // the down launch reads the kept list
#define S2M(DT_, RT_) return launch_stage2m_c<DT_, RT_>(x, nb, d, f, wt, scores, k_ff, mask, scores_copy, sbuf, nwg, sel_rule, br, act, klist, st)
    const int rt = stage2_row_tiles(nb);
    if (dtype == kBF16) {
        if (rt == 1) S2M(kBF16, 1);
        if (rt == 2) S2M(kBF16, 2);
        S2M(kBF16, 4);
    }
    if (rt == 1) S2M(kF16, 1);
    if (rt == 2) S2M(kF16, 2);
    S2M(kF16, 4);
#undef S2M
}

template <int DT, int RT>
static hipError_t launch_stage2d_t(int nb, int d, int f, const void *wd, const float *sbuf,
                                   const int32_t *klist, int n_max, float *ypart, int ystride,
                                   hipStream_t st) {
    const int groups = stage2_down_groups_mfma(d);
    const size_t lds = stage2_down_lds_bytes(DT, RT, n_max, groups);
    const hipError_t e = allow_lds(stage2_down_kernel<DT, RT>, lds);
    if (e != hipSuccess) return e;
    const dim3 grid((d + kDownCols - 1) / kDownCols, groups);
    stage2_down_kernel<DT, RT><<<grid, kBlock, lds, st>>>(
        nb, d, f, static_cast<const uint16_t *>(wd), sbuf, klist, ypart, ystride);
    return hipGetLastError();
}

hipError_t launch_stage2_down(int dtype, int nb, int d, int f, const void *wd, const float *sbuf,
                              const int32_t *klist, int n_max, float *ypart, int ystride,
                              hipStream_t st) {
    if (nb < 1 || nb > kStage2MfmaMaxRows || d % 128 != 0 || n_max < 0 || n_max > f || !sbuf ||
        (!klist && n_max != f))
        return hipErrorInvalidValue;
#define S2D(DT_, RT_) return launch_stage2d_t<DT_, RT_>(nb, d, f, wd, sbuf, klist, n_max, ypart, ystride, st)
    const int rt = stage2_row_tiles(nb);
    if (dtype == kBF16) {
        if (rt == 1) S2D(kBF16, 1);
        if (rt == 2) S2D(kBF16, 2);
        S2D(kBF16, 4);
    }
    if (rt == 1) S2D(kF16, 1);
    if (rt == 2) S2D(kF16, 2);
    S2D(kF16, 4);
#undef S2D
}

hipError_t launch_reduce(int dtype, const float *ypart, int nwg, int nb, int d, void *y,
                         hipStream_t st) {
    dim3 grid((d + kReduceCols - 1) / kReduceCols, nb);
    const int nbt = ypart_rows(nb);
    if (nwg < 1 || nwg > kStage2MaxWGs) return hipErrorInvalidValue;
    uint16_t *yb = static_cast<uint16_t *>(y);
    if (nwg <= kReduceSmall * kReduceGroups) {
        if (dtype == kBF16)
            reduce_kernel<kBF16, kReduceSmall><<<grid, kReduceThreads, 0, st>>>(ypart, nwg, nbt, d, yb);
        else
            reduce_kernel<kF16, kReduceSmall><<<grid, kReduceThreads, 0, st>>>(ypart, nwg, nbt, d, yb);
    } else if (dtype == kBF16) {
        reduce_kernel<kBF16, kReducePerThread><<<grid, kReduceThreads, 0, st>>>(ypart, nwg, nbt, d, yb);
    } else {
        reduce_kernel<kF16, kReducePerThread><<<grid, kReduceThreads, 0, st>>>(ypart, nwg, nbt, d, yb);
    }
    return hipGetLastError();
}

hipError_t launch_add_rmsnorm(int dtype, const void *x, const void *y, int batch, int d, float eps,
                              void *out, hipStream_t st) {
    auto *xp = static_cast<const uint16_t *>(x);
    auto *yp = static_cast<const uint16_t *>(y);
    auto *op = static_cast<uint16_t *>(out);
    if (dtype == kBF16) add_rmsnorm_kernel<kBF16><<<batch, 1024, 0, st>>>(xp, yp, d, eps, op);
    else add_rmsnorm_kernel<kF16><<<batch, 1024, 0, st>>>(xp, yp, d, eps, op);
    return hipGetLastError();
}

}  // namespace prox
