// Stage 1 of the sparse decode step for INT4 proxies and up to four batch rows
// (Sec. 4.1 Stage 1; proxies of Sec. 4.3): the input selection, the proxy GEMV of
// the kept input rows and the channel scores, as proxy.hip states them.  One
// workgroup per column tile of the blob.
//
// Wave-local lists.  Item r of thread t is input r * 1024 + t, so wave w owns C
// blocks of 64 inputs (one quantisation group each).  Once the k-th largest
// magnitude is known, a wave lists and streams the kept rows of its own blocks:
// no position depends on another wave, so the list needs no barrier.  Blocks are
// 1024 inputs apart, so a run of large inputs spreads over the waves.
//
// Rows in flight during the ranking.  HBM would idle while the block ranks its
// keys (~4 us).  Each wave therefore estimates the cut from 128 of its own keys,
// picks inputs that are surely kept (a margin below the kept fraction) and loads
// their codes before the ranking starts; no barrier of it waits for global loads.
// A guess that turns out wrong is multiplied by x = 0.
//
// Trips.  A wave's lane groups (one per row segment: 4 at 64 columns, 2 at 128)
// take a block each per round, or a share of one when fewer are left, and every
// round is padded to its longest lane group, with x = 0.  So all lanes run the
// same trips: quad t of a lane group stands at one place in LDS, and the quad U
// trips ahead is loaded as soon as one is used up, across rounds.
//
// Stream.  A lane reads 4 bytes (8 columns of one matrix) of four kept rows, a
// quad, and makes them the B operands (4 rows of k, the lane's column; Int4Quad) of
// 4 x 4 x 4 MFMAs whose A operand is x of up to four batch rows.  A ninth MFMA with
// B all ones sums x; at the end of a block the bias times that sum comes off and the
// group's scale is applied.  Batch rows meet nowhere before their scores, so their
// ranges may differ at will.
// From the kernel's start to its last workgroup's scores, against v_dot2 per two
// weights and row: 4096 x 12288, one row, 13.8 us (16.8); 8192 x 28672, one row,
// 27.8 (29.1); 4096 x 14336, four rows, 17.4 (20.3 on the 16-row matrix-core
// kernel); 6272 x 13056, four rows, the call 61.5 (70.0).  One batch of loads at a
// time, without the rolling reload, took 15.5, 30.8 and 20.4.  bf16 x scaled into
// fp16, with fp16 codes, is no faster: the call takes 44.0 us either way at 4096 x
// 12288 and 108.8 against 109.0 at 8192 x 28672, and a large row would take the
// others' low bits.
#include "common.hpp"
#include "kernels.hpp"
#include "topk.hpp"

namespace prox {

constexpr int kSmallHistWords = 4096 + 8;

// LDS: the histogram | per wave, row offsets [lane group][trip][4] u32 (C * 64 in
// all: rounds of up to 16 trips) and x [lane group][NB][trip][4]; after the
// stream the cross-wave sums [16][NB][2T] take the space of the lists.
__host__ __device__ constexpr size_t proxy_small_lds_bytes(int NB, int T, int C) {
    const size_t list = (size_t)C * kBlock * (4 + 2 * NB), red = (size_t)kMaxBlockWaves * NB * 2 * T * 4;
    return (size_t)kSmallHistWords * 4 + (list > red ? list : red);
}

template <int NB, int DT, int T, int C>
__global__ __launch_bounds__(kBlock) void proxy_small_kernel(
    const uint16_t *__restrict__ x, int nb, int d, int f, int group, int k_in,
    const uint8_t *__restrict__ blob, uint8_t *__restrict__ in_mask, float *__restrict__ scores,
    Select sel_rule, int act, ScoreBracket br) {
    constexpr int CPL = 8;                  // columns per lane
    constexpr int LPS = 2 * T / CPL;        // lanes per row segment (gate, then up)
    constexpr int NGRP = kWave / LPS;       // lane groups per wave: 4 or 2
    constexpr int U = 6;                    // quads in flight per lane group
    constexpr int MAXT = C * 16 / NGRP;     // trips of a wave, all inputs kept
    static_assert(LPS == 16 || LPS == 32, "lane groups are 16-lane rows or halves");
    const BlobLayout L(d, f, 4, group);
    const int tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    const int tile = stage1_tile<T == 64>(blockIdx.x, gridDim.x);
    const int ng = d / group;
    const int rows = (d + kBlock - 1) / kBlock;   // blocks per wave (the last may be empty)

    __shared__ SelScratch ss;
    __shared__ int eqtab[C][kMaxBlockWaves];
    __shared__ int kept_sh[kMaxBlockWaves];
    __shared__ uint32_t sc_tile[T];
    extern __shared__ __align__(16) unsigned char dsm[];
    uint32_t *hist = reinterpret_cast<uint32_t *>(dsm);
    uint32_t *offs = hist + kSmallHistWords + (size_t)wid * C * kWave;   // this wave's [NGRP][MAXT][4]
    uint16_t *xsh = reinterpret_cast<uint16_t *>(hist + kSmallHistWords + C * kBlock) +
                    (size_t)wid * C * NB * kWave;                        // this wave's [NGRP][NB][MAXT][4]

    // ---- keys: max over the batch of |x_i| as its 15-bit magnitude pattern ----
    // x of the projected rows stays in registers, two inputs per word.
    uint32_t key[C], xw[NB][C / 2];
    {
        const auto rx = buffer_of(x, (uint32_t)(nb * d) * 2);
        auto load_row = [&](int b, uint32_t (&w)[C / 2]) {   // inputs past d: 0
            const int base = b * d;
#pragma unroll
            for (int q = 0; q < C / 2; ++q) {
                uint32_t h[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = (2 * q + e) * kBlock + tid;
                    h[e] = buffer_load16(rx, i < d ? (base + i) * 2 : 0x7FFFFFFF);
                }
                w[q] = h[0] | (h[1] << 16);
            }
        };
#pragma unroll
        for (int b = 0; b < NB; ++b) load_row(min(b, nb - 1), xw[b]);
        for (int i = tid; i < kSmallHistWords / 4; i += kBlock)
            reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < C; ++r) {
            key[r] = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) key[r] = max(key[r], (xw[b][r / 2] >> (16 * (r & 1))) & 0x7FFFu);
        }
    }
    // The threshold rule's kept count, for what follows to be that of a top-k call
    // with this count (the order of the lists, and so the sums' bits).
    auto in_tau = [&](int r) {
        return r * kBlock + tid < d && half_to_float<DT>((uint16_t)key[r]) >= sel_rule.tau;
    };
    if (sel_rule.tau_mode) {
        int n = 0;
#pragma unroll
        for (int r = 0; r < C; ++r) n += __popcll(__ballot(in_tau(r)));
        if (lane == 0) kept_sh[wid] = n;
    }
    __syncthreads();   // the zeroed histogram, the counts
    if (sel_rule.tau_mode) {
        k_in = __builtin_amdgcn_readlane(
            wave_inclusive_scan(lane < kMaxBlockWaves ? kept_sh[lane] : 0), kMaxBlockWaves - 1);
        if (tile == 0 && tid == 0 && sel_rule.count) *sel_rule.count = k_in;
    }

    // ---- this wave's surely kept inputs of its first blocks, loads on their way ----
    // A round starting at block r0 covers nblk blocks, 1 << lp lane groups each: NGRP
    // blocks while there are as many, then two (halves of the lane groups), then one.
    constexpr int LG = NGRP == 4 ? 2 : 1;
    const bool third = NGRP == 4 && rows % 4 == 3;   // a last round of one block follows one of two
    auto round_of = [&](int r0, int &nblk, int &lp) {
        const int rem = rows - r0;
        nblk = rem >= NGRP ? NGRP : rem >= 2 ? 2 : 1;
        lp = nblk == NGRP ? 0 : nblk == 2 ? LG - 1 : LG;
    };
    const int lg = lane / LPS, li = lane % LPS;
    const int mat = li / (LPS / 2), colc = (li % (LPS / 2)) * CPL;
    const uint8_t *tbase = blob + L.codes_offset + (size_t)tile * L.row_bytes;
    const uint32_t rstride = (uint32_t)L.row_stride;
    const uint32_t lane_off = (uint32_t)(mat * (T / 2) + colc / 2);
    const uint16_t *sbase = reinterpret_cast<const uint16_t *>(blob + L.scales_offset) +
                            (size_t)tile * ng * 2 * T + mat * T + colc;
    const uint32_t gmagic = 0xFFFFFFFFu / (uint32_t)group + 1u;   // i / group, exact here
    auto scale_of = [&](int r) {   // this lane's 8 fp16 scales of its block r
        const int i0 = min(r * kBlock + wid * kWave, d - 1);
        return *reinterpret_cast<const uint4 *>(sbase + (size_t)__umulhi((uint32_t)i0, gmagic) * 2 * T);
    };
    int nblk, lp;
    round_of(0, nblk, lp);
    uint4 sc = scale_of(min(lg >> lp, nblk - 1));   // of this lane group's block of the round

    // The wave's estimate of the cut, as a key: of up to 128 keys, `want` lie at or
    // above it.
    uint32_t cut = 0xFFFFu;
    {
        const float frac = (float)k_in / (float)d - 0.06f;   // a 1.4-sigma margin of 128 keys
        const int i1 = wid * kWave;
        const int n = min(max(d - i1, 0), kWave) + min(max(d - kBlock - i1, 0), kWave);
        const int want = (int)(frac * (float)n);
        if (want >= 1) {
            cut = 0;
#pragma unroll
            for (int bit = 14; bit >= 4; --bit) {
                const uint32_t c = cut | (1u << bit);
                const int cnt = __popcll(__ballot(key[0] >= c)) + __popcll(__ballot(key[1] >= c));
                cut = cnt >= want ? c : cut;
            }
            if (cut == 0) cut = 0xFFFFu;   // nothing to go by
        }
    }
    // Place of the pos-th kept input of the round's b-th block, in the offset list.
    auto slot_of = [&](int b, int lp_, int trip0, int pos) {
        const int q = pos >> 2;
        return ((((b << lp_) + (q & ((1 << lp_) - 1))) * MAXT + trip0 + (q >> lp_)) << 2) + (pos & 3);
    };
    uint64_t guess[NGRP];   // per round-0 block: the inputs loaded early, whole quads
    int early = 0;          // lane r: quads loaded early of block r
#pragma unroll
    for (int r = 0; r < NGRP; ++r) {
        guess[r] = 0;
        if (r < nblk && r < C) {
            const uint64_t m = __ballot(key[r] >= cut);
            const int quads = min(__popcll(m) / 4, U << lp);
            const int pos = (int)lanes_below(m);
            const bool in = ((m >> lane) & 1) && pos < 4 * quads;
            guess[r] = __ballot(in);
            if (in) offs[slot_of(r, lp, 0, pos)] = (uint32_t)(r * kBlock + tid) * rstride;
            early = (int)write_lane((uint32_t)early, (uint32_t)quads, r);
        }
    }
    wave_lds_fence();
    uint32_t code[U][4];   // [quad][row]
    const uint4 *olist = reinterpret_cast<const uint4 *>(offs) + lg * MAXT;
    auto load_quad = [&](uint32_t (&w)[4], const uint4 &o) {
        w[0] = *reinterpret_cast<const uint32_t *>(tbase + (o.x + lane_off));
        w[1] = *reinterpret_cast<const uint32_t *>(tbase + (o.y + lane_off));
        w[2] = *reinterpret_cast<const uint32_t *>(tbase + (o.z + lane_off));
        w[3] = *reinterpret_cast<const uint32_t *>(tbase + (o.w + lane_off));
    };
    // Early trips of this lane group: quads (lg mod P) + P t below its block's count.
    const int eq = __shfl(early, lg >> lp);   // 0 past nblk
    const int my_early = (eq - (lg & ((1 << lp) - 1)) + (1 << lp) - 1) >> lp;   // may be <= 0
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint4 o = make_uint4(0, 0, 0, 0);   // none: row 0, read again below
        if (u < my_early) o = olist[u];
        load_quad(code[u], o);
    }

    // ---- the k-th largest key v; of its equals, `need` are in by index ----
    uint32_t v = 0;
    int need = 0, bucket = 0, eq_before = 0;   // lane r: equal keys before this wave's block r
    if (!sel_rule.tau_mode) {
        kth_magnitude<C>(key, d, k_in, hist, ss, v, need, bucket);
        if (need < bucket) {
            uint32_t cnt = 0;
#pragma unroll
            for (int r = 0; r < C; ++r)
                cnt = write_lane(cnt, (uint32_t)__popcll(__ballot(key[r] == v && r * kBlock + tid < d)), r);
            if (lane < C) eqtab[lane][wid] = (int)cnt;
            __syncthreads();
            // Exclusive prefix over entries r * 16 + w: lane l sums C / 4 of them.
            constexpr int E = C / 4;
            int e[E], run = 0;
            const int *tab = &eqtab[0][0];
#pragma unroll
            for (int q = 0; q < E; ++q) {
                e[q] = run;
                run += tab[lane * E + q];
            }
            const int base = wave_inclusive_scan(run) - run;
            // Lane r wants entry 16 r + wid: lane (16 r + wid) / E, element (16 r + wid) % E.
            const int src = lane < C ? (16 * lane + wid) / E : 0;
            int got = 0;
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const int t = __shfl(base + e[q], src);
                got = wid % E == q ? t : got;
            }
            eq_before = got;
        }
    }

    // ---- the lists: early quads first, then the other kept inputs, padded ----
    int cnts = 0;    // lane r: listed inputs of block r
    uint64_t kept[C];
#pragma unroll
    for (int r = 0; r < C; ++r) {
        if (sel_rule.tau_mode) {
            kept[r] = __ballot(in_tau(r));
        } else if (need < bucket) {
            const bool eq1 = key[r] == v && r * kBlock + tid < d;
            const int rank = __builtin_amdgcn_readlane(eq_before, r) + (int)lanes_below(__ballot(eq1));
            kept[r] = __ballot(key[r] > v || (eq1 && rank < need));
        } else {
            kept[r] = __ballot(key[r] >= v && (v != 0 || r * kBlock + tid < d));
        }
        cnts = (int)write_lane((uint32_t)cnts, (uint32_t)__popcll(r < NGRP ? kept[r] | guess[r < NGRP ? r : 0] : kept[r]), r);
    }
    // Running sum of the rounds' trips, wave-uniform; a third-block round comes on top.
    constexpr int NR = (C + NGRP - 1) / NGRP;
    int trip_end[NR], total = 0;
    auto trips_of = [&](int cnt, int lp_) { return (((cnt + 3) >> 2) + (1 << lp_) - 1) >> lp_; };
#pragma unroll
    for (int rr = 0; rr < NR; ++rr) {
        if (rr * NGRP < rows) {
            int nb_, lp_, most = 0;
            round_of(rr * NGRP, nb_, lp_);
#pragma unroll
            for (int b = 0; b < NGRP; ++b)
                if (rr * NGRP + b < C && b < nb_)
                    most = max(most, __builtin_amdgcn_readlane(cnts, rr * NGRP + b));
            total += trips_of(most, lp_);
        }
        trip_end[rr] = total;
    }
    if (third) total += trips_of(__builtin_amdgcn_readlane(cnts, rows - 1), LG);
#pragma unroll
    for (int r = 0; r < C; ++r) {
        const int i = r * kBlock + tid;
        const uint64_t g = r < NGRP ? guess[r < NGRP ? r : 0] : 0;
        const uint64_t rest = kept[r] & ~g;
        const bool is_kept = (kept[r] >> lane) & 1, is_early = (g >> lane) & 1;
        if (is_kept || is_early) {
            int nb_, lp_;
            round_of(r / NGRP * NGRP, nb_, lp_);
            const int pos = is_early ? (int)lanes_below(g) : __popcll(g) + (int)lanes_below(rest);
            int trip0 = r < NGRP ? 0 : trip_end[r < NGRP ? 0 : r / NGRP - 1], b = r % NGRP;
            if (third && r == rows - 1) {
                trip0 = trip_end[r / NGRP];
                lp_ = LG;
                b = 0;
            }
            const int at = slot_of(b, lp_, trip0, pos);
            if (!is_early) offs[at] = (uint32_t)i * rstride;
            // x: [lane group][NB][trip][4]
            const int xat = at + (at >> 2) / MAXT * ((NB - 1) * MAXT * 4);
#pragma unroll
            for (int b = 0; b < NB; ++b)
                xsh[xat + b * MAXT * 4] =
                    is_kept && b < nb ? (uint16_t)(xw[b][r / 2] >> (16 * (r & 1))) : (uint16_t)0;
        }
        if (tile == 0 && in_mask && i < d) in_mask[i] = is_kept ? 1 : 0;
    }
    // Pads up to the round's trips: row 0, x = 0.
    auto pad_round = [&](int r0, int t0, int t1) {
        int nb_, lp_;
        round_of(r0, nb_, lp_);
        const int n4 = (t1 - t0) * 4;
        for (int e0 = 0; e0 < n4 * NGRP; e0 += kWave) {   // every lane active for the shuffle
            const int e = e0 + lane;
            const int g = (int)((uint32_t)e / (uint32_t)n4), k = e - g * n4;   // lane group, entry of its round
            const int pos = ((((k >> 2) << lp_) + (g & ((1 << lp_) - 1))) << 2) + (k & 3);
            const int blk = g >> lp_;
            const int cnt = __shfl(cnts, min(r0 + blk, C - 1));
            if (g < NGRP && (blk >= nb_ || pos >= cnt)) {
                offs[(g * MAXT + t0) * 4 + k] = 0;
#pragma unroll
                for (int b = 0; b < NB; ++b) xsh[((g * NB + b) * MAXT + t0) * 4 + k] = 0;
            }
        }
    };
#pragma unroll
    for (int rr = 0; rr < NR; ++rr)
        if (rr * NGRP < rows) pad_round(rr * NGRP, rr == 0 ? 0 : trip_end[rr == 0 ? 0 : rr - 1], trip_end[rr]);
    if (third) pad_round(rows - 1, trip_end[NR - 1], total);
    wave_lds_fence();

    // ---- stream ----
    float tot[NB][CPL];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < CPL; ++e) tot[b][e] = 0.0f;
    const uint2 ones = make_uint2(Int4Magic<DT>::one, Int4Magic<DT>::one);
    const Int4Quad<DT> quad;
    const uint2 *xlist = reinterpret_cast<const uint2 *>(xsh) + (lg * NB + (NB == 1 ? 0 : lane % NB)) * MAXT;
    v4f acc[CPL], xacc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < CPL; ++e) acc[e] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u >= my_early && u < total) load_quad(code[u], olist[u]);
    int r_cur = 0, end = trip_end[0];   // the current round ends before trip `end`
    auto flush = [&]() {
        const uint32_t sw[4] = {sc.x, sc.y, sc.z, sc.w};
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            const float s = f16_bits_to_float((e & 1) ? (sw[e >> 1] >> 16) : (sw[e >> 1] & 0xFFFFu));
#pragma unroll
            for (int b = 0; b < NB; ++b) tot[b][e] = fmaf(s, acc[e][b] - Int4Quad<DT>::bias * xacc[b], tot[b][e]);
            acc[e] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
        xacc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        r_cur += third && rows - r_cur == 3 ? 2 : NGRP;
        if (r_cur < rows) {
            int nb_, lp_;
            round_of(r_cur, nb_, lp_);
            sc = scale_of(r_cur + min(lg >> lp_, nb_ - 1));
            end = total;   // a third-block round ends the stream
#pragma unroll
            for (int q = 0; q < NR; ++q) end = q * NGRP == r_cur ? trip_end[q] : end;
        }
    };
    for (int t0 = 0; t0 < total; t0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u;   // wave-uniform
            if (t >= total) break;
            while (t >= end) flush();   // a round may be empty
            const uint2 xq = xlist[t];
            const uint4 o = olist[min(t + U, total - 1)];
            xacc = mfma4<DT>(xq, ones, xacc);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint2 op[4];
                quad.columns(code[u], h, op);
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[4 * h + c] = mfma4<DT>(xq, op[c], acc[4 * h + c]);
            }
            // The quad U trips on (past the end: the last one again, unused).
            load_quad(code[u], o);
        }
    }
    flush();

    // ---- lane groups, then waves, in a fixed order ----
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            float t = tot[b][e];
            if constexpr (LPS == 16) t = add_swap16(t);
            tot[b][e] = add_swap32(t);
        }
    __syncthreads();   // every wave is done with its list
    float *red = reinterpret_cast<float *>(hist + kSmallHistWords);   // [16][NB][2T]
    if (lane < LPS) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<float4 *>(red + (wid * NB + b) * 2 * T + mat * T + colc + 4 * h) =
                    make_float4(tot[b][4 * h], tot[b][4 * h + 1], tot[b][4 * h + 2], tot[b][4 * h + 3]);
    }
    __syncthreads();
    if (tid < T) {
        const int j = tile * T + tid;
        float best = 0.0f;
        for (int b = 0; b < nb; ++b) {
            float gu[2];
#pragma unroll
            for (int m2 = 0; m2 < 2; ++m2) {
                float s8[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    s8[q] = red[((2 * q) * NB + b) * 2 * T + m2 * T + tid] +
                            red[((2 * q + 1) * NB + b) * 2 * T + m2 * T + tid];
                gu[m2] = ((s8[0] + s8[1]) + (s8[2] + s8[3])) + ((s8[4] + s8[5]) + (s8[6] + s8[7]));
            }
            best = fmaxf(best, fabsf(gate_act(gu[0], act) * gu[1]));
        }
        if (j < f) scores[j] = best;
        sc_tile[tid] = __float_as_uint(best);
    }
    if (br.stats && (tile + 1) * T <= f) {
        __syncthreads();
        tile_order_stats<T>(sc_tile, br.r1, br.r2, br.stats + 2 * tile);
    }
}

template <int NB, int DT, int T, int C>
static hipError_t launch_small_t(const void *x, int nb, int d, int f,
                                 int group, int k_in, const void *blob, uint8_t *in_mask,
                                 float *scores, Select sel, int act, ScoreBracket br,
                                 hipStream_t s) {
    const BlobLayout L(d, f, 4, group);
    constexpr size_t lds = proxy_small_lds_bytes(NB, T, C);
    static_assert(lds <= 152 * 1024, "the static tables take the rest");
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void *>(proxy_small_kernel<NB, DT, T, C>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    proxy_small_kernel<NB, DT, T, C><<<L.n_tiles, kBlock, lds, s>>>(
        static_cast<const uint16_t *>(x), nb, d, f, group, k_in,
        static_cast<const uint8_t *>(blob), in_mask, scores, sel, act, br);
    return hipGetLastError();
}

// C = blocks per wave: 4 up to d = 4096, 8 up to 8192, else 16 (one batch row).
template <int DT, int T>
static hipError_t launch_small_c(const void *x, int nb, int d, int f,
                                 int group, int k_in, const void *blob, uint8_t *in_mask,
                                 float *scores, Select sel, int act, ScoreBracket br,
                                 hipStream_t s) {
#define SM(NB_, C_) return launch_small_t<NB_, DT, T, C_>(x, nb, d, f, group, k_in, blob, in_mask, scores, sel, act, br, s)
    if (d <= 4 * kBlock) {
        if (nb == 1) SM(1, 4);
        if (nb == 2) SM(2, 4);
        SM(4, 4);
    }
    if (d <= 8 * kBlock) {
        if (nb == 1) SM(1, 8);
        if (nb == 2) SM(2, 8);
        SM(4, 8);
    }
    SM(1, 16);
#undef SM
}

hipError_t launch_proxy_small(int dtype, const void *x, int nb, int d,
                              int f, int group, int k_in, const void *blob, uint8_t *in_mask,
                              float *scores, Select sel, int act, ScoreBracket br,
                              hipStream_t s) {
    if (nb < 1 || nb > proxy_max_nb(d)) return hipErrorInvalidValue;
#define SM(DT_, T_) launch_small_c<DT_, T_>(x, nb, d, f, group, k_in, blob, in_mask, scores, sel, act, br, s)
    if (proxy_tile(f) == 128) return dtype == kBF16 ? SM(kBF16, 128) : SM(kF16, 128);
    return dtype == kBF16 ? SM(kBF16, 64) : SM(kF16, 64);
#undef SM
}

}  // namespace prox
