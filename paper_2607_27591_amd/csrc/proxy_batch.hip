// Stage 1 of the sparse decode step for INT4 proxies and more than 16 batch rows
// (more than four above d_model 4096, more than one above 8192): three launches that
// select once and read the codes once for up to 64 rows.
//
//  keys    max over the batch of |x_i|.
//  gather  the input selection, once: every workgroup ranks the keys and lists the
//          kept rows per quantisation group, padded to blocks of 16, and gathers its
//          share of x (16 rows, a run of blocks) into the operand order of the next
//          launch.
//  stream  one workgroup per column tile.  A wave takes a 64-byte window of the row
//          segment (T = 64: both matrices; T = 128: one), one tile of 16 batch rows
//          and a run of blocks.  A lane reads 4 bytes (8 columns) of four kept rows
//          as B operands (Int4Quad) of 16 x 16 x 16 MFMAs, x (from L2, in operand
//          order) the A operand, as in proxy_small_kernel but with 16 batch rows per
//          tile.
// The results meet in LDS in wave order.  At 4096 x 14336 and 64 rows keys, gather
// and stream take 3, 8 and 34 us (the stream issues the dequantisation once per row
// tile and window), against 4 x 27 us in launches of 16 rows, each listing again;
// the call 110 us, from 178 (108 with x scaled into fp16, which takes 32 instructions
// to unpack a quad where bf16 takes 36, but ties the rows' ranges together).
#include "common.hpp"
#include "kernels.hpp"
#include "topk.hpp"

namespace prox {

// 128 inputs per workgroup, four groups of threads over the batch rows.
__global__ __launch_bounds__(256) void proxy_keys_kernel(const uint16_t *__restrict__ x, int B, int d,
                                                         uint32_t *__restrict__ keys) {
    __shared__ uint32_t part[4][kWave][2];
    const int l = threadIdx.x % kWave, g = threadIdx.x / kWave;
    const auto rx = buffer_of(x, (uint32_t)(B * d) * 2);   // rows past B read 0
    const int off = (blockIdx.x * 128 + 2 * l) * 2;
    uint32_t v[16], lo = 0, hi = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = buffer_load32(rx, off + (g + 4 * q) * d * 2);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        lo = max(lo, v[q] & 0x7FFFu);
        hi = max(hi, (v[q] >> 16) & 0x7FFFu);
    }
    part[g][l][0] = lo;
    part[g][l][1] = hi;
    __syncthreads();
    if (g < 2) {
        const uint32_t m = max(max(part[0][l][g], part[1][l][g]), max(part[2][l][g], part[3][l][g]));
        keys[blockIdx.x * 128 + 2 * l + g] = m;
    }
}

template <int DT, int C>
__global__ __launch_bounds__(kBlock) void proxy_gather_kernel(
    const uint16_t *__restrict__ x, int B, int d, int group, int k_in, int rt_n,
    uint8_t *__restrict__ in_mask, Select sel_rule, unsigned char *__restrict__ scratch) {
    __shared__ SelScratch ss;
    __shared__ TopKOrder<C> ord;
    __shared__ int gsel0[kMaxDModel / 128 + 1];   // kept rows before each group
    __shared__ int gstart[kMaxDModel / 128 + 1];  // padded list position of each group
    extern __shared__ __align__(16) unsigned char dsm[];
    uint16_t *rows_sh = reinterpret_cast<uint16_t *>(dsm);   // bit 15: a pad
    const BatchScratch L(d, group, rt_n);
    const uint32_t *keys = reinterpret_cast<const uint32_t *>(scratch + L.keys);
    const int tid = threadIdx.x, wid = wave_id(), lane = lane_id();
    const int ng = d / group;
    uint32_t key[C];
    const auto rk = buffer_of(keys, (uint32_t)d * 4);   // past d: 0
#pragma unroll
    for (int r = 0; r < C; ++r) key[r] = buffer_load32(rk, (r * kBlock + tid) * 4);
    if (sel_rule.tau_mode) {
        uint64_t sel = 0;
#pragma unroll
        for (int r = 0; r < C; ++r)
            sel |= (uint64_t)(r * kBlock + tid < d && half_to_float<DT>((uint16_t)key[r]) >= sel_rule.tau) << r;
        topk_order<kBlock, C>(sel, ord);
    } else {
        topk_select_u15<kBlock, C>(key, d, k_in, reinterpret_cast<uint32_t *>(dsm), ss, ord);
    }
    for (int g = tid; g <= ng; g += kBlock) gsel0[g] = topk_selected_before<kBlock, C>(ord, g * group);
    __syncthreads();
    if (wid == 0) {
        int carry = 0;
        for (int g0 = 0; g0 <= ng; g0 += kWave) {
            const int g = g0 + lane;
            const int cnt = g < ng ? gsel0[g + 1] - gsel0[g] : 0;
            const int padded = (cnt + kBatchBlock - 1) / kBatchBlock * kBatchBlock;
            const int incl = wave_inclusive_scan(padded);
            if (g <= ng) gstart[g] = carry + incl - padded;
            carry += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
    }
    __syncthreads();
    // Kept rows at their positions; pads repeat the group's first input.
    const uint32_t gmagic = 0xFFFFFFFFu / (uint32_t)group + 1u;
#pragma unroll
    for (int r = 0; r < C; ++r) {
        const uint64_t bs = ord.sel[r][wid];
        const int g = (int)__umulhi((uint32_t)min(r * kBlock + wid * kWave, d - 1), gmagic);
        const bool s = (bs >> lane) & 1;   // inputs past d are never kept
        if (s) rows_sh[gstart[g] - gsel0[g] + ord.off[r * kMaxBlockWaves + wid] + (int)lanes_below(bs)] =
                   (uint16_t)(r * kBlock + tid);
        if (blockIdx.x == 0 && blockIdx.y == 0 && in_mask && r * kBlock + tid < d)
            in_mask[r * kBlock + tid] = s ? 1 : 0;
    }
    for (int it = tid; it < ng * kBatchBlock; it += kBlock) {
        const int g = it / kBatchBlock, p = gstart[g] + gsel0[g + 1] - gsel0[g] + it % kBatchBlock;
        if (p < gstart[g + 1]) rows_sh[p] = (uint16_t)(0x8000 | (g * group));
    }
    __syncthreads();
    const int n_pos = gstart[ng], nkb = n_pos / kBatchBlock;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        uint16_t *rows = reinterpret_cast<uint16_t *>(scratch + L.rows);
        int *groups = reinterpret_cast<int *>(scratch + L.groups);
        for (int p = tid; p < n_pos; p += kBlock) rows[p] = rows_sh[p] & 0x7FFFu;
        for (int kb = tid; kb < nkb; kb += kBlock)
            groups[kb] = (int)__umulhi((uint32_t)(rows_sh[kb * kBatchBlock] & 0x7FFFu), gmagic);
        if (tid == 0) {
            *reinterpret_cast<int *>(scratch + L.head) = nkb;
            if (sel_rule.tau_mode && sel_rule.count) *sel_rule.count = gsel0[ng];
        }
    }
    // This workgroup's blocks and row tile: thread = (batch row, quad of positions).
    const int rt = blockIdx.y;
    const int kb0 = (int)(blockIdx.x * nkb / gridDim.x), kb1 = (int)((blockIdx.x + 1) * nkb / gridDim.x);
    uint2 *xk = reinterpret_cast<uint2 *>(scratch + L.x);
    for (int e = tid; e < (kb1 - kb0) * kWave; e += kBlock) {
        const int kb = kb0 + e / kWave, lk = e % kWave;   // the operand's lane: row lk % 16, rows 4 (lk / 16) ..
        const int b = rt * 16 + lk % 16;
        const uint2 ids = *reinterpret_cast<const uint2 *>(rows_sh + kb * kBatchBlock + (lk / 16) * 4);
        const uint32_t id[4] = {ids.x & 0xFFFFu, ids.x >> 16, ids.y & 0xFFFFu, ids.y >> 16};
        uint16_t h[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) h[q] = x[(size_t)min(b, B - 1) * d + (id[q] & 0x7FFFu)];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((id[q] & 0x8000u) || b >= B) h[q] = 0;
        xk[((size_t)kb * rt_n + rt) * kWave + lk] =
            make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
    }
}

template <int DT, int T, int RT>
__global__ __launch_bounds__(kBlock) void proxy_stream_kernel(
    const unsigned char *__restrict__ scratch, int nb, int d, int f, int group,
    const uint8_t *__restrict__ blob, float *__restrict__ scores, int act, ScoreBracket br) {
    constexpr int WH = T / 64;                              // 64-byte windows of a segment
    constexpr int KS = kMaxBlockWaves / (WH * RT);          // waves splitting the blocks
    constexpr int CPL = 8, U = 4;                           // columns per lane, blocks in flight
    static_assert(KS >= 2, "waves per window and row tile");
    const BlobLayout L(d, f, 4, group);
    const BatchScratch S(d, group, RT);
    const int tid = threadIdx.x, lane = lane_id(), wid = wave_id();
    const int tile = stage1_tile<T == 64>(blockIdx.x, gridDim.x);
    const int ng = d / group;
    __shared__ uint32_t sc_tile[T];
    extern __shared__ __align__(16) unsigned char dsm[];
    uint32_t *offs = reinterpret_cast<uint32_t *>(dsm);   // row offsets of the list, then the sums
    const int nkb = *reinterpret_cast<const int *>(scratch + S.head);
    const uint16_t *rows = reinterpret_cast<const uint16_t *>(scratch + S.rows);
    const int *groups = reinterpret_cast<const int *>(scratch + S.groups);
    const uint32_t rstride = (uint32_t)L.row_stride;
    for (int p = tid; p < nkb * kBatchBlock; p += kBlock) offs[p] = (uint32_t)rows[p] * rstride;
    __syncthreads();

    const int wh = wid % WH, rt = wid / WH % RT, ks = wid / (WH * RT);
    const int kb0 = ks * nkb / KS, kb1 = (ks + 1) * nkb / KS;
    const int ln = lane % 16, lg = lane / 16;
    const uint8_t *tbase = blob + L.codes_offset + (size_t)tile * L.row_bytes;
    const uint32_t lane_off = (uint32_t)(wh * 64 + ln * 4);
    // The lane's 8 columns: of the segment's 2 T, gate first.
    const uint16_t *sbase = reinterpret_cast<const uint16_t *>(blob + L.scales_offset) +
                            (size_t)tile * ng * 2 * T + wh * 128 + ln * CPL;
    const uint2 *xk = reinterpret_cast<const uint2 *>(scratch + S.x) + (size_t)rt * kWave + lane;

    v4f acc[CPL], tot[CPL], xacc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < CPL; ++e) acc[e] = tot[e] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const uint2 ones = make_uint2(Int4Magic<DT>::one, Int4Magic<DT>::one);
    const Int4Quad<DT> quad;
    if (kb0 < kb1) {
        uint32_t code[U][4];
        uint2 xq[U];
        auto load = [&](int u, int kb) {
            const uint4 o = *reinterpret_cast<const uint4 *>(offs + kb * kBatchBlock + 4 * lg);
            code[u][0] = *reinterpret_cast<const uint32_t *>(tbase + (o.x + lane_off));
            code[u][1] = *reinterpret_cast<const uint32_t *>(tbase + (o.y + lane_off));
            code[u][2] = *reinterpret_cast<const uint32_t *>(tbase + (o.z + lane_off));
            code[u][3] = *reinterpret_cast<const uint32_t *>(tbase + (o.w + lane_off));
            xq[u] = xk[(size_t)kb * RT * kWave];
        };
#pragma unroll
        for (int u = 0; u < U; ++u) load(u, min(kb0 + u, kb1 - 1));
        int gcur = groups[kb0];
        uint4 sc = *reinterpret_cast<const uint4 *>(sbase + (size_t)gcur * 2 * T);
        auto flush = [&]() {
            const uint32_t sw[4] = {sc.x, sc.y, sc.z, sc.w};
#pragma unroll
            for (int e = 0; e < CPL; ++e) {
                const float s = f16_bits_to_float((e & 1) ? (sw[e >> 1] >> 16) : (sw[e >> 1] & 0xFFFFu));
#pragma unroll
                for (int j = 0; j < 4; ++j) tot[e][j] = fmaf(s, acc[e][j] - Int4Quad<DT>::bias * xacc[j], tot[e][j]);
                acc[e] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            }
            xacc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        };
        for (int k0 = kb0; k0 < kb1; k0 += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kb = k0 + u;   // wave-uniform
                if (kb >= kb1) break;
                const int g = groups[kb];
                if (g != gcur) {
                    flush();
                    gcur = g;
                    sc = *reinterpret_cast<const uint4 *>(sbase + (size_t)gcur * 2 * T);
                }
                xacc = mfma16<DT>(xq[u], ones, xacc);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint2 op[4];
                    quad.columns(code[u], h, op);
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[4 * h + c] = mfma16<DT>(xq[u], op[c], acc[4 * h + c]);
                }
                load(u, min(kb + U, kb1 - 1));   // past the end: the last block again, unused
            }
        }
        flush();
    }
    __syncthreads();   // the list is used up
    float4 *red = reinterpret_cast<float4 *>(dsm);   // [wave][column][lane]
#pragma unroll
    for (int e = 0; e < CPL; ++e)
        red[(wid * CPL + e) * kWave + lane] =
            make_float4(tot[e][0], tot[e][1], tot[e][2], tot[e][3]);
    __syncthreads();
    // Every (row, column): the sums of the KS waves of gate and up in order, |act(g~)
    // u~|, the max over the row tiles, then over the 16 lanes that hold one column.
    const float *rf = reinterpret_cast<const float *>(dsm);
    const int b16 = tid % 16;
#pragma unroll
    for (int q = 0; q < T / 64; ++q) {
        const int col = tid / 16 + q * 64;
        // Gate and up column in the segment: window, lane and column of the lane.
        auto at = [&](int c2, int r, int w2) {   // of wave w2 of row tile r
            const int win = c2 / 128, cl = c2 % 128;
            const int wave = (w2 * RT + r) * WH + win;
            return ((wave * CPL + cl % CPL) * kWave + (b16 / 4) * 16 + cl / CPL) * 4 + b16 % 4;
        };
        float v = 0.0f;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            float gs = 0.0f, us = 0.0f;
#pragma unroll
            for (int w2 = 0; w2 < KS; ++w2) {
                gs += rf[at(col, r, w2)];
                us += rf[at(T + col, r, w2)];
            }
            const float s = fabsf(gate_act(gs, act) * us);
            v = fmaxf(v, r * 16 + b16 < nb ? s : 0.0f);
        }
        v = fmaxf(v, dpp_move<kDppXor1>(v));
        v = fmaxf(v, dpp_move<kDppXor2>(v));
        v = fmaxf(v, dpp_move<kDppRor4>(v));
        v = fmaxf(v, dpp_move<kDppRor8>(v));
        const int j = tile * T + col;
        if (b16 == 0) {
            if (j < f) scores[j] = v;
            sc_tile[col] = __float_as_uint(v);
        }
    }
    if (br.stats && (tile + 1) * T <= f) {
        __syncthreads();
        tile_order_stats<T>(sc_tile, br.r1, br.r2, br.stats + 2 * tile);
    }
}

template <int DT, int C>
static hipError_t launch_gather_t(const void *x, int B, int d, int group, int k_in, int rt,
                                  uint8_t *in_mask, Select sel, void *scratch, hipStream_t s) {
    const size_t list = (size_t)batch_list_cap(d, group) * 2;
    const size_t lds = list > kSelHistU16Bytes ? list : kSelHistU16Bytes;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(proxy_gather_kernel<DT, C>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // 64 workgroups in all: a few blocks of 16 x 16 values each.
    proxy_gather_kernel<DT, C><<<dim3(64 / rt, rt), kBlock, lds, s>>>(
        static_cast<const uint16_t *>(x), B, d, group, k_in, rt, in_mask, sel,
        static_cast<unsigned char *>(scratch));
    return hipGetLastError();
}

template <int DT, int T, int RT>
static hipError_t launch_stream_t(const void *scratch, int nb, int d, int f, int group,
                                  const void *blob, float *scores, int act, ScoreBracket br,
                                  hipStream_t s) {
    const size_t list = (size_t)batch_list_cap(d, group) * 4, red = (size_t)kBlock * 32 * 4;
    const size_t lds = list > red ? list : red;   // 128 KiB
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(proxy_stream_kernel<DT, T, RT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const BlobLayout L(d, f, 4, group);
    proxy_stream_kernel<DT, T, RT><<<L.n_tiles, kBlock, lds, s>>>(
        static_cast<const unsigned char *>(scratch), nb, d, f, group, static_cast<const uint8_t *>(blob),
        scores, act, br);
    return hipGetLastError();
}

hipError_t launch_proxy_batch(int dtype, const void *x, int batch, int d, int f, int group, int k_in,
                              const void *blob, uint8_t *in_mask, float *scores, Select sel, int act,
                              ScoreBracket br, void *scratch, size_t scratch_bytes, hipStream_t s) {
    if (batch < 1 || batch > 64 || d % 128 != 0) return hipErrorInvalidValue;
    const int rt = stage2_row_tiles(batch);
    const BatchScratch L(d, group, rt);
    if (L.total > scratch_bytes) return hipErrorInvalidValue;
    proxy_keys_kernel<<<d / 128, 256, 0, s>>>(static_cast<const uint16_t *>(x), batch, d,
                                              reinterpret_cast<uint32_t *>(static_cast<char *>(scratch) + L.keys));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
#define GA(DT_, C_) launch_gather_t<DT_, C_>(x, batch, d, group, k_in, rt, in_mask, sel, scratch, s)
    if (d <= 4 * kBlock) e = dtype == kBF16 ? GA(kBF16, 4) : GA(kF16, 4);
    else if (d <= 8 * kBlock) e = dtype == kBF16 ? GA(kBF16, 8) : GA(kF16, 8);
    else e = dtype == kBF16 ? GA(kBF16, 16) : GA(kF16, 16);
#undef GA
    if (e != hipSuccess) return e;
#define ST(T_, RT_) return dtype == kBF16 ? launch_stream_t<kBF16, T_, RT_>(scratch, batch, d, f, group, blob, scores, act, br, s) \
                                          : launch_stream_t<kF16, T_, RT_>(scratch, batch, d, f, group, blob, scores, act, br, s)
    if (proxy_tile(f) == 128) {
        if (rt == 1) ST(128, 1);
        if (rt == 2) ST(128, 2);
        ST(128, 4);
    }
    if (rt == 1) ST(64, 1);
    if (rt == 2) ST(64, 2);
    ST(64, 4);
#undef ST
}

}  // namespace prox
