// Proxy packing (Sec. 4.3): symmetric per-(channel, group) quantisation of
// W_gate and W_up into the tiled, input-major proxy blob, and the inverse
// view used for inspection.
#include "common.hpp"
#include "kernels.hpp"

namespace prox {

// IEEE binary16 round-to-nearest-even of a binary64 value, from the bit
// fields of the double.
__device__ uint16_t f64_to_f16_rne(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint16_t sign = (uint16_t)((u >> 48) & 0x8000u);
    const uint64_t a = u & 0x7FFFFFFFFFFFFFFFull;
    if (a >= 0x7FF0000000000000ull) return sign | (a > 0x7FF0000000000000ull ? 0x7E00 : 0x7C00);
    if (a < 0x0010000000000000ull) return sign;   // below 2^-1022: rounds to zero
    const int e = (int)(a >> 52) - 1023;
    if (e > 15) return sign | 0x7C00;
    const uint64_t m = (a & 0x000FFFFFFFFFFFFFull) | 0x0010000000000000ull;  // 53 bits
    // Normal results keep 11 significant bits; subnormal ones count 2^-24 units.
    const int shift = e >= -14 ? 42 : 28 - e;
    if (shift > 62) return sign;
    uint64_t keep = m >> shift;
    const uint64_t rem = m & ((1ull << shift) - 1);
    const uint64_t half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (keep & 1))) ++keep;
    if (e >= -14) {
        int E = e;
        if (keep == 2048) { keep = 1024; ++E; }
        if (E > 15) return sign | 0x7C00;
        return sign | (uint16_t)((E + 15) << 10) | (uint16_t)(keep - 1024);
    }
    return sign | (uint16_t)keep;   // 1024 encodes the smallest normal
}

template <int DT>
__device__ __forceinline__ double w_to_f64(uint16_t h) { return (double)half_to_float<DT>(h); }

// Symmetric quantisation of one group: sigma = fp16_rne(amax / qmax) from the
// largest magnitude pattern (15 bits, ordered like the magnitudes).
struct GroupScale {
    float sigma, inv;   // sigma and 1 / sigma (0 when sigma is 0)
    uint16_t bits;
};
template <int DT>
__device__ __forceinline__ GroupScale group_scale(uint32_t amax_bits, int qmax) {
    GroupScale s;
    s.bits = f64_to_f16_rne(w_to_f64<DT>((uint16_t)amax_bits) / (double)qmax);
    s.sigma = f16_bits_to_float(s.bits);
    s.inv = s.sigma != 0.0f ? 1.0f / s.sigma : 0.0f;
    return s;
}

// clamp(round_half_even(w / sigma), -qmax, qmax), exactly as the fp64 quotient
// rounds.  w inv is within 2^-22 |w / sigma| of it, under 1e-4 for every
// quotient that occurs (at most 1.5 * 127, where sigma is subnormal), so the two
// round alike unless w inv lies within 1e-4 of a half: those (about 1 in 5000)
// take the fp64 division.
template <int DT>
__device__ __forceinline__ int quantise(uint32_t wbits, float sigma, float inv, float qmax) {
    const float w = half_to_float<DT>((uint16_t)wbits);
    const float r = w * inv;
    float n = rintf(r);
    if (fabsf(r - n) > 0.4999f) n = (float)rint((double)w / (double)sigma);
    return (int)fminf(fmaxf(n, -qmax), qmax);
}

// The largest finite-ordered magnitude pattern of 8 packed 16-bit floats (NaN
// patterns count as 0).
template <int DT>
__device__ __forceinline__ uint32_t abs_max8(const uint4 &v) {
    constexpr uint32_t inf = DT == kBF16 ? 0x7F80u : 0x7C00u;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t lo = w[q] & 0x7FFFu, hi = (w[q] >> 16) & 0x7FFFu;
        m = max(m, lo <= inf ? lo : 0u);
        m = max(m, hi <= inf ? hi : 0u);
    }
    return m;
}

// Maximum over each 16-lane row, in every lane of the row.
__device__ __forceinline__ uint32_t row16_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppXor1, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppXor2, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppRor4, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppRor8, 0xF, 0xF, false));
    return v;
}

__device__ __forceinline__ uint32_t half_of(const uint4 &v, int e) {   // e a constant
    const uint32_t w = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
    return (e & 1) ? w >> 16 : w & 0xFFFFu;
}

// Packing is a transposition: weights are channel-major, codes input-major.  It
// is bound by HBM (16-bit weights read once, codes written once).  A workgroup
// of 4 T threads takes one column tile of both matrices and one group of inputs
// in blocks of 128: 16 lanes read 256 contiguous bytes of a channel row, each
// thread the same 8 inputs of 8 channels (8 loads in flight), so it holds whole
// code words of 8 columns and the transposition goes through LDS in words; the
// blob is written in whole row segments of the tile.  A group of 128 is read
// once; a longer one is read twice (largest magnitude, then codes), the second
// time mostly from the last-level cache.
// 4096 x 12288 bf16 to INT4, group 128: 74 us (3.4 TB/s of the 253 MB moved; a
// large copy reaches 4.8), against 3276 us with a thread per column pair
// walking its two channel rows; 8192 x 28672: 490 us against 15.3 ms.  Held to
// 128 registers it spills and takes 77 us.
constexpr int kPackIn = 128;   // inputs per block
template <int QB>
__host__ __device__ constexpr int pack_pitch(int T) {   // LDS words per input: a segment and a pad
    return 2 * T * QB / 32 + (QB == 4 ? 1 : QB == 8 ? 2 : 4);
}

template <int DT, int QB, int T>
__global__ __launch_bounds__(4 * T) void pack_kernel(const uint16_t *__restrict__ wg,
                                                     const uint16_t *__restrict__ wu, int d, int f,
                                                     int group, uint8_t *__restrict__ blob) {
    constexpr int NT = 4 * T;
    constexpr int PITCH = pack_pitch<QB>(T);
    constexpr float qmax = QB == 4 ? 7.0f : 127.0f;
    extern __shared__ __align__(16) uint32_t codes_sh[];   // [kPackIn][PITCH]
    __shared__ uint32_t amax_sh[2 * T];
    __shared__ float sigma_sh[2 * T], inv_sh[2 * T];
    const BlobLayout L(d, f, QB, group);
    const int ng = d / group;
    const int tile = blockIdx.x, tid = threadIdx.x;
    // Unquantised weights have no group to scan: one block of inputs each.
    const int blocks = QB == 16 ? 1 : group / kPackIn;
    const int i_first = (int)blockIdx.y * blocks * kPackIn;
    const int g = i_first / group;
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
        BlobHeader h{};
        h.magic = kBlobMagic; h.version = kBlobVersion; h.fmt = QB == 4 ? 1u : QB == 8 ? 0u : 2u;
        h.group = (uint32_t)group; h.d_model = (uint32_t)d; h.d_ff = (uint32_t)f;
        h.tile = (uint32_t)L.tile; h.qbits = QB;
        h.codes_offset = L.codes_offset; h.scales_offset = L.scales_offset;
        h.total_bytes = L.total;
        *reinterpret_cast<BlobHeader *>(blob) = h;
    }
    // Thread: matrix mat, channels c0 .. c0 + 7 of the tile, inputs 8 l .. 8 l + 7 of a block.
    const int l = tid % 16, oct = tid / 16;
    const int mat = oct / (T / 8), c0 = (oct % (T / 8)) * 8;
    const uint16_t *w = (mat == 0 ? wg : wu) + (size_t)i_first + 8 * l;
    auto load = [&](int blk, uint4 (&v)[8]) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int j = tile * T + c0 + r;
            v[r] = j < f ? load_stream16(w + (size_t)j * d + blk * kPackIn) : make_uint4(0, 0, 0, 0);
        }
    };
    uint4 v[8];
    uint16_t *scales = reinterpret_cast<uint16_t *>(blob + L.scales_offset) + ((size_t)tile * ng + g) * 2 * T;
    if constexpr (QB == 16) {
        load(0, v);
        if (i_first == 0 && tid < 2 * T) scales[tid] = 0x3C00u;   // fp16 1.0
    } else {
        uint32_t m[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) m[r] = 0;
        for (int blk = 0; blk < blocks; ++blk) {
            load(blk, v);
#pragma unroll
            for (int r = 0; r < 8; ++r) m[r] = max(m[r], abs_max8<DT>(v[r]));
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            m[r] = row16_max(m[r]);
            if (l == r) amax_sh[mat * T + c0 + r] = m[r];
        }
        __syncthreads();
        if (tid < 2 * T) {
            const GroupScale s = group_scale<DT>(amax_sh[tid], (int)qmax);
            sigma_sh[tid] = s.sigma;
            inv_sh[tid] = s.inv;
            scales[tid] = s.bits;
        }
        __syncthreads();
    }
    for (int blk = 0; blk < blocks; ++blk) {
        if (QB != 16 && blocks > 1) load(blk, v);
        uint32_t word[8][QB / 4];   // code words of input e, channels c0 .. c0 + 7
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int q = 0; q < QB / 4; ++q) word[e][q] = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if constexpr (QB == 16) {
#pragma unroll
                for (int e = 0; e < 8; ++e) word[e][r / 2] |= half_of(v[r], e) << (16 * (r & 1));
            } else {
                const float sigma = sigma_sh[mat * T + c0 + r], inv = inv_sh[mat * T + c0 + r];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    int q = quantise<DT>(half_of(v[r], e), sigma, inv, qmax);
                    if (sigma == 0.0f) q = 0;   // a NaN weight too
                    if constexpr (QB == 4) word[e][0] |= (uint32_t)(q + 8) << (4 * r);
                    else word[e][r / 4] |= (uint32_t)(q + 128) << (8 * (r & 3));
                }
            }
        }
        if (blk > 0) __syncthreads();   // the previous block has been read out
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint32_t *dst = codes_sh + (8 * l + e) * PITCH + (mat * T + c0) * QB / 32;
#pragma unroll
            for (int q = 0; q < QB / 4; ++q) dst[q] = word[e][q];
        }
        __syncthreads();
        constexpr int SEG = 2 * T * QB / 128;   // 16-byte vectors per segment
        for (int k = tid; k < kPackIn * SEG; k += NT) {
            const int i = k / SEG, q = k % SEG;
            const uint32_t *src = codes_sh + i * PITCH + q * 4;
            *reinterpret_cast<uint4 *>(blob + L.codes_offset +
                                       (size_t)(i_first + blk * kPackIn + i) * L.row_stride +
                                       (size_t)tile * L.row_bytes + q * 16) =
                make_uint4(src[0], src[1], src[2], src[3]);
        }
    }
}

// Inverse view: one thread per (matrix, channel, group).
template <int QB>
__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t *__restrict__ blob, int d,
                                                     int f, int group, int8_t *cg, uint16_t *sg,
                                                     int8_t *cu, uint16_t *su) {
    const BlobLayout L(d, f, QB, group);
    const int ng = d / group;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= 2LL * f * ng) return;
    const int mat = (int)(gid / ((long long)f * ng));
    const int rem = (int)(gid % ((long long)f * ng));
    const int j = rem / ng, g = rem % ng;
    const int T = L.tile;
    const int tile = j / T, c = j % T;
    const uint16_t *scales = reinterpret_cast<const uint16_t *>(blob + L.scales_offset);
    (mat == 0 ? sg : su)[(size_t)j * ng + g] = scales[(((size_t)tile * ng + g) * 2 + mat) * T + c];
    int8_t *out = (mat == 0 ? cg : cu) + (size_t)j * d;
    for (int ii = 0; ii < group; ++ii) {
        const int i = g * group + ii;
        const uint8_t *seg = blob + L.codes_offset + (size_t)i * L.row_stride + (size_t)tile * L.row_bytes;
        int q;
        if constexpr (QB == 4) {
            const uint8_t byte = seg[mat * (T / 2) + c / 2];
            q = (int)((c & 1) ? (byte >> 4) : (byte & 15)) - 8;
        } else {
            q = (int)seg[mat * T + c] - 128;
        }
        out[i] = (int8_t)q;
    }
}

// INT4 base weights (W4A16), the same symmetric quantiser as the proxy, stored
// channel-major like the weights.  Bound by HBM: 16 lanes take one group (8
// inputs each per 16-byte load), a wave's four rows of lanes neighbouring
// groups, so loads and the 4-byte code stores are contiguous over the wave.  A
// group of 128 stays in registers between its largest magnitude and its codes,
// kW4PerRow groups per row of lanes, whose scales are worked out once, by a lane
// each; a longer group is read twice.
// 4096 x 14336 bf16, group 128: 105 us (4.2 TB/s), against 6.5 ms with a thread
// per group.
constexpr int kW4PerRow = 8;
template <int DT, bool G128>
__global__ __launch_bounds__(256) void pack_w4_kernel(const uint16_t *__restrict__ wg,
                                                      const uint16_t *__restrict__ wu,
                                                      const uint16_t *__restrict__ wd, int d, int f,
                                                      int group, uint8_t *__restrict__ blob) {
    const W4Layout L(d, f, group);
    const int ng = d / group;
    const int m = blockIdx.y;
    const uint16_t *w = m == 0 ? wg : m == 1 ? wu : wd;
    uint8_t *codes = blob + L.codes[m];
    uint16_t *scales = reinterpret_cast<uint16_t *>(blob + L.scales[m]);
    const long long n = (long long)f * ng;   // groups of the matrix, in memory order
    const int lane = lane_id(), l = lane % 16, row = lane / 16;
    const long long wave = (long long)blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    auto codes_of = [&](const uint4 &v, float sigma, float inv) {
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int q = quantise<DT>(half_of(v, e), sigma, inv, 7.0f);
            if (sigma == 0.0f) q = 0;   // a NaN weight too
            word |= (uint32_t)(q + 8) << (4 * e);
        }
        return word;
    };
    if constexpr (G128) {
        const long long g0 = wave * (4 * kW4PerRow) + row;   // groups g0 + 4 k
        uint4 v[kW4PerRow];
#pragma unroll
        for (int k = 0; k < kW4PerRow; ++k)   // past the end: the last group again
            v[k] = load_stream16(w + (size_t)min(g0 + 4 * k, n - 1) * 128 + 8 * l);
        uint32_t mine = 0;   // lane k of a row works out group k's scale
#pragma unroll
        for (int k = 0; k < kW4PerRow; ++k) {
            const uint32_t a = row16_max(abs_max8<DT>(v[k]));
            mine = l == k ? a : mine;
        }
        const GroupScale s = group_scale<DT>(mine, 7);
        if (l < kW4PerRow && g0 + 4 * l < n) scales[g0 + 4 * l] = s.bits;
#pragma unroll
        for (int k = 0; k < kW4PerRow; ++k) {
            const float sigma = __shfl(s.sigma, row * 16 + k), inv = __shfl(s.inv, row * 16 + k);
            const uint32_t word = codes_of(v[k], sigma, inv);
            const long long g = g0 + 4 * k;
            if (g < n) *reinterpret_cast<uint32_t *>(codes + (size_t)g * 64 + 4 * l) = word;
        }
    } else {
        const long long g = wave * 4 + row;
        if (g >= n) return;   // whole rows of lanes: the row maximum stays inside one
        const uint16_t *src = w + (size_t)g * group + 8 * l;
        uint32_t a = 0;
        for (int i = 0; i < group; i += 128) a = max(a, abs_max8<DT>(*reinterpret_cast<const uint4 *>(src + i)));
        const GroupScale s = group_scale<DT>(row16_max(a), 7);
        if (l == 0) scales[g] = s.bits;
        for (int i = 0; i < group; i += 128)
            *reinterpret_cast<uint32_t *>(codes + (size_t)g * (group / 2) + i / 2 + 4 * l) =
                codes_of(*reinterpret_cast<const uint4 *>(src + i), s.sigma, s.inv);
    }
}

// Inverse view of matrix m: codes int8 [f][d] and scales [f][d/group].
__global__ __launch_bounds__(256) void unpack_w4_kernel(const uint8_t *__restrict__ blob, int d,
                                                        int f, int group, int m, int8_t *codes,
                                                        uint16_t *scales) {
    const W4Layout L(d, f, group);
    const int ng = d / group;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (long long)f * ng) return;
    const int j = (int)(gid / ng), g = (int)(gid % ng);
    scales[(size_t)j * ng + g] =
        reinterpret_cast<const uint16_t *>(blob + L.scales[m])[(size_t)j * ng + g];
    const uint8_t *src = blob + L.codes[m] + (size_t)j * (d / 2) + (size_t)g * (group / 2);
    int8_t *out = codes + (size_t)j * d + (size_t)g * group;
    for (int i = 0; i < group; i += 2) {
        const uint8_t byte = src[i / 2];
        out[i] = (int8_t)((int)(byte & 15) - 8);
        out[i + 1] = (int8_t)((int)(byte >> 4) - 8);
    }
}

template <int DT>
static hipError_t launch_pack_w4_t(const uint16_t *wg, const uint16_t *wu, const uint16_t *wd,
                                   int d, int f, int group, uint8_t *blob, hipStream_t s) {
    const long long n = (long long)f * (d / group);
    const long long per = (256 / kWave) * 4 * (group == 128 ? kW4PerRow : 1);   // groups per workgroup
    const dim3 grid((unsigned)((n + per - 1) / per), 3);
    if (group == 128) pack_w4_kernel<DT, true><<<grid, 256, 0, s>>>(wg, wu, wd, d, f, group, blob);
    else pack_w4_kernel<DT, false><<<grid, 256, 0, s>>>(wg, wu, wd, d, f, group, blob);
    return hipGetLastError();
}

hipError_t launch_pack_w4(int dtype, const void *wg, const void *wu, const void *wd, int d, int f,
                          int group, void *blob, hipStream_t s) {
    auto *g = static_cast<const uint16_t *>(wg);
    auto *u = static_cast<const uint16_t *>(wu);
    auto *dn = static_cast<const uint16_t *>(wd);
    auto *b = static_cast<uint8_t *>(blob);
    return dtype == kBF16 ? launch_pack_w4_t<kBF16>(g, u, dn, d, f, group, b, s)
                          : launch_pack_w4_t<kF16>(g, u, dn, d, f, group, b, s);
}

hipError_t launch_unpack_w4(const void *blob, int d, int f, int group, int m, int8_t *codes,
                            uint16_t *scales, hipStream_t s) {
    const long long n = (long long)f * (d / group);
    const int nb = (int)((n + 255) / 256);
    unpack_w4_kernel<<<nb, 256, 0, s>>>(static_cast<const uint8_t *>(blob), d, f, group, m,
                                        codes, scales);
    return hipGetLastError();
}

template <int DT, int QB, int T>
static hipError_t launch_pack_t(const uint16_t *wg, const uint16_t *wu, int d, int f, int group,
                                uint8_t *blob, hipStream_t s) {
    const BlobLayout L(d, f, QB, group);
    const size_t lds = (size_t)kPackIn * pack_pitch<QB>(T) * 4;   // at most 66 KB
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(
            reinterpret_cast<const void *>(pack_kernel<DT, QB, T>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const dim3 grid(L.n_tiles, QB == 16 ? d / kPackIn : d / group);
    pack_kernel<DT, QB, T><<<grid, 4 * T, lds, s>>>(wg, wu, d, f, group, blob);
    return hipGetLastError();
}

hipError_t launch_pack(int dtype, int qbits, const void *wg, const void *wu, int d, int f,
                       int group, void *blob, hipStream_t s) {
    auto *g = static_cast<const uint16_t *>(wg);
    auto *u = static_cast<const uint16_t *>(wu);
    auto *b = static_cast<uint8_t *>(blob);
    const bool wide = proxy_tile(f) == 128;
#define PK(DT_, QB_) (wide ? launch_pack_t<DT_, QB_, 128>(g, u, d, f, group, b, s) \
                           : launch_pack_t<DT_, QB_, 64>(g, u, d, f, group, b, s))
    if (dtype == kBF16) return qbits == 4 ? PK(kBF16, 4) : qbits == 8 ? PK(kBF16, 8) : PK(kBF16, 16);
    return qbits == 4 ? PK(kF16, 4) : qbits == 8 ? PK(kF16, 8) : PK(kF16, 16);
#undef PK
}

hipError_t launch_unpack(int qbits, const void *blob, int d, int f, int group, int8_t *cg,
                         uint16_t *sg, int8_t *cu, uint16_t *su, hipStream_t s) {
    const long long n = 2LL * f * (d / group);
    const int nb = (int)((n + 255) / 256);
    auto *b = static_cast<const uint8_t *>(blob);
    if (qbits == 4) unpack_kernel<4><<<nb, 256, 0, s>>>(b, d, f, group, cg, sg, cu, su);
    else unpack_kernel<8><<<nb, 256, 0, s>>>(b, d, f, group, cg, sg, cu, su);
    return hipGetLastError();
}

}  // namespace prox
