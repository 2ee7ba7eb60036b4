// The data-free delta compressor on the GPU: a dense fp16 delta -> canonical compressed tables.
//
// Paper Section 4.1: step 2 prunes the delta to the 2:4 pattern (two of every four consecutive
// entries are kept, each with a 2-bit position), step 3 stores the kept values as b-bit codes.  The
// paper's Algorithm 1 picks mask and codes with calibration data; this kernel applies the data-free
// rule instead: keep the two entries of largest magnitude (ties: the lower position), and quantise the
// kept values of each row and group of `group` dense columns on an asymmetric uniform grid that
// contains zero, rounding to nearest (half to even), all in fp32:
//     lo = min(0, min v), hi = max(0, max v), s = f16((hi - lo) / (2^b - 1))  (s = 1, z = 0 if that is 0)
//     z = clamp(rint((0 - lo) / s), 0, 2^b - 1),  q = clamp(rint(v / s) + z, 0, 2^b - 1)
// Its output feeds dz_pack_delta.  Off the per-token path, but a variant is registered while others are
// being served, so it should take no longer than its bytes (2 in and 1 + 8 / group out per entry).
//
// What bounds it: vector instructions, before the bytes.  One lane per group of four with a byte store per
// table entry and two IEEE divisions took 26.2 us on 4096 x 4096 and 63.6 us on 11008 x 4096, 1.9
// and 2.1 TB/s.  Here a lane owns 16 columns (two 16-byte loads, two 8-byte stores), and
//   * the two kept entries of a group come from a three-exchange network over the keys
//     (|v| bits << 2 | 3 - position): larger magnitude first, then the lower position; the kept pair is
//     cut out of the group's two dwords with one byte permute;
//   * the range of a quantisation group is reduced as packed fp16 pairs (minimum and maximum of fp16 values
//     are exact) over its 8 or 4 lanes with lane-permuting moves;
//   * v / s is needed only as rint(v / s): one reciprocal per lane and group, then q = v r corrected once by
//     q += (v - q s) r.  v and s have 11-bit significands, so a quotient of magnitude 1/4 or more that is
//     no half-integer is at least 2^-13 away from every half-integer, far more than the error of q (below
//     2^-18 up to the clamp), and one that is a half-integer is representable, so that the corrected q is
//     that number: rint sees the same as after the IEEE division.  An infinite s (a range beyond fp16)
//     makes q a NaN where the division gives 0 or NaN; the clamp turns each of them into code 0.
// Some 240 vector instructions per lane for 16 columns; 11.7 and 24.4 us, 4.3 and 5.6 TB/s.
#include "dz_internal.h"

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
// the tables need no alignment beyond their element's, the delta 8 bytes
typedef uint32_t delta4 __attribute__((ext_vector_type(4), aligned(8)));
typedef uint32_t table2 __attribute__((ext_vector_type(2), aligned(1)));

__device__ __forceinline__ h2 pk_min(h2 a, h2 b) { return __builtin_elementwise_min(a, b); }
__device__ __forceinline__ h2 pk_max(h2 a, h2 b) { return __builtin_elementwise_max(a, b); }

template <int CTRL>
__device__ __forceinline__ h2 permuted(h2 v)
{
    return __builtin_bit_cast(h2, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// The kept two of the four fp16 in w0 (positions 0, 1) and w1 (2, 3), in position order; pos: their positions,
// first in bits 0..1, second in bits 8..9.
__device__ __forceinline__ uint32_t keep_two(uint32_t w0, uint32_t w1, uint32_t &pos)
{
    const uint32_t k0 = ((w0 & 0x7fffu) << 2) | 3u, k1 = (((w0 >> 16) & 0x7fffu) << 2) | 2u;
    const uint32_t k2 = ((w1 & 0x7fffu) << 2) | 1u, k3 = ((w1 >> 16) & 0x7fffu) << 2;
    const uint32_t a = max(k0, k1), b = min(k0, k1), c = max(k2, k3), d = min(k2, k3);
    const uint32_t top = max(a, c), next = max(max(min(a, c), b), d);
    const uint32_t p = ~top & 3u, q = ~next & 3u;
    const uint32_t first = min(p, q), second = max(p, q);
    pos = first | second << 8;
    // bytes 2 p, 2 p + 1 of {w1, w0} for both positions
    return __builtin_amdgcn_perm(w1, w0, 0x01000100u + first * 0x0202u + second * 0x02020000u);
}

template <int BITS, int GROUP>
__global__ __launch_bounds__(256) void compress_kernel(const uint16_t *__restrict__ delta, uint8_t *__restrict__ codes,
                                                        uint8_t *__restrict__ idx, _Float16 *__restrict__ scale,
                                                        _Float16 *__restrict__ zero)
{
    // rows follow one another without gaps in the delta and in every table, and neither a group of four nor
    // a quantisation group crosses a row: the whole matrix is one run of N K entries, 16 per lane
    const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 16;
    const delta4 lo4 = *(const delta4 *)(delta + e), hi4 = *(const delta4 *)(delta + e + 8);
    const uint32_t w[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
    uint32_t pair[4], pos[4];
    h2 mn = (h2){(_Float16)0.f, (_Float16)0.f}, mx = mn;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pair[i] = keep_two(w[2 * i], w[2 * i + 1], pos[i]);
        const h2 kept = __builtin_bit_cast(h2, pair[i]);
        mn = pk_min(mn, kept);
        mx = pk_max(mx, kept);
    }
    // the group's range: 4 lanes (64 columns) or 8 lanes (128) own its columns
    mn = pk_min(mn, permuted<0xB1>(mn)); mx = pk_max(mx, permuted<0xB1>(mx));       // lane ^ 1
    mn = pk_min(mn, permuted<0x4E>(mn)); mx = pk_max(mx, permuted<0x4E>(mx));       // lane ^ 2
    if (GROUP == 128) { mn = pk_min(mn, permuted<0x141>(mn)); mx = pk_max(mx, permuted<0x141>(mx)); }   // the other four of eight lanes
    const float lo = fminf((float)mn.x, (float)mn.y), hi = fmaxf((float)mx.x, (float)mx.y);
    constexpr float qmax = (float)((1 << BITS) - 1);
    _Float16 s16 = (_Float16)((hi - lo) / qmax);
    const bool dead = (float)s16 == 0.f;
    if (dead) s16 = (_Float16)1.f;
    const float s = (float)s16;
    const float r = __builtin_amdgcn_rcpf(s);
    auto rounded = [&](float v) {
        const float q = v * r;
        return rintf(fmaf(fmaf(-q, s, v), r, q));
    };
    float z = fminf(fmaxf(rounded(0.f - lo), 0.f), qmax);
    if (dead) z = 0.f;
    table2 c, p;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const h2 kept = __builtin_bit_cast(h2, pair[2 * i + (j >> 1)]);
            const float v = (float)((j & 1) ? kept.y : kept.x);
            word = __builtin_amdgcn_cvt_pk_u8_f32(fminf(fmaxf(rounded(v) + z, 0.f), qmax), j, word);
        }
        c[i] = word;
        p[i] = pos[2 * i] | pos[2 * i + 1] << 16;
    }
    *(table2 *)(codes + e / 2) = c;
    *(table2 *)(idx + e / 2) = p;
    if ((threadIdx.x & (GROUP / 16 - 1)) == 0) {
        scale[e / GROUP] = s16;
        zero[e / GROUP] = (_Float16)z;
    }
}

}  // namespace

int dz_launch_compress(dz_ctx *ctx, const void *delta, int N, int K, int bits, int group, uint8_t *codes, uint8_t *idx,
                       void *scale, void *zero, hipStream_t st)
{
    const long long blocks = (long long)N * K / 4096;       // exact: N % 16 == 0 and K % 256 == 0
    if (blocks > 0x7fffffffLL) return DZ_ERR_SHAPE;
    auto k = bits == 4 ? (group == 128 ? compress_kernel<4, 128> : compress_kernel<4, 64>)
                       : (group == 128 ? compress_kernel<2, 128> : compress_kernel<2, 64>);
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, st, (const uint16_t *)delta, codes, idx, (_Float16 *)scale,
                       (_Float16 *)zero);
    return dz_set_hip_error(ctx, hipGetLastError());
}
