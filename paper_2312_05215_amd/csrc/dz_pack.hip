// dz_pack_delta / dz_unpack_delta kernels: canonical tables <-> streaming layout (dz_layout.h).
// Off the per-token path: packing runs once per delta (the step that ends Algorithm 1), unpacking for checks.
// pack_kernel and merge_kernel, which a serving program calls while it serves, move whole tiles, one wave
// each; the quantisation-only and unpack kernels are plain gathers, one thread per dword, group or column.
#include "dz_internal.h"

namespace {

// the canonical tables need no alignment beyond their element's
typedef uint32_t table2 __attribute__((ext_vector_type(2), aligned(1)));

// Four bytes of a table, each holding one field -> the fields in the order of the packed words.
//   codes, 4-bit: bytes 0, 1 = {t0 | t2 << 4, t1 | t3 << 4};  2-bit: {t0 | t2 << 2, t1 | t3 << 2}
__device__ __forceinline__ uint32_t pair_up(uint32_t t, int bits) { return t | t >> (16 - bits); }
//   positions: byte 0 = t0 | t1 << 2 | t2 << 4 | t3 << 6
__device__ __forceinline__ uint32_t gather_positions(uint32_t t) { t |= t >> 6; return t | t >> 12; }

// One wave packs one tile (16 rows x 256 columns).  What bounds it is bytes: 1 + 8 / GROUP read and
// (2 BITS + 4) / 32 + 4 / GROUP written per column.  Lane 16 q + r reads what it will hold for the
// sparse MFMA: 8 codes and 8 positions of row r per step (a row's four lanes and four steps together take
// one 128-byte line of each table), turns the bytes into fields with a handful of shifts and byte permutes
// and stores 16 bytes of codes and 8 of positions; the tile's (scale, zero) pairs follow.
// 4-bit codes, groups of 128: 7.6 us on 4096 x 4096 and 14.2 us on 11008 x 4096 (3.2 and 4.7 TB/s); three
// launches that gathered byte by byte, for codes, positions and scales, took 11.1 and 21.2 us.
template <int BITS, int GROUP>
__global__ __launch_bounds__(256) void pack_kernel(DzLayout L, const uint8_t *__restrict__ codes, const uint8_t *__restrict__ idx,
                                                    const uint16_t *__restrict__ scale, const uint16_t *__restrict__ zero,
                                                    uint8_t *__restrict__ out)
{
    constexpr int GPT = 256 / GROUP;
    const unsigned tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    const unsigned rt = tile / (unsigned)L.KT, kt = tile - rt * (unsigned)L.KT;
    if (rt >= (unsigned)L.RT) return;
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const size_t from = ((size_t)rt * 16 + r) * (L.K / 2) + (size_t)kt * 128 + 8 * q;
    uint32_t c[4][2], p[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const table2 cv = *(const table2 *)(codes + from + 32 * s), pv = *(const table2 *)(idx + from + 32 * s);
        c[s][0] = cv.x; c[s][1] = cv.y; p[s][0] = pv.x; p[s][1] = pv.y;
    }
    constexpr int SZ = 16 * GPT;                        // (scale, zero) pairs of the tile
    uint32_t sz = 0;
    if (lane < SZ) {
        const size_t g = ((size_t)rt * 16 + lane / GPT) * (L.K / GROUP) + (size_t)kt * GPT + lane % GPT;
        sz = (uint32_t)scale[g] | (uint32_t)zero[g] << 16;
    }
    uint32_t pw[2];                                     // steps 2h (low half) and 2h + 1
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = gather_positions(p[2 * h + (i >> 1)][i & 1] & 0x03030303u);
        pw[h] = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
    }
    if (BITS == 4) {
        uint32_t cw[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            cw[s] = __builtin_amdgcn_perm(pair_up(c[s][1] & 0x0f0f0f0fu, 4), pair_up(c[s][0] & 0x0f0f0f0fu, 4), 0x05010400u);
        *(uint4 *)(out + (size_t)tile * 1024 + lane * 16) = (uint4){cw[0], cw[1], cw[2], cw[3]};
        *(uint2 *)(out + L.off_idx + (size_t)tile * 512 + lane * 8) = (uint2){pw[0], pw[1]};
    } else {
        uint32_t u[4];                                  // bytes 0, 1: codes 0, 2, 4, 6 / 1, 3, 5, 7 of a step
#pragma unroll
        for (int s = 0; s < 4; ++s) u[s] = pair_up(c[s][0] & 0x03030303u, 2) | pair_up(c[s][1] & 0x03030303u, 2) << 4;
        *(uint4 *)(out + (size_t)tile * 1024 + lane * 16) =
            (uint4){__builtin_amdgcn_perm(u[1], u[0], 0x05010400u), __builtin_amdgcn_perm(u[3], u[2], 0x05010400u), pw[0], pw[1]};
    }
    if (lane < SZ) *(uint32_t *)(out + L.off_scale + (size_t)tile * (SZ * 4) + lane * 4) = sz;
}

__global__ void pack_scale_kernel(DzLayout L, const uint16_t *__restrict__ scale,
                                  const uint16_t *__restrict__ zero, uint32_t *__restrict__ out)
{
    const int ng = L.K / L.group;
    size_t total = (size_t)L.N * ng;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int n = (int)(i / ng), gq = (int)(i % ng);
    out[dz_scale_dword(L, n, gq)] = (uint32_t)scale[i] | ((uint32_t)zero[i] << 16);
}

__device__ inline float half_bits_to_float(uint16_t h)
{
    _Float16 v;
    __builtin_memcpy(&v, &h, 2);
    return (float)v;
}

// One thread per (row, group of four): writes the two codes, two positions and, if asked, the
// four dense fp32 values  (code - zero) * scale  (an exact product in fp32).
__global__ void unpack_kernel(DzLayout L, const uint32_t *__restrict__ blob, uint8_t *__restrict__ codes,
                              uint8_t *__restrict__ idx, float *__restrict__ dense)
{
    const int g4n = L.K / 4;
    size_t total = (size_t)L.N * g4n;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int n = (int)(i / g4n), g4 = (int)(i % g4n);
    const uint32_t mask = (1u << L.bits) - 1u;
    uint32_t c[2], p[2];
    for (int j = 0; j < 2; ++j) {
        DzSlot s = dz_slot_of(L, n, 2 * g4 + j);
        c[j] = (blob[dz_code_dword(L, s)] >> dz_code_shift(L, s)) & mask;
        p[j] = (blob[dz_idx_dword(L, s)] >> dz_idx_shift(s)) & 3u;
    }
    size_t e = (size_t)n * (L.K / 2) + 2 * (size_t)g4;
    if (codes) { codes[e] = (uint8_t)c[0]; codes[e + 1] = (uint8_t)c[1]; }
    if (idx) { idx[e] = (uint8_t)p[0]; idx[e + 1] = (uint8_t)p[1]; }
    if (dense) {
        uint32_t sz = blob[dz_scale_dword(L, n, (4 * g4) / L.group)];
        float s = half_bits_to_float((uint16_t)(sz & 0xffff));
        float z = half_bits_to_float((uint16_t)(sz >> 16));
        float a = ((float)c[0] - z) * s, b = ((float)c[1] - z) * s;
        float *o = dense + (size_t)n * L.K + 4 * (size_t)g4;
#pragma unroll
        for (uint32_t pos = 0; pos < 4; ++pos) o[pos] = (p[1] == pos) ? b : (p[0] == pos) ? a : 0.f;
    }
}

__global__ void unpack_scale_kernel(DzLayout L, const uint32_t *__restrict__ blob,
                                    uint16_t *__restrict__ scale, uint16_t *__restrict__ zero)
{
    const int ng = L.K / L.group;
    size_t total = (size_t)L.N * ng;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int n = (int)(i / ng), gq = (int)(i % ng);
    uint32_t sz = blob[dz_scale_dword(L, n, gq)];
    if (scale) scale[i] = (uint16_t)(sz & 0xffff);
    if (zero) zero[i] = (uint16_t)(sz >> 16);
}

// ---- quantisation-only format: one thread per dword of codes (pack) or per column (unpack)
__global__ void qpack_codes_kernel(DzLayout L, const uint8_t *__restrict__ codes, uint32_t *__restrict__ out)
{
    const int per_dword = 32 / L.bits;                  // 8 or 16 codes
    const size_t total = (size_t)L.N * L.K / per_dword;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    // dword i of plane C: find (tile, half, lane, dword-in-lane), then gather its codes
    const size_t tile_dwords = (L.bits == 4) ? 512 : 256;
    const size_t tile = i / tile_dwords;
    const int r = (int)(i % tile_dwords);
    int h, lane, d;
    if (L.bits == 4) { h = r / 256; lane = (r % 256) / 4; d = r % 4; }
    else { lane = r / 4; d = r % 4; h = d >> 1; }
    const int rt = (int)(tile / L.KT), kt = (int)(tile % L.KT);
    const int n = rt * 16 + (lane & 15), q = lane >> 4;
    const uint8_t *row = codes + (size_t)n * L.K;
    const uint32_t mask = (1u << L.bits) - 1u;
    uint32_t w = 0;
    const int nsteps = (L.bits == 4) ? 1 : 2;
    for (int ss = 0; ss < nsteps; ++ss) {
        const int step = (L.bits == 4) ? d : 2 * (d & 1) + ss;
        const int k0 = kt * 256 + step * 64 + q * 16;   // first column of this lane's step
        for (int j = 0; j < 4; ++j)
            for (int hh = 0; hh < 2; ++hh) {
                const uint32_t c = row[k0 + 4 * j + 2 * h + hh] & mask;
                w |= c << ((L.bits == 4) ? 16 * hh + 4 * j : 16 * hh + 8 * ss + 2 * j);
            }
    }
    out[i] = w;
}

__global__ void qunpack_kernel(DzLayout L, const uint32_t *__restrict__ blob, uint8_t *__restrict__ codes,
                               float *__restrict__ dense)
{
    const size_t total = (size_t)L.N * L.K;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int n = (int)(i / L.K), k = (int)(i % L.K);
    const uint32_t c = (blob[dz_qcode_dword(L, n, k)] >> dz_qcode_shift(L, k)) & ((1u << L.bits) - 1u);
    if (codes) codes[i] = (uint8_t)c;
    if (dense) {
        const uint32_t sz = blob[dz_scale_dword(L, n, k / L.group)];
        dense[i] = ((float)c - half_bits_to_float((uint16_t)(sz >> 16))) * half_bits_to_float((uint16_t)(sz & 0xffff));
    }
}

// merged[n][k] = f16( float(W[n][k]) + (code - zero) * scale at the kept columns ).  One wave per tile of
// 16 rows x 256 columns, all of its loads requested before the first is used.  What bounds it is bytes:
// 4 + (2 BITS + 4) / 32 + 4 / GROUP per column.  W is read and the result written in 16-byte pieces, a row's
// four lanes side by side: lane 16 q + r handles columns 32 i + 8 q .. + 7 of each step, i = 0, 1, whose codes
// and positions are half of the words that lane 16 (2 i + q / 2) + r of the sparse MFMA would hold (the same
// 64-byte pieces of the tile serve two lanes).
// 4-bit, groups of 128: 18.3 us on 4096 x 4096 and 40.3 us on 11008 x 4096 (4.1 and 4.9 TB/s); one thread
// per group of four, whose blocks read each line of the tile 16 times over, took 22.8 and 55.4 us.
template <int BITS, int GROUP>
__global__ __launch_bounds__(256) void merge_kernel(DzLayout L, const _Float16 *__restrict__ W, const uint8_t *__restrict__ blob,
                                                     _Float16 *__restrict__ merged)
{
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    constexpr int GPT = 256 / GROUP;
    const unsigned tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    const unsigned rt = tile / (unsigned)L.KT, kt = tile - rt * (unsigned)L.KT;
    if (rt >= (unsigned)L.RT) return;
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const size_t at = ((size_t)rt * 16 + r) * L.K + (size_t)kt * 256 + 8 * q;
    h8 w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = *(const h8 *)(W + at + 32 * i);      // step i / 2, half i % 2
    uint32_t c[2][4], p[2][2], sz[GPT];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int from = 16 * (2 * i + (q >> 1)) + r;
        const uint4 v = *(const uint4 *)(blob + (size_t)tile * 1024 + from * 16);
        if (BITS == 4) {
            const uint2 x = *(const uint2 *)(blob + L.off_idx + (size_t)tile * 512 + from * 8);
            c[i][0] = v.x; c[i][1] = v.y; c[i][2] = v.z; c[i][3] = v.w;
            p[i][0] = x.x; p[i][1] = x.y;
        } else {
            c[i][0] = v.x; c[i][1] = v.x >> 8; c[i][2] = v.y; c[i][3] = v.y >> 8;
            p[i][0] = v.z; p[i][1] = v.w;
        }
    }
#pragma unroll
    for (int g = 0; g < GPT; ++g) sz[g] = *(const uint32_t *)(blob + L.off_scale + ((size_t)tile * 16 + r) * (GPT * 4) + g * 4);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int s = i >> 1;
        const uint32_t szw = sz[s * GPT / 4];
        const float sc = half_bits_to_float((uint16_t)(szw & 0xffff)), z = half_bits_to_float((uint16_t)(szw >> 16));
        // kept slots e = 4 (q % 2) .. + 3 of the word's eight: two groups of four columns
        const uint32_t cw = c[i & 1][s] >> (2 * BITS * (q & 1));
        const uint32_t pw = p[i & 1][s >> 1] >> (16 * (s & 1) + 8 * (q & 1));
        h8 o;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (float)w[i][4 * g + k];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t code = (cw >> (16 * j + BITS * g)) & ((1u << BITS) - 1u);
                const uint32_t at4 = (pw >> (4 * g + 2 * j)) & 3u;
                const float d = ((float)code - z) * sc;
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) v[k] += (at4 == k) ? d : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) o[4 * g + k] = (_Float16)v[k];
        }
        *(h8 *)(merged + at + 32 * i) = o;
    }
}

inline unsigned blocks_for(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

int dz_launch_pack(dz_ctx *ctx, const uint8_t *codes, const uint8_t *idx, const void *scale,
                   const void *zero, int N, int K, int bits, int group, void *packed, hipStream_t st)
{
    const DzLayout L = dz_make_layout(N, K, bits, group);
    auto k = bits == 4 ? (group == 128 ? pack_kernel<4, 128> : pack_kernel<4, 64>)
                       : (group == 128 ? pack_kernel<2, 128> : pack_kernel<2, 64>);
    hipLaunchKernelGGL(k, dim3(blocks_for((size_t)L.RT * L.KT, 4)), dim3(256), 0, st, L, codes, idx, (const uint16_t *)scale,
                       (const uint16_t *)zero, (uint8_t *)packed);
    return dz_set_hip_error(ctx, hipGetLastError());
}

int dz_launch_unpack(dz_ctx *ctx, const void *packed, int N, int K, int bits, int group, uint8_t *codes,
                     uint8_t *idx, void *scale, void *zero, float *dense, hipStream_t st)
{
    DzLayout L = dz_make_layout(N, K, bits, group);
    const int bs = 256;
    if (codes || idx || dense)
        hipLaunchKernelGGL(unpack_kernel, dim3(blocks_for((size_t)N * (K / 4), bs)), dim3(bs), 0, st, L,
                           (const uint32_t *)packed, codes, idx, dense);
    if (scale || zero)
        hipLaunchKernelGGL(unpack_scale_kernel, dim3(blocks_for((size_t)N * (K / group), bs)), dim3(bs), 0, st,
                           L, (const uint32_t *)packed, (uint16_t *)scale, (uint16_t *)zero);
    return dz_set_hip_error(ctx, hipGetLastError());
}

int dz_launch_qpack(dz_ctx *ctx, const uint8_t *codes, const void *scale, const void *zero, int N, int K, int bits,
                    int group, void *packed, hipStream_t st)
{
    DzLayout L = dz_make_qlayout(N, K, bits, group);
    const int bs = 256;
    hipLaunchKernelGGL(qpack_codes_kernel, dim3(blocks_for((size_t)N * K * bits / 32, bs)), dim3(bs), 0, st, L, codes,
                       (uint32_t *)packed);
    hipLaunchKernelGGL(pack_scale_kernel, dim3(blocks_for((size_t)N * (K / group), bs)), dim3(bs), 0, st, L,
                       (const uint16_t *)scale, (const uint16_t *)zero, (uint32_t *)packed);
    return dz_set_hip_error(ctx, hipGetLastError());
}

int dz_launch_qunpack(dz_ctx *ctx, const void *packed, int N, int K, int bits, int group, uint8_t *codes, void *scale,
                      void *zero, float *dense, hipStream_t st)
{
    DzLayout L = dz_make_qlayout(N, K, bits, group);
    const int bs = 256;
    if (codes || dense)
        hipLaunchKernelGGL(qunpack_kernel, dim3(blocks_for((size_t)N * K, bs)), dim3(bs), 0, st, L, (const uint32_t *)packed,
                           codes, dense);
    if (scale || zero)
        hipLaunchKernelGGL(unpack_scale_kernel, dim3(blocks_for((size_t)N * (K / group), bs)), dim3(bs), 0, st, L,
                           (const uint32_t *)packed, (uint16_t *)scale, (uint16_t *)zero);
    return dz_set_hip_error(ctx, hipGetLastError());
}

int dz_launch_merge(dz_ctx *ctx, const void *W, const void *packed, int N, int K, int bits, int group, void *merged,
                    hipStream_t st)
{
    const DzLayout L = dz_make_layout(N, K, bits, group);
    auto k = bits == 4 ? (group == 128 ? merge_kernel<4, 128> : merge_kernel<4, 64>)
                       : (group == 128 ? merge_kernel<2, 128> : merge_kernel<2, 64>);
    hipLaunchKernelGGL(k, dim3(blocks_for((size_t)L.RT * L.KT, 4)), dim3(256), 0, st, L, (const _Float16 *)W,
                       (const uint8_t *)packed, (_Float16 *)merged);
    return dz_set_hip_error(ctx, hipGetLastError());
}
