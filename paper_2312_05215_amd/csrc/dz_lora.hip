// Low-rank adapters served like compressed deltas (paper Section 3.2: adapters are registered next to
// deltas and served by the same engine; Section 6.4).  For request t with adapter m = Idx[t]
//
//     y[t] = B_m . (A_m . x[t]),        A_m [rank][K],  B_m [N][rank],  fp16
//
// the selective batched product of Section 5.2 with a low-rank matrix in place of a delta.  Adapters
// are a few hundred KB per layer, so neither kernel is shaped by bandwidth or by the matrix cores: what
// bounds a decode-sized call is how long one workgroup waits for its loads, and the launches themselves.
//   shrink: u[t] = A_m . x[t]  (fp32 [T][rank]) -- one workgroup of four waves per (request, 8 ranks): the
//           lanes stride over k with 16-byte loads and packed dot products, 16 K at most of a row per lane
//           and wave, then a reduction over the lanes in which a lane passes on half of its sums at each
//           step (10 exchanges for 8 sums instead of 48) and one over the waves through LDS;
//   expand: y[t] = B_m . u[t]  -- one thread per (request, 4 outputs), fp32, one rounding at the store.
// The requests keep their own order.  Sorting them by adapter first cost a launch of its own and brought
// nothing: neighbouring workgroups run on different XCDs, and what all requests read of the adapters for one
// set of 8 ranks (D x 16 K bytes) stays in the L2s either way.  Larger calls do not miss it: on T = 1 .. 2048, K = 1024 ..
// 8192, up to 128 adapters of rank 64, mixed and in runs, a call took 0.2 to 0.97 times as long as with the sort (T = 2048,
// 32 adapters of rank 64, 8192 x 8192: 851 -> 655 us mixed, 596 -> 565 in runs).
// T = 64, rank 16, 4096 x 4096: shrink 4.4 us and expand 4.1 us; with one wave per shrink workgroup behind
// a sort of the requests it was 7.3 + 3.8 us and 3.9 us for the sort.
#include "dz_internal.h"

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

struct LoraPtrs { const void *p[DZ_MAX_DELTAS]; };

__device__ __forceinline__ float dot8(h8 a, h8 b, float acc)
{
    acc = __builtin_amdgcn_fdot2((h2){a[0], a[1]}, (h2){b[0], b[1]}, acc, false);
    acc = __builtin_amdgcn_fdot2((h2){a[2], a[3]}, (h2){b[2], b[3]}, acc, false);
    acc = __builtin_amdgcn_fdot2((h2){a[4], a[5]}, (h2){b[4], b[5]}, acc, false);
    acc = __builtin_amdgcn_fdot2((h2){a[6], a[7]}, (h2){b[6], b[7]}, acc, false);
    return acc;
}

// grid: (T, rank / 8); block: four waves
__global__ __launch_bounds__(256) void lora_shrink_kernel(const _Float16 *__restrict__ x, LoraPtrs A, int D, int rank,
                                                           const int32_t *__restrict__ ids, float *__restrict__ u, int T, int K)
{
    __shared__ float s_part[4][8];
    const int t = blockIdx.x;
    const int m = ids[t];
    if (m < 0 || m >= D) return;                // no adapter: the expand pass writes the zero
    const int r0 = blockIdx.y * 8;
    const _Float16 *a = (const _Float16 *)A.p[m] + (size_t)r0 * K;
    const _Float16 *xr = x + (size_t)t * K;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int k = threadIdx.x * 8; k < K; k += 256 * 8) {
        const h8 xv = *(const h8 *)(xr + k);
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[r] = dot8(*(const h8 *)(a + (size_t)r * K + k), xv, acc[r]);
    }
    // lanes with bit 5 / 4 / 3 set go on with the upper half of the sums they still hold
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 4; h >= 1; h >>= 1) {
        const bool upper = (lane & (8 * h)) != 0;
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const float keep = upper ? acc[i + h] : acc[i], give = upper ? acc[i] : acc[i + h];
            acc[i] = keep + __shfl_xor(give, 8 * h, 64);
        }
    }
#pragma unroll
    for (int d = 4; d >= 1; d >>= 1) acc[0] += __shfl_xor(acc[0], d, 64);
    if ((lane & 7) == 0) s_part[threadIdx.x >> 6][lane >> 3] = acc[0];
    __syncthreads();
    if (threadIdx.x < 8) {
        const int r = threadIdx.x;
        u[(size_t)t * rank + r0 + r] = (s_part[0][r] + s_part[1][r]) + (s_part[2][r] + s_part[3][r]);
    }
}

// grid: (ceil(N / 1024), T); block: 256 threads, 4 outputs each
__global__ __launch_bounds__(256) void lora_expand_kernel(const float *__restrict__ u, LoraPtrs B, int D, int rank,
                                                           const int32_t *__restrict__ ids, _Float16 *__restrict__ out, int T, int N,
                                                           int accumulate, int32_t *__restrict__ err_flag)
{
    const int t = blockIdx.y;
    const int n0 = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (n0 >= N) return;
    const int m = ids[t];
    const bool valid = m >= 0 && m < D;
    if (!valid && m != -1 && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err_flag, 1);
    float y[4] = {0.f, 0.f, 0.f, 0.f};
    if (valid) {
        const _Float16 *b = (const _Float16 *)B.p[m] + (size_t)n0 * rank;
        const float *ut = u + (size_t)t * rank;
        for (int r = 0; r < rank; r += 8) {
            float uv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) uv[i] = ut[r + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const h8 bv = *(const h8 *)(b + (size_t)j * rank + r);
#pragma unroll
                for (int i = 0; i < 8; ++i) y[j] = fmaf((float)bv[i], uv[i], y[j]);
            }
        }
    }
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    _Float16 *o = out + (size_t)t * N + n0;
    if (accumulate) {
        const h4 prev = *(const h4 *)o;
        y[0] += (float)prev.x; y[1] += (float)prev.y; y[2] += (float)prev.z; y[3] += (float)prev.w;
    }
    *(h4 *)o = (h4){(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
}

}  // namespace

int dz_launch_lora(dz_ctx *ctx, const void *x, const void *const *A, const void *const *B, int D, int rank, const int32_t *ids,
                   float *u, void *out, int T, int N, int K, int accumulate, hipStream_t st)
{
    LoraPtrs pa, pb;
    for (int m = 0; m < DZ_MAX_DELTAS; ++m) { pa.p[m] = m < D ? A[m] : nullptr; pb.p[m] = m < D ? B[m] : nullptr; }
    hipLaunchKernelGGL(lora_shrink_kernel, dim3(T, rank / 8), dim3(256), 0, st, (const _Float16 *)x, pa, D, rank, ids, u, T, K);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return dz_set_hip_error(ctx, e);
    hipLaunchKernelGGL(lora_expand_kernel, dim3((N + 1023) / 1024, T), dim3(256), 0, st, (const float *)u, pb, D, rank, ids,
                       (_Float16 *)out, T, N, accumulate, ctx->err_flag);
    return dz_set_hip_error(ctx, hipGetLastError());
}
