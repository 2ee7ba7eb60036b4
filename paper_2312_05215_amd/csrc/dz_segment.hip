// Request reordering on the device (paper Section 5.2: requests of one delta are grouped together
// before the delta product).  A stable counting sort of the request->delta index vector, done by
// one workgroup of 16 waves.  Each wave owns a contiguous run of requests and, where LDS has room, a
// histogram of its own; 64 requests rank themselves without a loop over the keys (the lanes that hold
// the same key are the intersection of one ballot per key bit; a lane's rank among them is the population
// count of the lower lanes in that mask).  A prefix sum over (key, wave) turns the histograms into write
// cursors, and a second walk over the run writes every request to its place.
//
// What bounds it is latency: one launch, two walks over the index vector, LDS round trips.  With one wave that
// walked all requests, and all distinct keys of each 64 in turn, a call took 122 us at T = 2048 over 16 deltas in
// mixed order (17.5 us where every 64 name one or two), 54 us at T = 512 over 32; it takes 8 us from T = 65 to
// 2048 (calls back to back, of which the launch is most) and 16 us at T = 8192 over 128, before 1480.
// The prefix sum is shared by the waves too: one wave that walked all of it took 55 us for one request over 8192 keys
// and 29 over 4096 (10 and 8 here), and 248 us at T = 8192 over 8192 (202 here).
#include "dz_internal.h"

namespace {

constexpr int SEG_WAVES = 16, SEG_THREADS = SEG_WAVES * 64;
constexpr int SEG_LDS = 64 * 1024 - SEG_WAVES * 4;      // what a launch may use without an attribute, less s_total, the only static array

__device__ inline unsigned lanes_below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// For each active lane: where its request goes, given the cursor of its key in `cur`, which moves on by the number
// of lanes with that key.  All lanes of the wave call it.
__device__ inline int place(int32_t *cur, int key, bool active, int key_bits, int lane)
{
    unsigned long long same = __ballot(active);
    for (int b = 0; b < key_bits; ++b) {
        const bool bit = (key >> b) & 1;
        const unsigned long long m = __ballot(bit);
        same &= bit ? m : ~m;
    }
    const int leader = active ? (int)__builtin_ctzll(same) : lane;
    int at = 0;
    if (active && lane == leader) at = atomicAdd(&cur[key], __builtin_popcountll(same));
    return __shfl(at, leader, 64) + (int)lanes_below(same);
}

// The column tiles of the fused kernel (DzFusedTile), by one thread: segments in their order, up to DZ_FUSED_BLOCKS blocks of
// 16 rows and two segments a tile.  A segment that fills more than a tile is cut into equal ones, and the end of a segment
// waits for the next segment unless it has ten blocks by itself and the next one does not fit whole: a step costs six
// blocks' time beside the blocks', so few wide tiles are the cheapest.  (Lists for nine narrower limits as well, for each
// launch to choose the one that fills its last round best, brought less than the pass grew by: 5 to 10 us.)
__host__ __device__ void plan_tiles(const int32_t *start, int T, int D, DzFusedTile *plan)
{
    constexpr int CAP = DZ_FUSED_BLOCKS;
    int n = 0, most = 0, o_start = 0, o_rows = 0, o_key = 0;        // the open tile's first segment, if it has rows
    auto emit = [&](int s0, int r0, int k0, int s1, int r1, int k1) {
        plan[++n] = DzFusedTile{s0, r0, k0, s1, r1, k1, {0, 0}};
        const int cost = dz_fused_cost((r1 ? (r0 + 31) >> 5 << 1 : (r0 + 15) >> 4) + ((r1 + 15) >> 4));
        most = cost > most ? cost : most;
    };
    for (int key = 0; key <= D; ++key) {
        int at = start[key], rows = (key < D ? start[key + 1] : T) - at;
        if (key == D && o_rows) {                       // rows of the base model have tiles of their own
            emit(o_start, o_rows, o_key, 0, 0, 0);
            o_rows = 0;
        }
        while (rows > 0) {
            const int blocks = (rows + 15) >> 4, open = (o_rows + 31) >> 5 << 1;     // (a second segment begins at an even block)
            int take = 0;                               // rows that leave with a tile
            if (open == 0 && blocks <= CAP) {
                o_start = at; o_rows = rows; o_key = key;
                break;
            }
            if (open == 0) {
                const int pieces = (blocks + CAP - 1) / CAP;
                take = (blocks + pieces - 1) / pieces * 16;
                emit(at, take, key, 0, 0, 0);
            } else if (open + blocks <= CAP) {
                take = rows;
                emit(o_start, o_rows, o_key, at, take, key);
            } else if (open >= 10) {
                emit(o_start, o_rows, o_key, 0, 0, 0);
            } else {
                take = (CAP - open) * 16;
                emit(o_start, o_rows, o_key, at, take, key);
            }
            o_rows = 0;
            at += take;
            rows -= take;
        }
    }
    if (o_rows) emit(o_start, o_rows, o_key, 0, 0, 0);
    plan[0] = DzFusedTile{n, most, 0, 0, 0, 0, {0, 0}};
}

// key = delta index, or D for "no delta" (index -1 or out of range).  `runs` waves share the requests.
__global__ __launch_bounds__(SEG_THREADS) void segment_kernel(const int32_t *__restrict__ ids, int T, int D, int runs, int key_bits,
                                                              int32_t *__restrict__ counts,
                                                              int32_t *__restrict__ offsets,
                                                              int32_t *__restrict__ perm,
                                                              int32_t *__restrict__ key_out,
                                                              DzFusedTile *__restrict__ plan,
                                                              int32_t *__restrict__ err_flag)
{
    extern __shared__ int32_t cursor[];          // [runs][D + 1] histograms, then running write cursors
    __shared__ int32_t s_total[SEG_WAVES];       // requests of each wave's run of keys
    int32_t *const s_start = cursor + runs * (D + 1);    // first sorted position of each key: there only with a plan
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < runs * (D + 1); i += SEG_THREADS) cursor[i] = 0;
    __syncthreads();
    const int len = (T + 64 * runs - 1) / (64 * runs) * 64;         // requests per run
    const int begin = min(wave * len, T), end = wave < runs ? min(begin + len, T) : begin;
    int32_t *const mine = cursor + (wave < runs ? wave : 0) * (D + 1);
    bool bad = false;
    for (int t0 = begin; t0 < end; t0 += 64) {
        const int t = t0 + lane, id = t < end ? ids[t] : -1;
        const bool valid = id >= 0 && id < D;
        bad |= !valid && id != -1;
        (void)place(mine, valid ? id : D, t < end, key_bits, lane);
    }
    if (__ballot(bad) && lane == 0) atomicOr(err_flag, 1);
    __syncthreads();
    // Exclusive prefix sum over the D + 1 keys and the runs within a key.  Each wave owns a run of keys, 64 at a time, on
    // top of the totals of the waves below it; where 64 keys are all, wave 0 has them and needs no totals.
    const int keys = (D + 64 * SEG_WAVES) / (64 * SEG_WAVES) * 64;  // keys per wave: a multiple of 64
    const int first = min(wave * keys, D + 1), last = min(first + keys, D + 1);
    int base = 0;
    if (D + 1 > 64) {
        int sum = 0;
        for (int i = first + lane; i < last; i += 64)
            for (int w = 0; w < runs; ++w) sum += cursor[w * (D + 1) + i];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if (lane == 0) s_total[wave] = sum;
        __syncthreads();
        for (int w = 0; w < wave; ++w) base += s_total[w];
    }
    for (int i0 = first; i0 < last; i0 += 64) {
        const int i = i0 + lane;
        int c = 0;
        if (i < last)
            for (int w = 0; w < runs; ++w) c += cursor[w * (D + 1) + i];
        int incl = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, 64);
            if (lane >= d) incl += up;
        }
        int excl = base + incl - c;
        if (i < last) {
            if (counts && i < D) counts[i] = c;
            if (offsets) offsets[i] = excl;
            if (plan) s_start[i] = excl;
            for (int w = 0; w < runs; ++w) {
                const int n = cursor[w * (D + 1) + i];
                cursor[w * (D + 1) + i] = excl;
                excl += n;
            }
        }
        base += __shfl(incl, 63, 64);
    }
    __syncthreads();
    if (plan && tid == SEG_THREADS - 1) plan_tiles(s_start, T, D, plan);
    for (int t0 = begin; t0 < end; t0 += 64) {
        const int t = t0 + lane, id = t < end ? ids[t] : -1;
        const int key = (id >= 0 && id < D) ? id : D;
        const int pos = place(mine, key, t < end, key_bits, lane);
        if (t < end) {
            if (perm) perm[pos] = t;
            if (key_out) key_out[pos] = key;
        }
    }
}

// The list alone, for an order that a call of another kernel made without it: from the offsets of that sort, by one thread.
// Kernel times in us, this one | a sort without | a sort with the list: 777 rows over 3 deltas 2.3 | 3.8 | 4.5, 2048 over 8
// 4.2 | 5.2 | 7.9, 4096 over 32 9.4 | 8.4 | 16.1, 16384 over 128 36 | 30 | 60.  So an order is not made twice for the list, and a
// sort leaves it only where its own call wants it: layers that never do would pay for it.
__global__ __launch_bounds__(64) void fused_list_kernel(const int32_t *__restrict__ offsets, int T, int D, DzFusedTile *__restrict__ plan)
{
    __shared__ int32_t s_start[DZ_MAX_DELTAS + 1];
    for (int i = threadIdx.x; i <= D; i += 64) s_start[i] = offsets[i];
    __syncthreads();
    if (threadIdx.x == 0) plan_tiles(s_start, T, D, plan);
}

}  // namespace

// The list of the order that the last sort left, D <= DZ_MAX_DELTAS.
int dz_launch_fused_list(dz_ctx *ctx, int T, int D, hipStream_t st)
{
    if (D > DZ_MAX_DELTAS) return DZ_ERR_ARG;
    hipLaunchKernelGGL(fused_list_kernel, dim3(1), dim3(64), 0, st, ctx->seg_offsets, T, D, ctx->seg_plan);
    return dz_set_hip_error(ctx, hipGetLastError());
}

int dz_launch_segment(dz_ctx *ctx, const int32_t *ids, int T, int D, int32_t *counts, int32_t *offsets,
                      int32_t *perm, int32_t *key, DzFusedTile *plan, hipStream_t st)
{
    // as many runs as have 64 requests each and whose histograms fit (D <= DZ_SEG_MAX_D: one always does), with one more of the
    // same size where a plan is wanted (D <= DZ_MAX_DELTAS)
    const int extra = plan ? 1 : 0;
    const int fit = SEG_LDS / ((D + 1) * (int)sizeof(int32_t)) - extra, chunks = (T + 63) / 64;
    int runs = fit < SEG_WAVES ? fit : SEG_WAVES;
    if (runs > chunks) runs = chunks > 0 ? chunks : 1;
    int key_bits = 0;
    while ((D >> key_bits) > 0) ++key_bits;
    const size_t lds = (size_t)(runs + extra) * (D + 1) * sizeof(int32_t);
    hipLaunchKernelGGL(segment_kernel, dim3(1), dim3(SEG_THREADS), lds, st, ids, T, D, runs, key_bits, counts, offsets, perm, key,
                       plan, ctx->err_flag);
    return dz_set_hip_error(ctx, hipGetLastError());
}

// The list that a sort leaves where key d begins at start[d] (start[D]: the rows of the base model), for tests without a GPU:
// its head and tiles.  Returns the most tiles there can be, which is what the workspace and the grid are sized for.
extern "C" int dz_fused_list(const int32_t *start, int T, int D, DzFusedTile *list)
{
    if (list) plan_tiles(start, T, D, list);
    return dz_fused_tiles_max(T, D);
}
