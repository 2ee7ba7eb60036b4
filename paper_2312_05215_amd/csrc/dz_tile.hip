// The wide tiled kernel for the base product of large batches (prefill):
//
//   out[t] = f16( x[t] . W^T )      (the batched base GEMM of paper Section 5.1 Eq. (2))
//
// What bounds a tiled kernel on this chip is the operand bytes a CU has to bring in per flop (a CU
// keeps only so many cache lines in flight, and they arrive with HBM latency), so the tile is as
// large as the registers allow and both operands travel the cheapest way:
//   * a workgroup (8 waves, 4 x 2) owns 256 rows of N x 256 request rows and walks k in steps of
//     64; a wave owns 4 row tiles x 8 column blocks = 32 accumulator tiles (128 registers), the
//     squarest wave tile, which needs the fewest fragment bytes from LDS per MFMA.  Tiles of 5 to 7
//     column blocks a wave, or of 5 to 7 row tiles with the waves as 2 x 4, are chosen where they fill
//     the last round of one tile per CU better;
//   * the W and x slices of a step go from global memory straight into LDS (buffer loads with an
//     LDS destination: no staging registers, no LDS store instructions), double buffered, one
//     barrier per step.  Such a load writes the 64 lanes' 16-byte pieces side by side, so LDS rows
//     are unpadded 128-byte runs; to keep fragment reads off one bank set, slot s of row r holds
//     piece s ^ ((r >> 1) & 7) of the row -- the swizzle is applied to the global address a lane
//     fetches, and again by the lanes that read fragments.  A wave's load covers 8 rows x 128
//     bytes: whole cache lines.  A and B fragments of the MFMAs are read from LDS, B two column
//     blocks ahead of the MFMAs that use it;
//   * the tiles of the last, partly filled round of one-tile-per-CU are cut into k slices that
//     meet in fp32, as in the narrower tiled kernel.
//   * the projections of one call are one launch, their row blocks numbered one projection after the other:
//     dz_linear_group without deltas, us in one launch of the narrower kernel -> here: 65 x (3 x 1024) x 1024 20.5 ->
//     15.2, 777 x (3 x 4096) x 4096 116 -> 74 (154 with a launch here for each), 2048 x (2 x 11008) x 4096 455 -> 346,
//     1000 x (2 x 28672) x 8192 1089 -> 815; 0.5 to 1.1 times as long over 310 sizes of two to four projections, the
//     1.1 where a batch of up to 256 rows just fills the narrower kernel's last round.
// Fused and delta-only calls stay with the narrower kernel: with 128 registers of accumulators the
// packed-delta operands of a wave no longer fit beside them.
#include "dz_mma.h"
#include <algorithm>


namespace {

constexpr int TLD = 64;             // LDS row stride in halfs of a 64-k slice (no padding: see the swizzle)
constexpr int TW = 8;               // waves per workgroup
constexpr int TTHREADS = TW * 64;

// 16 bytes per lane from global memory to LDS: 1 KB side by side, in lane order
__device__ __forceinline__ void to_lds(__amdgpu_buffer_rsrc_t rs, _Float16 *lds, uint32_t voff, uint32_t soff)
{
    typedef __attribute__((address_space(3))) void lds_void;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)lds, 16, voff, soff, 0, 0);
}

// TWR x (8 / TWR) waves along the rows of N and along the request rows, each with TRT row tiles x TJ column blocks
template <int TWR, int TRT, int TJ, bool GROUP>
__global__ __launch_bounds__(TTHREADS) void tile_kernel(DzStreamArgs a, DzGroup gp, int NRB, int nchunks)
{
    constexpr int TWC = TW / TWR;
    constexpr int TROWS = TWR * TRT * 16;   // rows of N per tile
    constexpr int TCH = TWC * TJ * 16;      // request rows per tile
    extern __shared__ __attribute__((aligned(16))) _Float16 lds[];     // W: 2 x [TROWS][TLD]; x: 2 x [TCH][TLD]
    _Float16 *const ws = lds;
    _Float16 *const xs = lds + 2 * TROWS * TLD;
    __shared__ int s_last;

    const int tid = threadIdx.x;
    Geo g;
    g.lane = tid & 63; g.row = g.lane & 15; g.q = g.lane >> 4;
    g.KT = a.K >> 8;
    g.LDW = TLD;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % TWR, wc = wave / TWR;     // this wave's block of rows and of request rows

    // tile of this workgroup: as in the narrower tiled kernel (whole tiles first, XCD by XCD, then
    // the tiles of the last round cut into S slices of k)
    const int I0 = a.max_slots, tiles = NRB * nchunks;
    const int Tt = (tiles - 8 * I0 + 7) / 8;
    const int xcd = (int)(blockIdx.x % 8), bi = (int)(blockIdx.x / 8);
    int tile, ks = 0, S = 1;
    if (bi < I0) {
        tile = xcd * I0 + bi;
        if (tile >= tiles) return;
    } else {
        S = a.S;
        const int tt = (bi - I0) / S;
        ks = (bi - I0) - tt * S;
        tile = 8 * I0 + xcd * Tt + tt;
        if (tt >= Tt || tile >= tiles) return;
    }
    const int slot0 = (tile - 8 * I0) * S;
    const int rb = tile / nchunks;
    const int chunk = tile - rb * nchunks;
    const int kb = (int)((uint32_t)ks * (uint32_t)g.KT / (uint32_t)S);      // k tiles [kb, ke)
    const int ke = (int)((uint32_t)(ks + 1) * (uint32_t)g.KT / (uint32_t)S);
    const int p0 = chunk * TCH;
    // The projection this row block belongs to: their row blocks are numbered one after the other.  A call of one projection
    // has a kernel of its own, since looking the projection up makes the start 0.4 us longer (15.2 -> 15.6 us at
    // 256 x 1024 x 1024).
    int pj = 0;
    if constexpr (GROUP) {
        while (pj + 1 < gp.P && rb >= gp.rb_start[pj + 1]) ++pj;
    }
    const int rbl = GROUP ? rb - gp.rb_start[pj] : rb;
    const int Np = GROUP ? gp.N[pj] : a.N;
    const int RT = Np >> 4;

    int rtc[TRT];
    bool rvalid[TRT];
#pragma unroll
    for (int r = 0; r < TRT; ++r) {
        const int rt = rbl * (TWR * TRT) + wr * TRT + r;
        rvalid[r] = rt < RT;
        rtc[r] = rvalid[r] ? rt : RT - 1;
    }
    f4 acc[TRT][TJ];
#pragma unroll
    for (int r = 0; r < TRT; ++r)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[r][j] = (f4){0.f, 0.f, 0.f, 0.f};

    // ---- the W and x slices: piece u of a thread is row u * 64 + tid / 8 of the slice, LDS slot
    // tid % 8 of that row, which holds global piece (tid % 8) ^ ((row >> 1) & 7).  A wave's 64
    // lanes cover 8 consecutive rows = 1 KB of LDS in lane order, as the LDS-destination load
    // writes it.  Rows that do not exist get an offset beyond the resource (the hardware reads
    // zeros; whatever lands in LDS for them only reaches output rows that are never stored).
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(GROUP ? gp.W[pj] : a.W, (uint32_t)Np * (uint32_t)a.K * 2u);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (uint32_t)a.T * (uint32_t)a.K * 2u);
    constexpr int WU = (TROWS + 63) / 64, XU = (TCH + 63) / 64;      // pieces per thread
    uint32_t woff[WU], xoff[XU];
#pragma unroll
    for (int u = 0; u < WU; ++u) {
        const int r = u * 64 + (tid >> 3), n = rbl * TROWS + r;
        woff[u] = n < Np ? (uint32_t)n * (uint32_t)a.K * 2u + (uint32_t)((tid & 7) ^ ((r >> 1) & 7)) * 16u : 0x80000000u;
    }
#pragma unroll
    for (int u = 0; u < XU; ++u) {
        const int r = u * 64 + (tid >> 3), t = p0 + r;
        xoff[u] = t < a.T ? (uint32_t)t * (uint32_t)a.K * 2u + (uint32_t)((tid & 7) ^ ((r >> 1) & 7)) * 16u : 0x80000000u;
    }
#define TK_LOAD(buf, step)                                                                                         \
    do {                                                                                                           \
        /* (a slice whose rows are no multiple of 64 ends before the last pieces of the later waves) */            \
        _Pragma("unroll") for (int u = 0; u < WU; ++u)                                                            \
            if (u * 64 + 64 <= TROWS || u * 64 + wave * 8 < TROWS)                                                 \
                to_lds(rw, ws + (buf) * TROWS * TLD + (u * 64 + wave * 8) * TLD, woff[u], (uint32_t)(step) * 128u); \
        _Pragma("unroll") for (int u = 0; u < XU; ++u)                                                            \
            if (u * 64 + 64 <= TCH || u * 64 + wave * 8 < TCH)                                                     \
                to_lds(rx, xs + (buf) * TCH * TLD + (u * 64 + wave * 8) * TLD, xoff[u], (uint32_t)(step) * 128u); \
    } while (0)

    const int s_first = 4 * kb, s_final = 4 * ke - 1;
    TK_LOAD(0, s_first);

    const int sw = (g.row >> 1) & 7;                 // swizzle of this lane's fragment rows (row & 15 decides it)
    const int f0 = (g.q ^ sw) * 8, f1 = ((g.q + 4) ^ sw) * 8;      // slots of k 8q.. and 32 + 8q.. (halfs)
    const int aoff = (wr * TRT * 16 + g.row) * TLD;
    const int boff = (wc * TJ * 16 + g.row) * TLD;
    // One step: wait for the slice, request the next one into the other buffer, multiply.  A
    // workgroup walks a multiple of four steps, so the loop is unrolled by two and the buffer of a
    // step is known at compile time (all LDS addresses become immediates).
    // A wave holds the fragments of the operand of which it has fewer, and streams the other's.
    constexpr bool HOLD_A = TRT <= TJ;
    constexpr int NH = HOLD_A ? TRT : TJ, NM = HOLD_A ? TJ : TRT;
#define TK_STEP(BUF, step)                                                                                         \
    do {                                                                                                           \
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  /* this wave's pieces of slice `step` are in LDS */      \
        lds_barrier();                       /* everybody's are, and slice step - 1 is no longer read */           \
        TK_LOAD((BUF) ^ 1, min((step) + 1, s_final));                                                              \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        const _Float16 *wb = ws + (BUF) * TROWS * TLD;                                                             \
        const _Float16 *xb = xs + (BUF) * TCH * TLD;                                                               \
        const _Float16 *hb = HOLD_A ? wb + aoff : xb + boff, *mb = HOLD_A ? xb + boff : wb + aoff;                 \
        h8 hf[NH][2], mq[2][2];                                                                                    \
        _Pragma("unroll") for (int i = 0; i < NH; ++i) {                                                          \
            hf[i][0] = *(const h8 *)(hb + i * 16 * TLD + f0);                                                      \
            hf[i][1] = *(const h8 *)(hb + i * 16 * TLD + f1);                                                      \
        }                                                                                                          \
        mq[0][0] = *(const h8 *)(mb + f0);                                                                         \
        mq[0][1] = *(const h8 *)(mb + f1);                                                                         \
        mq[1][0] = *(const h8 *)(mb + 16 * TLD + f0);                                                              \
        mq[1][1] = *(const h8 *)(mb + 16 * TLD + f1);                                                              \
        _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                                          \
            const h8 m0 = mq[m & 1][0], m1 = mq[m & 1][1];                                                         \
            if (m + 2 < NM) {                                                                                      \
                mq[m & 1][0] = *(const h8 *)(mb + (m + 2) * 16 * TLD + f0);                                        \
                mq[m & 1][1] = *(const h8 *)(mb + (m + 2) * 16 * TLD + f1);                                        \
            }                                                                                                      \
            _Pragma("unroll") for (int i = 0; i < NH; ++i) {                                                      \
                f4 &c = acc[HOLD_A ? i : m][HOLD_A ? m : i];                                                       \
                c = __builtin_amdgcn_mfma_f32_16x16x32_f16(HOLD_A ? hf[i][0] : m0, HOLD_A ? m0 : hf[i][0], c, 0, 0, 0); \
                c = __builtin_amdgcn_mfma_f32_16x16x32_f16(HOLD_A ? hf[i][1] : m1, HOLD_A ? m1 : hf[i][1], c, 0, 0, 0); \
            }                                                                                                      \
            __builtin_amdgcn_sched_barrier(0);   /* keep the reads two blocks ahead of their MFMAs */               \
        }                                                                                                          \
    } while (0)
    for (int step = s_first; step <= s_final; step += 2) {
        TK_STEP(0, step);
        TK_STEP(1, step + 1);
    }
#undef TK_STEP
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // the last, redundant request has landed too
#undef TK_LOAD

    // ---- k slices of one tile meet in fp32 (as in the narrower tiled kernel): every slice stores
    // its accumulators with agent-scope stores, waits for them and bumps the tile's arrival
    // counter; the last one adds all slices in slice order, 16 loads of each lane in flight at once.
    if (S > 1) {
        constexpr int AGENT = 0x10;
        const uint32_t tile_bytes = (uint32_t)(TRT * TJ) * TTHREADS * 16u;
        const __amdgpu_buffer_rsrc_t prs = make_rsrc(a.partial, (uint32_t)(8 * Tt * S) * tile_bytes);
        const uint32_t lane_off = (uint32_t)tid * 16u;
#pragma unroll
        for (int r = 0; r < TRT; ++r)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[r][j]), prs,
                                                       lane_off + (uint32_t)(r * TJ + j) * TTHREADS * 16u,
                                                       (uint32_t)(slot0 + ks) * tile_bytes, AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            int32_t *ctr = a.counters + (tile - 8 * I0);
            const int old = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int last = (old == S - 1);
            if (last) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
            s_last = last;
        }
        __syncthreads();
        if (!s_last) return;
#pragma unroll
        for (int r = 0; r < TRT; ++r)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[r][j] = (f4){0.f, 0.f, 0.f, 0.f};
        constexpr int NV = TRT * TJ, BATCH = 16;
#pragma unroll 1
        for (int sl = 0; sl < S; ++sl) {
#pragma unroll
            for (int h = 0; h < NV; h += BATCH) {
                f4 v[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
                    if (h + u < NV)
                        v[u] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          prs, lane_off + (uint32_t)(h + u) * TTHREADS * 16u,
                                                          (uint32_t)(slot0 + sl) * tile_bytes, AGENT));
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
                    if (h + u < NV) acc[(h + u) / TJ][(h + u) % TJ] += v[u];
            }
        }
    }
    // ---- results: lane 16q + c holds rows 4q..4q+3 of each row tile for request column c
    _Float16 *out = (_Float16 *)(GROUP ? gp.out[pj] : a.out);
#pragma unroll
    for (int r = 0; r < TRT; ++r) {
        if (!rvalid[r]) continue;
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int tok = p0 + (wc * TJ + j) * 16 + g.row;
            if (tok < a.T) store_row4(out + (size_t)tok * Np + rtc[r] * 16 + 4 * g.q, acc[r][j], a.accumulate);
        }
    }
}

template <int TWR, int TRT, int TJ, bool GROUP>
hipError_t launch_tile(const DzStreamArgs &a, const DzGroup &gp, int NRB, int nchunks, hipStream_t st)
{
    const size_t lds = (size_t)2 * 16 * (TWR * TRT + TW / TWR * TJ) * TLD * sizeof(_Float16);
    static unsigned long long lds_allowed = 0;      // per instantiation
    auto k = tile_kernel<TWR, TRT, TJ, GROUP>;
    const hipError_t e = dz_allow_lds((const void *)k, (int)lds, lds_allowed);
    if (e != hipSuccess) return e;
    const int tail = NRB * nchunks - 8 * a.max_slots;
    const int grid = 8 * (a.max_slots + ((tail + 7) / 8) * a.S);
    hipLaunchKernelGGL(k, dim3(grid), dim3(TTHREADS), lds, st, a, gp, NRB, nchunks);
    return hipGetLastError();
}

// The tile shapes: 256 x 256 and the ones that are smaller in one direction.
struct TileShape {
    int twr, trt, tj;
    int rows() const { return twr * trt * 16; }
    int cols() const { return TW / twr * tj * 16; }
    size_t partial_bytes() const { return (size_t)trt * tj * TTHREADS * 16; }   // of one slice of one tile
};
const TileShape shapes[] = {{4, 4, 8}, {4, 4, 7}, {4, 4, 6}, {4, 4, 5}, {4, 4, 4}, {2, 7, 4}, {2, 6, 4}, {2, 5, 4}};

struct TilePlan {
    const TileShape *shape = nullptr;
    int NRB = 0, nchunks = 0;           // row blocks (of all projections), blocks of request rows
    int S = 1;                          // slices of k of the tiles of the last round
    int whole_per_xcd = 0;              // tiles that run whole, per XCD
    int sliced() const { return 8 * ((int)((long long)NRB * nchunks - 8 * whole_per_xcd + 7) / 8); }
    size_t partial_bytes() const { return (size_t)sliced() * S * shape->partial_bytes(); }
};

template <bool GROUP>
hipError_t launch_shape(const TileShape &t, const DzStreamArgs &a, const DzGroup &gp, int NRB, int nchunks, hipStream_t st)
{
    if (t.twr == 4) {
        switch (t.tj) {
        case 8: return launch_tile<4, 4, 8, GROUP>(a, gp, NRB, nchunks, st);
        case 7: return launch_tile<4, 4, 7, GROUP>(a, gp, NRB, nchunks, st);
        case 6: return launch_tile<4, 4, 6, GROUP>(a, gp, NRB, nchunks, st);
        case 5: return launch_tile<4, 4, 5, GROUP>(a, gp, NRB, nchunks, st);
        default: return launch_tile<4, 4, 4, GROUP>(a, gp, NRB, nchunks, st);
        }
    }
    switch (t.trt) {
    case 7: return launch_tile<2, 7, 4, GROUP>(a, gp, NRB, nchunks, st);
    case 6: return launch_tile<2, 6, 4, GROUP>(a, gp, NRB, nchunks, st);
    default: return launch_tile<2, 5, 4, GROUP>(a, gp, NRB, nchunks, st);
    }
}

}  // namespace

// Does the wide kernel take this call?  Base products only, requests in their own order, and every
// real byte offset below 2^31 (its missing-row trick uses the upper half of the offset range).
bool dz_tile_fits(const DzStreamArgs &a, const DzGroup &gp)
{
    if (!a.has_base || a.has_delta || a.perm != nullptr) return false;
    for (int p = 0; p < gp.P; ++p)
        if ((unsigned long long)gp.N[p] * a.K * 2ull >= (1ull << 31)) return false;
    return (unsigned long long)a.T * a.K * 2ull < (1ull << 31);
}

// Tiles of a call: one workgroup per CU, the tiles of the full rounds whole, those of the last, partly filled round cut
// into up to eight slices of k, of two k tiles at least, as many as still fit the CUs at once and `room` bytes of partial
// tiles.  Of the shapes the call takes the one with the least estimated time.  The estimate is in us, from measurements on
// a full chip: a step takes 0.75 + 0.87 times the tile's area in units of 256 x 256 (1.61 for 256 x 256, 1.51 for 224 x 256,
// 1.30 for 160 x 256), a round some 6 more for its start and end, and a meeting moves the partial tiles of all slices twice.
// With slices of the smaller shapes even one tile fills the chip: 128 x 1024 x 8192 39.9 us in slices of the narrower
// kernel, 29.8 here.  T = 2048: 5120 x 5120 139 us with 256 x 256 tiles (160 for 256 CUs), 107 with 160 x 256 (256);
// 13824 x 5120 272 us with 256 x 256 (432: the second round is 69 % full), 257 with 224 x 256 (496).
static TilePlan plan_tiles(int P, const int *N, int T, int K, int cus, int force_splits, size_t room)
{
    TilePlan best;
    double best_cost = 0;
    const int n = cus > 0 ? cus : 256;
    for (const TileShape &t : shapes) {
        int rb = 0;                     // row blocks of all projections; a row block never spans two
        for (int p = 0; p < P; ++p) rb += (N[p] + t.rows() - 1) / t.rows();
        const int ch = (T + t.cols() - 1) / t.cols();
        const long long tiles = (long long)rb * ch;
        if (tiles > 0x3fffffff) continue;
        int S = 1;
        long long whole = tiles;
        if (force_splits > 0) {
            S = force_splits; whole = 0;
        } else if (cus >= 8 && tiles % cus != 0) {
            const int tail = (int)(tiles % cus), sliced = (tail + 7) / 8 * 8;       // (dealt out to the XCDs in eights)
            const int fit = std::min({cus / sliced, 8, K / 512, (int)(room / ((size_t)sliced * t.partial_bytes()))});
            if (fit > 1) { S = fit; whole = tiles - tail; }
        }
        const double area = t.rows() * t.cols() / 65536.0, step = 0.75 + 0.87 * area;
        double cost = (double)((whole + n - 1) / n) * (step * (K / 64) + 6.0);
        if (whole < tiles) cost += step * ((K / 64 + S - 1) / S) + 6.0 + 5.0 * S * area * ((double)(tiles - whole) * S / n);
        if (!best.shape || cost < best_cost) {
            best_cost = cost;
            best.shape = &t; best.NRB = rb; best.nchunks = ch; best.S = S;
            best.whole_per_xcd = S > 1 ? (int)(whole / 8) : (int)((tiles + 7) / 8);
        }
    }
    return best;
}

// The plan of a call with 64 MB of room, for tests without a GPU: {waves along the rows, row tiles and column blocks of a
// wave, k slices, tiles that run whole, tiles}.
extern "C" void dz_tile_plan(int P, const int *N, int T, int K, int cus, int *plan)
{
    const TilePlan t = plan_tiles(P, N, T, K, cus, 0, (size_t)64 << 20);
    if (!t.shape) return;
    const int tiles = t.NRB * t.nchunks;
    const int v[6] = {t.shape->twr, t.shape->trt, t.shape->tj, t.S, std::min(8 * t.whole_per_xcd, tiles), tiles};
    for (int i = 0; i < 6; ++i) plan[i] = v[i];
}

int dz_launch_tile(dz_ctx *ctx, const DzStreamArgs &args, const DzGroup &group, hipStream_t st)
{
    DzStreamArgs a = args;
    DzGroup gp = group;
    if (!dz_tile_fits(a, gp)) return DZ_ERR_SHAPE;
    int cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    cus -= cus % 8;
    // The partial tiles of a call take up to 64 MB, twice what dz_create makes room for.  A call that is being captured
    // into a graph without an eager call before it cannot grow the workspace: it takes the best split that fits.
    TilePlan plan = plan_tiles(gp.P, gp.N, a.T, a.K, cus, ctx->force_splits, (size_t)64 << 20);
    if (plan.shape && plan.S > 1 && plan.partial_bytes() > ctx->partial_bytes) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        const hipError_t e = hipStreamIsCapturing(st, &cs);
        if (e != hipSuccess) return dz_set_hip_error(ctx, e);
        if (cs != hipStreamCaptureStatusNone && ctx->force_splits == 0)
            plan = plan_tiles(gp.P, gp.N, a.T, a.K, cus, 0, ctx->partial_bytes);
    }
    if (!plan.shape) return DZ_ERR_SHAPE;
    const TileShape &shape = *plan.shape;
    gp.rb_start[0] = 0;
    for (int p = 0; p < DZ_MAX_GROUP; ++p)
        gp.rb_start[p + 1] = gp.rb_start[p] + (p < gp.P ? (gp.N[p] + shape.rows() - 1) / shape.rows() : 0);
    const int tiles = plan.NRB * plan.nchunks;
    if (plan.S > a.K / 256) plan.S = a.K / 256;
    if (plan.S > 1 && plan.partial_bytes() >= ((size_t)1 << 32)) plan.S = 1;     // 32-bit byte offsets
    if (plan.S <= 1) { plan.S = 1; plan.whole_per_xcd = (tiles + 7) / 8; }
    if (plan.S > 1) {
        int rc = dz_ensure_partial(ctx, plan.partial_bytes(), st);
        if (rc == DZ_OK) rc = dz_ensure_counters(ctx, plan.sliced(), st);
        if (rc != DZ_OK) return rc;
    }
    a.S = plan.S;
    a.max_slots = plan.whole_per_xcd;
    a.partial = ctx->partial;
    a.counters = ctx->counters;
    if (gp.P > 1) return dz_set_hip_error(ctx, launch_shape<true>(shape, a, gp, plan.NRB, plan.nchunks, st));
    a.N = gp.N[0]; a.W = gp.W[0]; a.out = gp.out[0];
    return dz_set_hip_error(ctx, launch_shape<false>(shape, a, gp, plan.NRB, plan.nchunks, st));
}
