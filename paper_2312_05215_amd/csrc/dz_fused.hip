// The fused kernel for prompt-sized batches of long segments: base GEMM + SBMM + merge.
//
//   out[t] = f16( x[t] . W^T + x[t] . Delta_{Idx[t]}^T )      (paper Section 5.1 Eq. (2); Section 5.2)
//
// Where a delta has dozens of request rows the product is bound by the matrix pipes.  The narrower tiled kernel keeps them 40 %
// busy on a 13B layer of T = 2048 and 16 deltas: its 256 x 128 tile brings in a byte of W per 128 request rows, straight from
// global memory in 64-byte pieces, and dequantises a packed tile for every segment of each 128 rows.  Here
//   * a workgroup (8 waves) owns 256 rows of N x up to 256 request rows; a wave owns 2 row tiles x 16 column blocks (128
//     accumulator registers), so a packed tile is dequantised once for all its columns, and every fragment of x that a
//     wave reads from LDS feeds four dense and two sparse MFMAs;
//   * column tiles follow the segments: one or two segments each, every segment at an even column block of its own.  No
//     column block is shared, so no product is masked; columns without a request are zeros that are never stored.  The
//     segment pass leaves the list of tiles in the workspace (DzFusedTile): the host does not know it, and starts as many
//     workgroups as there can be tiles;
//   * W and x travel to LDS by loads with an LDS destination, 64 columns of k at a time.  A wave reads its own rows of W into
//     registers at the start of a step and refills them at once; x has three buffers;
//   * the eight waves are two groups, one on each SIMD, half a step apart: while one multiplies, the other reads its
//     fragments, dequantises and requests the next slices (a request moves 1 KB and holds its wave up for some 90 cycles,
//     64 of them a step).  One barrier ends each half;
//   * packed tiles wait in stage registers, loaded a step before they are needed.
// us, 13824 x 5120, T = 2048, narrower kernel -> here (medians of seven turns): one delta 438 -> 384 (the rule below still leaves
// that call to the narrower kernel), 8 segments of 256 rows 459 -> 402, 16 of 128 469 -> 434, 16 random ones 517 -> 483.  The launches
// of that 13B layer: q,k,v 662 -> 613, o 233 -> 218, gate,up 1151 -> 1087, down 577 -> 530; of a 7B layer of 777 rows and three 2-bit
// deltas, which the rule leaves to the narrower kernel: 168 -> 153, 70 -> 70, 281 -> 257, 158 -> 137.  On the 13B layer the pipes are
// busy 44 % of the time at some 1.9 GHz (nominal 2.4), waves wait for operands 34 % of theirs, and a launch moves 2.1 GB (2.5 before).
#include "dz_mma.h"
#include <algorithm>
#include <cmath>


namespace {

constexpr int FW = 8;                   // waves per workgroup
constexpr int FTHREADS = FW * 64;
constexpr int FR = 2;                   // row tiles of a wave
constexpr int FROWS = FW * FR * 16;     // rows of N per tile
constexpr int FJ = DZ_FUSED_BLOCKS;     // column blocks of 16 request rows per tile, at most
constexpr int FCH = 16 * FJ;
constexpr int FPB = 3;                  // column blocks whose fragments of x are in registers or on their way there
constexpr int FLD = 64;                 // LDS row stride in halfs of a 64-k slice (no padding: see the swizzle)
constexpr int FXB = 3;                  // x buffers
static_assert(FJ == 16, "four pieces of x per wave; the step is written out for it");

__device__ __forceinline__ void to_lds(__amdgpu_buffer_rsrc_t rs, _Float16 *lds, uint32_t voff, uint32_t soff)
{
    typedef __attribute__((address_space(3))) void lds_void;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)lds, 16, voff, soff, 0, 0);
}

__device__ __forceinline__ void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

constexpr int WAIT_VM(int n) { return 0x0F70 | n; }      // s_waitcnt vmcnt(n), n < 16
constexpr int WAIT_LDS = 0xC07F;        // s_waitcnt lgkmcnt(0)

// A step's operands from the stage registers (step_dequant).  The scale pair goes through an opaque copy: shared between the
// steps of a quantisation group, what is derived from it would stay in 8 to 32 registers that are not there.
template <int BITS, int GROUP, int R>
__device__ __forceinline__ void fused_dequant(const uint32_t (&st)[R][Fmt<BITS, GROUP, false>::SD], int s, h8 (&av)[R], uint32_t (&ix)[R])
{
    typedef Fmt<BITS, GROUP, false> F;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t sz = st[r][F::SC0 + s * F::GPT / 4];
        asm volatile("" : "+v"(sz));
        const h2 sz2 = as_h2(sz);
        const uint32_t w = step_codes<BITS, false>(st[r], s, 0, ix[r]);
        av[r] = dequant_step<BITS>(w, (h2){sz2.x, sz2.x}, (h2){sz2.y, sz2.y});
    }
}

// Into how many slices of k to cut each of the tiles that are left after the full rounds of one tile per CU: the number that
// gives the least estimated time `est`, in units of dz_fused_cost and steps.  The slices themselves may take two rounds (160 tiles
// in thirds are two rounds of thirds, where 160 whole ones or 320 halves take as long as 256 tiles).  70 is a start and an
// end, and a meeting reads and writes every slice's partial tile.
__host__ __device__ inline int tail_slices(int left, int KT, int cus, int slots, float most, float &est)
{
    const int tail = (left + 7) / 8 * 8;                // (dealt out to the XCDs in eights)
    const float steps = 4.f * (float)KT;
    int S = 1;
    est = left ? most * steps + 70.f : 0.f;
    for (int s = 2; s <= 8; ++s) {
        if (s > KT / 2 || tail * s > (2 * cus < slots ? 2 * cus : slots)) break;
        const float e = (tail * s > cus ? 2.f : 1.f) * (most * steps / (float)s + 70.f) + 30.f + 2.4f * (float)s * most;
        if (left && e < est) { est = e; S = s; }
    }
    return S;
}

template <int BITS, int GROUP>
__global__ __launch_bounds__(FTHREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void fused_kernel(DzStreamArgs a, DzGroup gp, DzGroupPtrs dp, const DzFusedTile *__restrict__ plan, int NRB, int cus, int slots)
{
    typedef Fmt<BITS, GROUP, false> F;
    constexpr int SD = F::SD;
    extern __shared__ __attribute__((aligned(128))) _Float16 lds[];    // W: [FROWS][FLD]; x: FXB x [FCH][FLD]
    _Float16 *const ws = lds;
    _Float16 *const xs = lds + FROWS * FLD;
    __shared__ int s_tok[256];              // request row of each column (-1: none)
    __shared__ uint32_t s_xoff[256];        // and where it begins in x, past the end for none
    __shared__ int s_last;

    const int tid = threadIdx.x;
    Geo g;
    g.lane = tid & 63; g.row = g.lane & 15; g.q = g.lane >> 4;
    g.KT = a.K >> 8;
    g.LDW = FLD;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int late = wave / (FW / 2);        // 1: this wave's group runs one phase behind the other

    // ---- the tile of this workgroup: whole tiles first, XCD by XCD (column tiles fastest, so that the tiles of a row block share
    // the XCD's L2 copy of the W rows), then the tiles of the last, partly filled round cut into S slices of k
    const int nt = plan[0].start0;
    const int tiles = NRB * nt;
    float est;
    int S = tail_slices(tiles % cus, g.KT, cus, slots, (float)plan[0].rows0, est);
    const int I0 = S > 1 ? tiles / cus * cus / 8 : (tiles + 7) / 8;
    const int Tt = (tiles - 8 * I0 + 7) / 8;            // sliced tiles per XCD
    const int xcd = (int)(blockIdx.x % 8), bi = (int)(blockIdx.x / 8);
    int tile, ks = 0;
    if (bi < I0) {
        tile = xcd * I0 + bi;
        if (tile >= tiles) return;
        S = 1;
    } else {
        const int tt = (bi - I0) / S;
        ks = (bi - I0) - tt * S;
        tile = 8 * I0 + xcd * Tt + tt;
        if (tt >= Tt || tile >= tiles) return;
    }
    tile = __builtin_amdgcn_readfirstlane(tile);
    ks = __builtin_amdgcn_readfirstlane(ks);
    S = __builtin_amdgcn_readfirstlane(S);
    const int slot0 = (tile - 8 * I0) * S;
    const int rb = tile / nt;
    const DzFusedTile ct = plan[1 + tile - rb * nt];
    const int kb = (int)((uint32_t)ks * (uint32_t)g.KT / (uint32_t)S);      // k tiles [kb, ke)
    const int ke = (int)((uint32_t)(ks + 1) * (uint32_t)g.KT / (uint32_t)S);
    // column blocks: of the first segment (an even number where a second one follows), of both, and that rounded up to an even
    // number; and the first block at which something happens
    const int nb0 = ct.rows1 > 0 ? ((ct.rows0 + 31) >> 5) * 2 : (ct.rows0 + 15) >> 4;
    const int nb = nb0 + ((ct.rows1 + 15) >> 4), nbe = (nb + 1) & ~1;
    const int nbs = ct.rows1 > 0 ? nb0 : nbe;
    const bool v0 = ct.key0 < a.D, v1 = ct.rows1 > 0;       // (rows of the base model share no tile with others)
    int pj = 0;
    while (pj + 1 < gp.P && rb >= gp.rb_start[pj + 1]) ++pj;
    const int rbl = rb - gp.rb_start[pj];
    const int Np = gp.N[pj];
    const int RT = Np >> 4;
    const uint32_t off_idx = gp.off_idx[pj], off_scale = gp.off_scale[pj], blob_bytes = gp.blob_total[pj];

    const __amdgpu_buffer_rsrc_t rw = make_rsrc(gp.W[pj], (uint32_t)Np * (uint32_t)a.K * 2u);
    // W: piece u of a wave is rows 8 (u % 2) .. + 7 of its row tile u / 2; rows past the end of N repeat the last row tile
    int rtc[FR];
    bool rvalid[FR];
#pragma unroll
    for (int r = 0; r < FR; ++r) {
        const int rt = rbl * (FW * FR) + wave * FR + r;
        rvalid[r] = rt < RT;
        rtc[r] = rvalid[r] ? rt : RT - 1;
    }
    const uint32_t woff = (uint32_t)(g.lane >> 3) * (uint32_t)a.K * 2u + (uint32_t)((g.lane & 7) ^ (g.lane >> 4)) * 16u;
    // (the LDS address is rebuilt from one scalar: kept for every piece and buffer they would spill)
#define FU_W(step, u)                                                                                              \
    do {                                                                                                           \
        int w_ = wave * FR * 16 * FLD;                                                                             \
        asm volatile("" : "+s"(w_));                                                                               \
        to_lds(rw, ws + w_ + (u) * 8 * FLD, ((u) & 1) ? woff ^ 64u : woff,                                         \
               ((uint32_t)rtc[(u) >> 1] * 16u + ((u) & 1) * 8u) * (uint32_t)a.K * 2u + (uint32_t)(step) * 128u);       \
    } while (0)
#define FU_X(buf, step, u)                                                                                         \
    do {                                                                                                           \
        int w_ = wave * 8 * FLD;                                                                                   \
        asm volatile("" : "+s"(w_));                                                                               \
        to_lds(rx, xs + w_ + ((buf) * FCH + (u) * 64) * FLD, xo_[u] + xpiece, (uint32_t)(step) * 128u); \
    } while (0)
    const int s_final = 4 * ke - 1;
#pragma unroll
    for (int u = 0; u < 4; ++u) FU_W(4 * kb, u);

    // ---- packed tiles: one set of stage registers per segment of the tile
    const void *d0 = v0 ? dp.p[pj * a.D + ct.key0] : a.x, *d1 = v1 ? dp.p[pj * a.D + ct.key1] : a.x;
    const __amdgpu_buffer_rsrc_t rd0 = make_rsrc(d0, v0 ? blob_bytes : 0u), rd1 = make_rsrc(d1, v1 ? blob_bytes : 0u);
    uint32_t st[2][FR][SD];
#define FU_STAGE(d, kt)                                                                                            \
    do {                                                                                                           \
        uint32_t ln_ = (uint32_t)g.lane;            /* offsets worked out anew, once a k tile, to save registers */ \
        asm volatile("" : "+v"(ln_));                                                                              \
        LaneOffs lo;                                                                                               \
        lo.c = ln_ * 16u; lo.i = ln_ * 8u; lo.s = (ln_ & 15u) * (uint32_t)(F::GPT * 4);                            \
        _Pragma("unroll") for (int r = 0; r < FR; ++r)                                                            \
            tile_loads<BITS, GROUP, false>((d) ? rd1 : rd0, (uint32_t)rtc[r] * (uint32_t)g.KT + (uint32_t)(kt), lo, off_idx, off_scale, st[d][r]); \
    } while (0)
    FU_STAGE(0, kb);
    FU_STAGE(1, kb);

    // ---- request rows of the tile's columns: each segment starts at a column block of its own
    if (tid < 256) {
        const bool second = tid >= 16 * nb0;
        const int i = second ? tid - 16 * nb0 : tid;
        const bool there = i < (second ? ct.rows1 : ct.rows0);
        const int tok = there ? a.perm[(second ? ct.start1 : ct.start0) + i] : -1;
        s_tok[tid] = tok;
        s_xoff[tid] = there ? (uint32_t)tok * (uint32_t)a.K * 2u : 0x80000000u;
    }
    lds_barrier();
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, (uint32_t)a.T * (uint32_t)a.K * 2u);
    // piece u of a wave: rows u * 64 + wave * 8 .. + 7
    const int xrow = wave * 8 + (g.lane >> 3);
    const uint32_t xpiece = (uint32_t)((g.lane & 7) ^ ((xrow >> 1) & 7)) * 16u;
    uint32_t xo_[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) xo_[u] = s_xoff[u * 64 + xrow];
#pragma unroll
    for (int u = 0; u < 4; ++u) { FU_X(0, 4 * kb, u); FU_X(1, 4 * kb + 1, u); }

    f4 acc[FR][FJ];
#pragma unroll
    for (int r = 0; r < FR; ++r)
#pragma unroll
        for (int j = 0; j < FJ; ++j) acc[r][j] = (f4){0.f, 0.f, 0.f, 0.f};

    const int sw = (g.row >> 1) & 7;                 // swizzle of this lane's fragment rows (row & 15 decides it)
    // a lane's fragment in the first 16 rows: k 8q .. in slot q ^ sw, k 32 + 8q .. in slot (q + 4) ^ sw, 64 bytes across
    const int frag = g.row * FLD + (g.q ^ sw) * 8;
    h8 af[FR][2], av[2][FR];
    uint32_t ix[2][FR];
    h16 bq[FPB];
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int r = 0; r < FR; ++r) { av[d][r] = (h8)(_Float16)0.f; ix[d][r] = 0u; }
    const int px = (nb + 3) / 4;                     // pieces of x this wave requests per step
    int xb = 0;                                      // the x buffer of the step at hand

    __builtin_amdgcn_s_waitcnt(0);
    phase_barrier();
    if (late) phase_barrier();

#define FU_READ_A()                                                                                                \
    do {                                                                                                           \
        _Pragma("unroll") for (int r = 0; r < FR; ++r) {                                                          \
            af[r][0] = *(const h8 *)(ws + (wave * FR + r) * 16 * FLD + frag);                                      \
            af[r][1] = *(const h8 *)(ws + (wave * FR + r) * 16 * FLD + (frag ^ 32));                               \
        }                                                                                                          \
    } while (0)
#define FU_READ_B(j)                                                                                               \
    do {                                                                                                           \
        const h8 l_ = *(const h8 *)(xr0 + (j) * 16 * FLD), h_ = *(const h8 *)(xr1 + (j) * 16 * FLD);               \
        bq[(j) % FPB] = __builtin_shufflevector(l_, h_, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);     \
    } while (0)
    // Two column blocks.  A wave's MFMAs leave no time for branches (one per block lengthened it from 104 to 150 cycles), so
    // there is one comparison for the two: with the next block at which something happens, the first of the second
    // segment, whose operands then replace the first one's, or the one past the last, where the step ends.  The comparison is
    // made there, on a scalar the compiler cannot see through: made once for all steps it would be a lane mask, and spill.
#define FU_PAIR(j, ODD, HD, END)                                                                                   \
    do {                                                                                                           \
        if ((j) > 0) {                                                                                             \
            asm volatile("" : "+s"(event));                                                                        \
            if (__builtin_expect((j) == event, 0)) {                                                               \
                if ((j) >= nb) goto END;                                                                           \
                event = nbe;                                                                                       \
                if (HD) {                                                                                          \
                    _Pragma("unroll") for (int r = 0; r < FR; ++r) { av[0][r] = av[1][r]; ix[0][r] = ix[1][r]; }  \
                }                                                                                                  \
            }                                                                                                      \
        }                                                                                                          \
        _Pragma("unroll") for (int j_ = (j); j_ < (j) + 2; ++j_) {                                                \
            const h16 b = bq[j_ % FPB];                                                                            \
            const h8 b0 = __builtin_shufflevector(b, b, 0, 1, 2, 3, 4, 5, 6, 7);                                   \
            const h8 b1 = __builtin_shufflevector(b, b, 8, 9, 10, 11, 12, 13, 14, 15);                             \
            _Pragma("unroll") for (int r = 0; r < FR; ++r)                                                        \
                acc[r][j_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[r][0], b0, acc[r][j_], 0, 0, 0);            \
            _Pragma("unroll") for (int r = 0; r < FR; ++r)                                                        \
                acc[r][j_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[r][1], b1, acc[r][j_], 0, 0, 0);            \
            if (HD) {                                                                                              \
                _Pragma("unroll") for (int r = 0; r < FR; ++r)                                                    \
                    acc[r][j_] = smfmac<ODD>(av[0][r], b, acc[r][j_], (int)ix[0][r]);                              \
            }                                                                                                      \
            __builtin_amdgcn_sched_barrier(0);      /* the fragments are read blocks ahead of their MFMAs */        \
            if (j_ + FPB < FJ) FU_READ_B(j_ + FPB);                                                                \
            __builtin_amdgcn_sched_barrier(0);                                                                     \
        }                                                                                                          \
    } while (0)
#define FU_STEP(s_, HD, kt, END)                                                                                   \
    {                                                                                                              \
        const int wn = min(4 * (kt) + (s_) + 1, s_final), xn = min(4 * (kt) + (s_) + 1 + late, s_final);           \
        const int xf = xb + 1 + late, xfree = xf >= FXB ? xf - FXB : xf;                                           \
        const _Float16 *const xr0 = xs + xb * FCH * FLD + frag, *const xr1 = xs + xb * FCH * FLD + (frag ^ 32);    \
        int event = nbs, px_ = px;                                                                                 \
        asm volatile("" : "+s"(event), "+s"(px_));                                                                 \
        {                                                                                                          \
            uint32_t xo_[4];                                                                                       \
            _Pragma("unroll") for (int u = 0; u < 4; ++u) xo_[u] = s_xoff[u * 64 + xrow];                         \
            __builtin_amdgcn_sched_barrier(0);                                                                     \
            FU_READ_A();                                                                                           \
            __builtin_amdgcn_sched_barrier(0);                                                                     \
            FU_X(xfree, xn, 0);                                                                                    \
            if (px_ > 1) FU_X(xfree, xn, 1);                                                                       \
            if (px_ > 2) FU_X(xfree, xn, 2);                                                                       \
            if (px_ > 3) FU_X(xfree, xn, 3);                                                                       \
        }                                                                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        if (HD) fused_dequant<BITS, GROUP, FR>(st[0], s_, av[0], ix[0]);                                           \
        if (HD && event < nbe) fused_dequant<BITS, GROUP, FR>(st[1], s_, av[1], ix[1]);                            \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);   /* this wave has read its rows of W out of the buffer */           \
        _Pragma("unroll") for (int j = 0; j < FPB; ++j) FU_READ_B(j);                                             \
        FU_W(wn, 0);                                                                                               \
        FU_W(wn, 1);                                                                                               \
        FU_W(wn, 2);                                                                                               \
        FU_W(wn, 3);                                                                                               \
        phase_barrier();                                                                                           \
        FU_PAIR(0, (s_) & 1, HD, END);                                                                             \
        if (HD && (s_) == 3) {                  /* the stage registers are free: request the next packed tiles */  \
            FU_STAGE(0, min((kt) + 1, ke - 1));                                                                    \
            FU_STAGE(1, min((kt) + 1, ke - 1));                                                                    \
        }                                                                                                          \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        FU_PAIR(2, (s_) & 1, HD, END);                                                                             \
        FU_PAIR(4, (s_) & 1, HD, END);                                                                             \
        FU_PAIR(6, (s_) & 1, HD, END);                                                                             \
        FU_PAIR(8, (s_) & 1, HD, END);                                                                             \
        FU_PAIR(10, (s_) & 1, HD, END);                                                                            \
        FU_PAIR(12, (s_) & 1, HD, END);                                                                            \
        FU_PAIR(14, (s_) & 1, HD, END);                                                                            \
    END:                                                                                                           \
        __builtin_amdgcn_sched_barrier(0);                                                                         \
        __builtin_amdgcn_s_waitcnt(WAIT_VM(0));                                                                    \
        phase_barrier();                                                                                           \
        xb = xb == FXB - 1 ? 0 : xb + 1;                                                                           \
    }
    if (ct.key0 < a.D) {
        for (int kt = kb; kt < ke; ++kt) {
            FU_STEP(0, true, kt, end_d0)
            FU_STEP(1, true, kt, end_d1)
            FU_STEP(2, true, kt, end_d2)
            FU_STEP(3, true, kt, end_d3)
        }
    } else {                    // request rows of the base model alone
        for (int kt = kb; kt < ke; ++kt) {
            FU_STEP(0, false, kt, end_b0)
            FU_STEP(1, false, kt, end_b1)
            FU_STEP(2, false, kt, end_b2)
            FU_STEP(3, false, kt, end_b3)
        }
    }
    if (!late) phase_barrier();
    __builtin_amdgcn_s_waitcnt(0);              // the last, redundant requests have landed too
#undef FU_STEP
#undef FU_PAIR
#undef FU_READ_A
#undef FU_READ_B
#undef FU_STAGE
#undef FU_W
#undef FU_X

    // ---- k slices of one tile meet in fp32, as in the other tiled kernels
    if (S > 1) {
        constexpr int AGENT = 0x10;
        constexpr uint32_t tile_bytes = (uint32_t)(FR * FJ) * FTHREADS * 16u;
        const __amdgpu_buffer_rsrc_t prs = make_rsrc(a.partial, (uint32_t)(8 * Tt * S) * tile_bytes);
        const uint32_t lane_off = (uint32_t)tid * 16u;
#pragma unroll
        for (int j = 0; j < FJ; ++j)
            if (j < nb)
#pragma unroll
                for (int r = 0; r < FR; ++r)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[r][j]), prs,
                                                           lane_off + (uint32_t)(j * FR + r) * FTHREADS * 16u,
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
        for (int r = 0; r < FR; ++r)
#pragma unroll
            for (int j = 0; j < FJ; ++j) acc[r][j] = (f4){0.f, 0.f, 0.f, 0.f};
        constexpr int NV = FR * FJ, BATCH = 16;
        static_assert(NV % BATCH == 0, "batches");
        const uint32_t used = (uint32_t)(nb * FR) * FTHREADS * 16u;         // pieces of blocks that are not there read nothing
#pragma unroll 1
        for (int sl = 0; sl < S; ++sl) {
#pragma unroll
            for (int h = 0; h < NV; h += BATCH) {
                f4 v[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const uint32_t o = lane_off + (uint32_t)(h + u) * FTHREADS * 16u;
                    v[u] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(prs, o < used ? o : 0x80000000u,
                                                                                       (uint32_t)(slot0 + sl) * tile_bytes, AGENT));
                }
#pragma unroll
                for (int u = 0; u < BATCH; ++u) acc[(h + u) % FR][(h + u) / FR] += v[u];
            }
        }
    }
    // ---- results: lane 16q + c holds rows 4q..4q+3 of each row tile for request column c
    _Float16 *out = (_Float16 *)gp.out[pj];
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
        if (j >= nb) continue;
        const int tok = s_tok[16 * j + g.row];
#pragma unroll
        for (int r = 0; r < FR; ++r)
            if (tok >= 0 && rvalid[r]) store_row4(out + (size_t)tok * Np + rtc[r] * 16 + 4 * g.q, acc[r][j], 0);
    }
}

template <int BITS, int GROUP>
hipError_t launch_fused(const DzStreamArgs &a, const DzGroup &gp, const DzGroupPtrs &dp, const DzFusedTile *plan, int NRB, int cus,
                        int slots, int grid, hipStream_t st)
{
    const size_t lds = (size_t)(FROWS + FXB * FCH) * FLD * sizeof(_Float16);
    static unsigned long long lds_allowed = 0;      // per instantiation
    auto k = fused_kernel<BITS, GROUP>;
    const hipError_t e = dz_allow_lds((const void *)k, (int)lds, lds_allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(grid), dim3(FTHREADS), lds, st, a, gp, dp, plan, NRB, cus, slots);
    return hipGetLastError();
}

}  // namespace

// Estimated times of a call here and in the narrower kernel, in units of dz_fused_cost and steps.  The host knows T and D and
// not the segments: it takes them to fill tiles of 16 blocks to nine tenths.  A step of the narrower kernel's tile of 128
// columns takes 13 units where one segment has all of them, and up to 9 more the more of the tiles are mixed.
static float fused_estimate(int NRB, int T, int D, int KT, int cus, int more)
{
    const float blocks = (float)T / 16.f + 0.75f * (float)D;
    const int n = std::max((int)std::ceil(blocks / (0.9f * DZ_FUSED_BLOCKS)), (D + 1) / 2) + more;
    const int wide = std::min(DZ_FUSED_BLOCKS, (int)std::ceil(blocks / (float)n));
    const long long M = (long long)NRB * n;
    float e;
    (void)tail_slices((int)(M % cus), KT, cus, 2 * cus, (float)dz_fused_cost(std::min(DZ_FUSED_BLOCKS, wide + 2)), e);
    return e + (float)(M / cus) * ((float)(4 * KT * dz_fused_cost(wide)) + 70.f);
}

static float narrow_estimate(int NRB, int T, int D, int KT, int cus)
{
    const int ch = (T + 127) / 128;
    const long long M = (long long)NRB * ch;
    const float step = 13.f + 6.f * std::min(1.5f, (float)(D - 1) / (float)ch), steps = 4.f * (float)KT;
    float e = (float)(M / cus) * (step * steps + 50.f);
    if (const int left = (int)(M % cus)) {
        const int S = std::min({cus / ((left + 7) / 8 * 8), 16, KT / 2});
        e += S > 1 ? step * steps / (float)S + 70.f + 20.f * (float)S : step * steps + 50.f;
    }
    return e;
}

// Does the fused kernel take this call?  Base and 2:4 deltas, every byte offset of W and x below 2^31 (a missing row is an
// offset in the upper half), the number of k slices not given, 128 request rows a delta at least (half a tile: two segments of
// that size fill one), and an estimate 5 % below the narrower kernel's, also with two column tiles more than even segments need:
// the host does not know the segments' lengths, and uneven ones are what made looser rules wrong.  Chosen on 344 random sizes
// (T = 65 to 2048, up to 32 deltas) and checked on 355 others: of those it sends 46 here, 0.86 times the narrower kernel's time in the
// geometric mean, two of them slower (1127 x 5120 x 5120, eight uneven deltas, 151 us there and 157 here, is the worst).  64 rows
// a delta and 10 %, without the two tiles, takes 155 of the 355, but 28 of them are slower, the worst 1.40 times.
// DZ_OPT_WIDE_TILE = 2 leaves the estimate out.
bool dz_fused_takes(const dz_ctx *ctx, const DzStreamArgs &a, const DzGroup &gp)
{
    if (!ctx->tile_kernel || ctx->force_splits > 0 || !a.has_base || !a.has_delta || a.quant_only || a.T <= 64) return false;
    if (a.D > DZ_MAX_DELTAS || (unsigned long long)a.T * a.K * 2ull >= (1ull << 31)) return false;
    long long NRB = 0;
    for (int p = 0; p < gp.P; ++p) {
        if ((unsigned long long)gp.N[p] * a.K * 2ull >= (1ull << 31)) return false;
        NRB += (gp.N[p] + FROWS - 1) / FROWS;
    }
    if (NRB * dz_fused_tiles_max(a.T, a.D) > 0x3fffffff) return false;
    if (ctx->tile_kernel == 2) return true;
    int cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    cus = std::max(cus - cus % 8, 8);
    if (a.T < 128 * a.D) return false;
    const int KT = a.K / 256;
    const float e = std::max(fused_estimate((int)NRB, a.T, a.D, KT, cus, 0), fused_estimate((int)NRB, a.T, a.D, KT, cus, 2));
    return e < 0.95f * narrow_estimate((int)NRB, a.T, a.D, KT, cus);
}

// Does a call of base and 2:4 deltas with the default options come here?  For callers that name the kernel they time.
extern "C" int dz_fused_route(int P, const int *N, int T, int K, int D, int cus)
{
    if (P < 1 || P > DZ_MAX_GROUP) return 0;
    dz_ctx ctx;
    ctx.num_cus = cus;
    DzStreamArgs a = {};
    a.T = T; a.K = K; a.D = D;
    a.has_base = 1; a.has_delta = D > 0;
    DzGroup gp = {};
    gp.P = P;
    for (int p = 0; p < P; ++p) gp.N[p] = N[p];
    return dz_fused_takes(&ctx, a, gp) ? 1 : 0;
}

int dz_launch_fused(dz_ctx *ctx, const DzStreamArgs &args, const DzGroup &group, const DzGroupPtrs &dp, hipStream_t st)
{
    DzStreamArgs a = args;
    DzGroup gp = group;
    int NRB = 0;                            // row blocks of all projections; a row block never spans two
    for (int p = 0; p < gp.P; ++p) {
        const DzLayout L = dz_make_layout(gp.N[p], a.K, a.bits, a.group);
        gp.off_idx[p] = (uint32_t)L.off_idx; gp.off_scale[p] = (uint32_t)L.off_scale; gp.blob_total[p] = (uint32_t)L.total;
        gp.rb_start[p] = NRB;
        NRB += (gp.N[p] + FROWS - 1) / FROWS;
    }
    for (int p = gp.P; p <= DZ_MAX_GROUP; ++p) gp.rb_start[p] = NRB;
    int cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    cus = std::max(cus - cus % 8, 8);
    // the number of column tiles is known on the device only: enough workgroups for the most there can be
    const long long most = (long long)NRB * dz_fused_tiles_max(a.T, a.D);
    const int grid = (int)((most + 7) / 8 * 8 + 2 * cus);
    // Partial tiles of the last round: tail * S is the most that tail_slices can ask for.  A call that needs more room than
    // there is makes room for every later one, two slots per compute unit: the workspace grows once.  Where that much memory is
    // not to be had, or the call is being captured into a graph without an eager call before it, the kernel cuts into as many
    // slices as fit.
    constexpr size_t tile_bytes = (size_t)FR * FJ * FTHREADS * 16;
    const int tail = ((int)std::min(most, (long long)cus - 1) + 7) / 8 * 8;
    const int S = std::min(a.K / 512, 8);
    if (S > 1 && (size_t)std::min(2 * cus, tail * S) * tile_bytes > ctx->partial_bytes)
        if (int rc = dz_want_partial(ctx, (size_t)2 * cus * tile_bytes, st)) return rc;
    const int slots = (int)std::min((size_t)2 * cus, ctx->partial_bytes / tile_bytes);
    if (int rc = dz_ensure_counters(ctx, cus, st)) return rc;
    a.partial = ctx->partial;
    a.counters = ctx->counters;
    if (a.bits == 4 && a.group == 128) return dz_set_hip_error(ctx, launch_fused<4, 128>(a, gp, dp, ctx->seg_plan, NRB, cus, slots, grid, st));
    if (a.bits == 4) return dz_set_hip_error(ctx, launch_fused<4, 64>(a, gp, dp, ctx->seg_plan, NRB, cus, slots, grid, st));
    if (a.group == 128) return dz_set_hip_error(ctx, launch_fused<2, 128>(a, gp, dp, ctx->seg_plan, NRB, cus, slots, grid, st));
    return dz_set_hip_error(ctx, launch_fused<2, 64>(a, gp, dp, ctx->seg_plan, NRB, cus, slots, grid, st));
}
