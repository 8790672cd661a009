// Reconstruction (Sec. 2.2, eq. (6)): cone-weighted bilinear backprojection of
// every square from its decimated sub-sinogram (s > 0), or of the whole slice
// from the filtered projections (s = 0: direct FDK, the same inner loop).
//
//   f(x, y, z) = (pi / P') sum_m U^-2 Bil(Y_q[m], v*, tau)
//   U = depth / R,  tau = a(x, y) - a_c + c_u - u0  (eq. (1), folded back-shift),
//   v* = z R / depth + c_v                            (eq. (9))
//
// Workgroup = a 16 x 16 (or 8 x 8) tile of one square times a run of ZP
// slices and their mirror images about the mid-plane; every thread owns one
// (x, y) and 2 ZP accumulators in registers.  Slices z and -z see detector
// rows c_v + b and c_v - b at every angle, so a pair shares its row index, its
// fraction and its LDS address: the mirrored footprint is staged in reversed
// row order, and the pair's second sample lies at a constant offset from the
// first.  For each angle the footprint of the tile's run on the (local)
// detector is bounded with eq. (1) at the tile's corners (columns) and eq. (9)
// at its corner depths and end slices (rows) -- the paper's vertex bound
// applied to the block -- and staged in LDS as quads (Y, dU, dV, dUV) of
// forward differences, so one 128-bit LDS read fetches all four samples of a
// bilinear interpolation, which is then three FMAs.  Per (x, y, angle) a
// thread computes tau, U and the weight once; along z only the row coordinate
// moves, linearly (b = z / U): four instructions for each pair (row, fraction,
// index, address) and four FMAs for each update.
//
// Bound: VALU issue, with the LDS close behind.  Counters at N = 512, s = 3,
// FP32 (16 pairs per thread): 7.8 VALU instructions per update issued at one
// wave-instruction per compute unit and cycle, LDS busy 75 % (4 cycles per
// wave for a 128-bit read, 13.6 for a 128-bit write, which is why only the
// rows an angle needs are staged).  With one slice per index (10.4 per update)
// 1.70 ms, 2000^2 x 1000 slices, s = 4: 50 ms, direct FDK at N = 256: 1.86 ms;
// now 1.36, 41.5 and 1.41 ms (4.4e12 updates/s).
//
// A close source widens the footprints, and the LDS then sets the waves that
// hide the staging; so the staged width follows the geometry in steps of eight
// columns, and the rows end where one more workgroup fits.  Update times
// relative to R = 4 N: 1.34 (R = 2.5 N), 1.53 (2 N), 1.77 (1.75 N), 2.7 (1.5 N);
// with footprints of 32 or 64 columns only (one workgroup per compute unit
// below R = 2.3 N, its loads not ahead of the arithmetic) 1.9, 5.5, 5.6 and 5.6,
// one slice per index 2.6, 3.2, 3.2 and 4.1.
#include "internal.h"
#include "dtype.h"
#include "offsets.h"

namespace fdkod {

// event counters of a checked build (see CheckKind)
static __device__ unsigned g_checks_bp[kCheckKinds];

hipError_t checks_read_backproject(unsigned long long* out, bool reset) {
    unsigned h[kCheckKinds] = {};
    hipError_t e = hipMemcpyFromSymbol(h, HIP_SYMBOL(g_checks_bp), sizeof(h), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    for (int k = 0; k < kCheckKinds; ++k) out[k] += h[k];
    if (reset) {
        const unsigned z[kCheckKinds] = {};
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_checks_bp), z, sizeof(z), 0, hipMemcpyHostToDevice);
    }
    return e;
}

typedef float f4v __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(3))) const char* lds_cptr;
typedef __attribute__((address_space(3))) const f4v* lds_f4ptr;

// Per-angle footprints and constants are computed for kFpChunk angles at a
// time (one lane per angle) and kept for two such chunks.
constexpr int kFpChunk = 8;

// Margin of a block's footprint, in samples: far above the rounding of the
// footprint's and the voxels' coordinates (about 1e-7 of N), far below a sample.
constexpr float kBpMargin = 0.01f;

// One angle's constants of a 16 x 16 tile and run.
struct BpAngle {
    float ax, ay, cs, sn;        // R (dL Dc - Lc dD) / Dc = ax dx + ay dy; cos, sin
    float dc, kc, top, kr[2];    // Dc, c_u - u0 - c0, R (or Dc on cone-corrected rows), c_v - r0 of each footprint
    int c0, off[2];              // the footprints' first column; byte offset of the first sample of each
    int nq;                      // quad rows per staging lane
    int pad[3];
};

// LDS row pitch in quads of a footprint of tw columns: 4 or 12 mod 16, so that
// the 16 lanes of one 4 x 4 patch of voxels (at most six columns of one or two
// rows) read distinct groups of four banks.
constexpr int bp_pitch(int tw) { return (tw + 3) / 8 * 8 + 4; }

// LDS of one group of BX BX threads: two staged footprints (the quads of TH
// detector rows: TH - 1 rows) and, for two chunks of angles, the per-angle
// constants.
template <int TW, int TH>
struct BpSmem {
    float4 tile[2 * (TH - 1) * bp_pitch(TW)];
    BpAngle ang[2][kFpChunk];
};

// Waves per SIMD that a shape's LDS allows, five at most (the registers of the
// arithmetic allow no more).
constexpr int kBpLds = 160 * 1024;
template <int BX, int TW, int TH, int AG>
constexpr int bp_waves() {
    constexpr int groups = kBpLds / (int)(sizeof(BpSmem<TW, TH>) * AG);
    constexpr int waves = groups * (BX * BX * AG / 64) / 4;
    return waves < 1 ? 1 : waves < 5 ? waves : 5;
}

// Lane l receives lane l + 1's value (a DPP wave shift; lane 63 receives 0).
__device__ __forceinline__ float from_next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130 /* wave_shl:1 */, 0xf, 0xf, false));
}

// A run of ZP lower slices from l0 (side 0), or of their mirror images (1).
struct BpRun {
    int l0, side;
};

// Backprojection of one BX x BX (x, y) tile tl (BX = 16 or 8).  PAIR: the ZP
// lower slices from run a's first and their mirror images (l' = N_z - 1 - l).
// Otherwise (slabs): the runs a and b, with row indices of their own (b only
// if `two`); the arithmetic of a slice is the same, so a slab whose runs start
// where the whole volume's do gives its bits.
//
// AG groups of BX BX threads share the angles (each takes a contiguous part)
// and their sums are added in group order at the end.  Every thread of the
// workgroup calls it (it contains barriers).
//
// While angle m is accumulated from LDS, the detector samples of angle m + 1
// are already being loaded into registers, so global-memory latency overlaps
// the arithmetic; two barriers per angle separate the LDS phases.
template <int BX, int ZP, bool PAIR, int TW, int TH, int AG, int STORE>
__device__ __forceinline__ void bp_block(const BpVol& v, BpRun a, BpRun b, bool two, const BpTile& tl,
                                         BpSmem<TW, TH> (&sms)[AG]) {
    // fused only where written: every instantiation rounds alike, and
    // D = Dc + dD rounds once
#pragma clang fp contract(off)
    // the thread within its group, and the group's part of the angles
    constexpr int NTHR = BX * BX;
    const int tid = AG == 1 ? threadIdx.x : threadIdx.x & (NTHR - 1);
    const int grp = AG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NTHR);
    BpSmem<TW, TH>& sm = sms[grp];
    const int per = (v.pd + AG - 1) / AG;
    const int mbeg = grp * per, mend = min(mbeg + per, v.pd);
    using S = Store<STORE>;
    using T = typename S::T;
    constexpr int TWP = bp_pitch(TW);
    constexpr int SIDE = (TH - 1) * TWP;   // quads from a lower sample to the mirrored one
    auto& tile = sm.tile;
    const SquareDesc sq = v.squares[tl.sq];
    const int2 gd = v.grid[tl.sq];
    const int u0 = gd.x, width = gd.y;

    const int n = v.n;
    // The 16 lanes that one cycle of a 128-bit LDS read serves take a 4 x 4
    // patch of voxels, a wave four patches (along x, or 2 x 2 of an 8 x 8
    // tile).  Measured: those lanes are, in each half of the wave, the groups
    // of four lanes with an even number of bits in their index, then those
    // with an odd one.
    const int lq = tid >> 2;                     // group of four lanes
    const int patch = ((lq ^ (lq >> 1) ^ (lq >> 2)) & 1) | ((lq >> 2) & 2);
    const int tx = (tid & 3) + 4 * (BX == 16 ? patch : patch & 1);
    const int ty = ((lq >> 1) & 3) + 4 * (BX == 16 ? tid >> 6 : patch >> 1);
    const int ix1 = min(tl.x0 + BX - 1, sq.x1 - 1);
    const int iy1 = min(tl.y0 + BX - 1, sq.y1 - 1);
    const int i = tl.x0 + tx, j = tl.y0 + ty;
    const bool own = (i <= ix1) && (j <= iy1);
    // offsets from the square centre; threads outside the square use the
    // block's last voxel so every address they form stays in bounds
    const float dx = (float)min(i, ix1) - v.cu - sq.xc;
    const float dy = (float)min(j, iy1) - v.cu - sq.yc;
    const float bx0 = (float)tl.x0 - v.cu - sq.xc, bx1 = (float)ix1 - v.cu - sq.xc;
    const float by0 = (float)tl.y0 - v.cu - sq.yc, by1 = (float)iy1 - v.cu - sq.yc;

    // the run covers ZP slices even past the volume's middle (those voxels
    // are computed and discarded), so the staged rows always hold the whole run
    // first slice of each footprint's run
    const float z0[2] = {(float)a.l0 - v.cz, (float)(PAIR ? a.l0 : b.l0) - v.cz};

    const bool direct = v.row_stride_direct != 0;
    const int row_stride = direct ? v.row_stride_direct : width;
    const size_t plane = (size_t)v.nv * row_stride;
    const T* data = (const T*)v.data + (direct ? 0 : sq.y_off_row * v.nv);
    const float kq = v.cu - (float)u0;            // tau = rel + kq

    // staging map: footprint t is staged by half of the threads; a lane keeps
    // one footprint column and nq consecutive rows (their quads), for which
    // it loads nq + 1 rows
    constexpr int SIDE_THR = NTHR / 2;
    constexpr int SW = TW <= 16 ? 16 : TW <= 32 ? 32 : 64;   // lanes of a row (columns from TW on idle)
    constexpr int NGRP = SIDE_THR / SW;
    static_assert((TH - 1) % NGRP == 0, "uniform staging trip count");
    constexpr int NQ = (TH - 1) / NGRP;          // at most; an angle's own count is BpAngle::nq
    constexpr int NR = NQ + 1;
    constexpr int NQMIN = NQ < 4 ? NQ : NQ / 2 + 1;  // rows staged without a branch
    const int scol = tid % SW;
    const int sgrp = (tid % SIDE_THR) / SW;
    // the footprint this thread stages (uniform over a wave unless one wave
    // stages both), and whether it is a mirrored one
    constexpr bool kSideUniform = SIDE_THR >= 64;
    const int st_t = kSideUniform ? __builtin_amdgcn_readfirstlane(tid / SIDE_THR) : tid / SIDE_THR;
    const int mirrored = PAIR ? st_t : st_t ? b.side : a.side;

    // footprints of the block at the kFpChunk angles from m0 (a multiple of
    // kFpChunk), one lane of the first wave per angle: eq. (1) at the block's
    // corners bounds the columns, eq. (9) at its corner depths and end slices
    // the rows; kBpMargin of a sample on every side covers the rounding of the
    // reciprocals.  The mirrored run's rows are n - 1 minus these.  Angle m's
    // constants sit at [(m / kFpChunk) % 2][m % kFpChunk].
    constexpr int ES = (int)sizeof(T);
    const uint32_t plane_bytes = (uint32_t)(plane * ES);
    auto footprint = [&](int m0) {
        const int slot = (m0 / kFpChunk) & 1;
        const int m = mbeg + m0 + tid;
        if (tid < kFpChunk && m < mend) {
            const float2 t = v.trig[m];
            const float dc = fmaf(sq.yc, t.y, fmaf(sq.xc, t.x, v.r));
            const float lc = fmaf(sq.yc, t.x, -(sq.xc * t.y));
            const float rdc = __builtin_amdgcn_rcpf(dc);
            float tlo = INFINITY, iulo = INFINITY, iuhi = -INFINITY;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float cx = (k & 1) ? bx1 : bx0;
                const float cy = (k & 2) ? by1 : by0;
                const float dl = fmaf(cy, t.x, -(cx * t.y));
                const float dd = fmaf(cx, t.x, cy * t.y);
                const float rd = __builtin_amdgcn_rcpf(dc + dd);
                tlo = fminf(tlo, fmaf(v.r * fmaf(dl, dc, -(lc * dd)) * rdc, rd, kq));
                const float iu = (v.cone ? dc : v.r) * rd;   // row offset per unit z
                iulo = fminf(iulo, iu);
                iuhi = fmaxf(iuhi, iu);
            }
            const int c0 = (int)floorf(tlo - kBpMargin);
            int r0[2], quads = 0;
#pragma unroll
            for (int f = 0; f < (PAIR ? 1 : 2); ++f) {
                const float zl = z0[f] + (float)(ZP - 1);
                const float vlo = fminf(fminf(fmaf(z0[f], iulo, v.cv), fmaf(z0[f], iuhi, v.cv)),
                                        fminf(fmaf(zl, iulo, v.cv), fmaf(zl, iuhi, v.cv)));
                const float vhi = fmaxf(fmaxf(fmaf(z0[f], iulo, v.cv), fmaf(z0[f], iuhi, v.cv)),
                                        fmaxf(fmaf(zl, iulo, v.cv), fmaf(zl, iuhi, v.cv)));
                r0[f] = (int)floorf(vlo - kBpMargin);
                quads = max(quads, (int)floorf(vhi + kBpMargin) + 1 - r0[f]);    // quad rows r0 .. floor(vhi)
            }
            if (PAIR) r0[1] = r0[0];
            const float lr = v.r * lc * rdc;
            BpAngle an;
            an.ax = -fmaf(v.r, t.y, lr * t.x);
            an.ay = fmaf(v.r, t.x, -(lr * t.y));
            an.cs = t.x;
            an.sn = t.y;
            an.dc = dc;
            an.kc = kq - (float)c0;
            an.top = v.cone ? dc : v.r;
            an.c0 = c0;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const bool mir = PAIR ? f == 1 : (f ? b.side : a.side) != 0;
                an.kr[f] = v.cv - (float)r0[f];
                an.off[f] = (((mir ? n - 1 - r0[f] : r0[f]) - v.v0) * row_stride + c0) * ES;
            }
            an.nq = min((quads + NGRP - 1) / NGRP, NQ);
            sm.ang[slot][tid] = an;
        }
    };
    // detector samples of angle m's footprint into registers, as raw bits of
    // the storage type (converted when staged, so no load is waited for
    // early).  One buffer resource spans the angle's plane of the data: rows
    // outside the buffer fall outside it and read zero (a row above the first
    // wraps to a huge unsigned offset), and a column outside [0, width) gets
    // an offset beyond every plane, so its samples read zero too.  A lane's
    // samples are consecutive rows (downwards for a mirrored footprint), so
    // each costs one add.  Footprints of more than 16 samples per thread are
    // loaded after the arithmetic instead where their registers would cost
    // occupancy (at three waves per SIMD or fewer the LDS has cost it already).
    constexpr bool kPrefetch = NR <= (bp_waves<BX, TW, TH, AG>() <= 3 ? 32 : 16);
    const int rstep_bytes = (mirrored ? -row_stride : row_stride) * ES;
    uint32_t pre[NR];
    auto fetch = [&](int m) {
        const BpAngle& an = sm.ang[(m / kFpChunk) & 1][m % kFpChunk];
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            uniform_ptr(data + (size_t)(mbeg + m) * plane), (short)0, (int)plane_bytes, 0x00020000);
        const int nq = __builtin_amdgcn_readfirstlane(an.nq);
        const int col = an.c0 + scol, at = an.off[st_t] + scol * ES + __mul24(sgrp, nq * rstep_bytes);
        const uint32_t off0 = column_offset((unsigned)col < (unsigned)width && (SW == TW || scol < TW), at);
        // (each offset in its own register, never folded into the
        // instruction's constant offset: the range check must see the
        // whole offset of every sample)
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            if (q > NQMIN && q > nq) break;      // uniform
            uint32_t off;
            if (q == 0) {
                off = off0;
                asm volatile("" : "+v"(off));
            } else if constexpr (!kSideUniform) {
                off = moved(off0, q * rstep_bytes);
                asm volatile("" : "+v"(off));
            } else {
                asm volatile("v_add_u32 %0, %1, %2" : "=v"(off) : "s"(q * rstep_bytes), "v"(off0));
            }
            pre[q] = S::raw_bits(rs, (int)off);
        }
    };
    // quads (Y, dU, dV, dUV) into LDS: at (r, c), Y = Y[r][c], dU = Y[r][c+1]
    // - Y[r][c], dV = Y[r+1][c] - Y[r][c], dUV = dU[r+1] - dU[r], so that the
    // bilinear sample at (r + fv, c + fu) is Y + fu dU + fv (dV + fu dUV).
    // The last column's quad is never read, so the lane that receives the
    // next group's first sample writes an unused quad; nor are rows below the
    // footprint's last.
    auto stage = [&](int m) {
        const int nq = __builtin_amdgcn_readfirstlane(sm.ang[(m / kFpChunk) & 1][m % kFpChunk].nq);
        float4* dst = tile + st_t * SIDE + scol + __mul24(sgrp, nq * TWP);
        float y0 = S::from_bits(pre[0]);
        float du0 = from_next_lane(y0) - y0;
#pragma unroll
        for (int r = 0; r < NQ; ++r) {
            if (r >= NQMIN && r >= nq) break;    // uniform
            const float y1 = S::from_bits(pre[r + 1]);
            const float du1 = from_next_lane(y1) - y1;
            const float4 quad = make_float4(y0, du0, y1 - y0, du1 - du0);
            if (SW == TW || scol < TW) dst[r * TWP] = quad;
            y0 = y1;
            du0 = du1;
        }
    };

    const float sr2 = v.scale * v.r * v.r;
    float acc[2][ZP];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < ZP; ++k) acc[t][k] = 0.0f;

    // the first chunk's footprints; the next chunk's are computed while the
    // first angle of a chunk is accumulated (two barriers before their first
    // use, and after the last use of the chunk two before them)
    // (m counts the group's angles; a group with fewer than `per` only joins
    // the barriers of the last rounds)
    const int count = mend - mbeg;
    if (tid < 64) footprint(0);
    __syncthreads();
    if (AG == 1 || count > 0) {
        fetch(0);
        stage(0);
    }
    __syncthreads();
#pragma unroll 1
    for (int m = 0; m < per; ++m) {
        if (AG > 1 && m >= count) {
            __syncthreads();
            __syncthreads();
            continue;
        }
        const bool more = m + 1 < count;
        if (kPrefetch && more) fetch(m + 1);             // in flight during the arithmetic below
        if (m % kFpChunk == 0 && m + kFpChunk < count && tid < 64) footprint(m + kFpChunk);
        const BpAngle& an = sm.ang[(m / kFpChunk) & 1][m % kFpChunk];
        const float d = an.dc + fmaf(dx, an.cs, dy * an.sn);
        const float rd = __builtin_amdgcn_rcpf(d);
        float tau = fmaf(fmaf(dx, an.ax, dy * an.ay), rd, an.kc);
        const float w = sr2 * rd * rd;               // (pi / P') U^-2, U = D / R
        // row offset per unit z: R / D (eq. (9)), or D_c / D on cone-corrected rows
        const float vstep = an.top * rd;
        FDKOD_CHECK_EVENT(g_checks_bp, kCheckBpCols, own && !(tau >= 0.0f && tau < (float)(TW - 1)));
        // the footprint holds every column and row of the run (the planner's
        // bounds); the clamps keep the reads inside the tile all the same
        tau = __builtin_amdgcn_fmed3f(tau, 0.0f, (float)(TW - 1) - 0.01f);
        const float vmost = fmaf(-(float)(ZP - 1), vstep, (float)(TH - 1) - 0.01f);
        float v0[2];
#pragma unroll
        for (int f = 0; f < (PAIR ? 1 : 2); ++f) {
            v0[f] = fmaf(z0[f], vstep, an.kr[f]);
            FDKOD_CHECK_EVENT(g_checks_bp, kCheckBpRows, own && !(v0[f] >= 0.0f && v0[f] < vmost + 0.01f));
            v0[f] = __builtin_amdgcn_fmed3f(v0[f], 0.0f, vmost);
        }
        const float fu = __builtin_amdgcn_fractf(tau);
        // 32-bit LDS byte address of the thread's column in the footprints
        uint32_t tga = (uint32_t)(uintptr_t)(lds_cptr)(tile + (int)tau);
        asm volatile("" : "+v"(tga));   // keep it one register: address = mad24(row, pitch, tga)
        // one update: the sample of footprint t at row ri + fv
        auto update = [&](int t, int k, lds_f4ptr p, float fv) {
            const f4v Q = p[t * SIDE];
            const float top = fmaf(fu, Q.y, Q.x);          // row ri at tau
            const float dv = fmaf(fu, Q.w, Q.z);           // row ri + 1 minus row ri at tau
            acc[t][k] = fmaf(w, fmaf(fv, dv, top), acc[t][k]);
        };
        auto row_of = [&](int t, int k, float* fv) -> lds_f4ptr {
            const float vv = k == 0 ? v0[t] : fmaf((float)k, vstep, v0[t]);
            *fv = __builtin_amdgcn_fractf(vv);
            return (lds_f4ptr)(uintptr_t)(tga + __umul24((uint32_t)(int)vv, (uint32_t)(TWP * sizeof(float4))));
        };
        // four updates per group: their accumulators are complete before the
        // next group's reads are issued (without these fences the compiler may
        // issue all reads first and trade occupancy for the registers that
        // holds them)
        if constexpr (PAIR) {
#pragma unroll
            for (int k = 0; k < ZP; ++k) {
                float fv;
                const lds_f4ptr p = row_of(0, k, &fv);
                update(0, k, p, fv);
                update(1, k, p, fv);
                if ((k & 1) == 1)
                    asm volatile("" : "+v"(acc[0][k - 1]), "+v"(acc[1][k - 1]), "+v"(acc[0][k]), "+v"(acc[1][k])
                                 :: "memory");
            }
        } else {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t == 1 && !two) break;           // uniform
#pragma unroll
                for (int k = 0; k < ZP; ++k) {
                    float fv;
                    const lds_f4ptr p = row_of(t, k, &fv);
                    update(t, k, p, fv);
                    if ((k & 3) == 3)
                        asm volatile("" : "+v"(acc[t][k - 3]), "+v"(acc[t][k - 2]), "+v"(acc[t][k - 1]), "+v"(acc[t][k])
                                     :: "memory");
                }
            }
        }
        __syncthreads();
        if (more) {
            if (!kPrefetch) fetch(m + 1);
            stage(m + 1);
        }
        __syncthreads();
    }
    if constexpr (AG > 1) {
        // the groups' sums, added in group order (the tiles are no longer
        // needed; thread t's value e lies at word NTHR e + t)
        static_assert(sizeof(sm.tile) >= sizeof(float) * NTHR * 2 * ZP, "sums fit the tile");
        float* mine = (float*)sm.tile;
        if (grp > 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int k = 0; k < ZP; ++k) mine[NTHR * (t * ZP + k) + tid] = acc[t][k];
        }
        __syncthreads();
        if (grp > 0) return;
        for (int g = 1; g < AG; ++g) {
            const float* other = (const float*)sms[g].tile;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int k = 0; k < ZP; ++k) acc[t][k] += other[NTHR * (t * ZP + k) + tid];
        }
    }
    if (own) {
        // lower slices up to the middle, mirrored ones above it; of the
        // output's slices [zbase, zbase + nz)
        const size_t slice = (size_t)n * n;
        float* out = v.vol + (size_t)j * n + i;
#pragma unroll
        for (int k = 0; k < ZP; ++k) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (!PAIR && t == 1 && !two) continue;
                const bool mir = PAIR ? t == 1 : (t ? b.side : a.side) != 0;
                const int l = (PAIR || t == 0 ? a.l0 : b.l0) + k, lm = v.nzf - 1 - l;
                const int o = (mir ? lm : l) - v.zbase;
                if ((mir ? l < lm : l <= lm) && o >= 0 && o < v.nz) out[(size_t)o * slice] = acc[t][k];
            }
        }
    }
}

// Whole volume: workgroup = tile x run of slice pairs.
template <int BX, int ZP, int TW, int TH, int AG, int STORE>
__global__ __launch_bounds__(BX * BX * AG, (bp_waves<BX, TW, TH, AG>())) void k_backproject(BpArgs a) {
    __shared__ BpSmem<TW, TH> sm[AG];
    // XCD-aware order: each XCD runs a contiguous range of logical blocks
    const int b = blockIdx.x;
    const int lblk = (b & 7) * a.chunk + (b >> 3);
    if (lblk >= a.nlogical) return;               // before any barrier
    const int zt = lblk / a.ntiles;
    const BpTile tl = a.tiles[lblk - zt * a.ntiles];
    bp_block<BX, ZP, true, TW, TH, AG, STORE>(a.v, BpRun{zt * ZP, 0}, BpRun{0, 0}, true, tl, sm);
}

// A slab of slices: workgroup = tile x two (one where there are few)
// consecutive runs of the list of the lower runs that meet the slab and then
// of those whose images do.
template <int BX, int ZP, int TW, int TH, int AG, int STORE>
__global__ __launch_bounds__(BX * BX * AG, (bp_waves<BX, TW, TH, AG>())) void k_backproject_slab(BpArgs a) {
    __shared__ BpSmem<TW, TH> sm[AG];
    const int b = blockIdx.x;
    const int lblk = (b & 7) * a.chunk + (b >> 3);
    if (lblk >= a.nlogical) return;               // before any barrier
    const int zt = lblk / a.ntiles;
    const BpTile tl = a.tiles[lblk - zt * a.ntiles];
    auto run = [&](int i) { return i < a.nlow ? BpRun{a.low0 + ZP * i, 0} : BpRun{a.up0 + ZP * (i - a.nlow), 1}; };
    const int i = zt * a.per;
    const bool two = a.per == 2 && i + 1 < a.nruns;
    bp_block<BX, ZP, false, TW, TH, AG, STORE>(a.v, run(i), run(two ? i + 1 : i), two, tl, sm);
}

// Persistent backprojection over the work items of many volumes.  Workgroup
// b runs on XCD b mod 8 (round-robin dispatch) and first takes tickets from
// that XCD's range of items, so the tiles that share footprints (same volume,
// square and run) meet in one L2; when its range is exhausted it takes
// tickets from the other XCDs' ranges in turn.  Every workgroup leaves after
// all eight ranges are exhausted.  The counters must be zero at launch
// (launch_reset_counter).
template <int BX, int ZP, int TW, int TH, int STORE>
__global__ __launch_bounds__(BX * BX, (bp_waves<BX, TW, TH, 1>() < 4 ? bp_waves<BX, TW, TH, 1>() : 4)) void k_backproject_batch(BpBatchArgs a) {
    __shared__ BpSmem<TW, TH> sm[1];
    __shared__ int ticket;
    const int home = blockIdx.x & (kXcds - 1);
    for (int k = 0; k < kXcds; ++k) {
        const int x = (home + k) & (kXcds - 1);
        const int beg = a.xstart[x];
        const int count = a.xstart[x + 1] - beg;
        for (;;) {
            if (threadIdx.x == 0) ticket = (int)atomicAdd(a.counter + x * kCounterStride, 1u);
            __syncthreads();
            const int it = __builtin_amdgcn_readfirstlane(ticket);
            __syncthreads();      // all threads read the ticket before it is replaced
            if (it >= count) break;
            // item and volume parameters are workgroup-uniform: keep them in
            // scalar registers, as the single-volume kernel's arguments are
            const BatchItem bi = uniform_load(a.items + beg + it);
            const BpVol v = uniform_load(a.vols + bi.vol);
            bp_block<BX, ZP, true, TW, TH, 1, STORE>(v, BpRun{bi.zt * ZP, 0}, BpRun{0, 0}, true,
                                                     BpTile{bi.sq, bi.x0, bi.y0, 0}, sm);
        }
    }
}

__global__ void k_reset_counter(unsigned* c) {
    if (threadIdx.x < kXcds) c[threadIdx.x * kCounterStride] = 0u;
}

hipError_t launch_reset_counter(unsigned* counter, hipStream_t st) {
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, st, counter);
    return hipGetLastError();
}

// Kernel shapes: (tile side, slice pairs per thread, footprint columns,
// footprint rows, angle groups, cost).  The whole-volume and slab kernels
// exist for each, the batch kernel for those of one group.  The cost is the
// time per update on a full chip (N = 333..1000, 250..1000 slices, FP32), 100
// for the first shape.  What the narrower ones save: 36 columns against 44 at
// R = 2.5 N 3.62 / 4.57 ms (N = 1000, s = 4, 360 projections, 500 slices), 44
// against 52 at 2 N 4.57 / 5.31, 52 against 60 at 1.75 N 5.31 / 8.05, 60 against
// 64 at 1.5 N 8.06 / 10.1; 45 rows against 49 (three workgroups, not two)
// N = 333, 1000 slices, R = 3 N 1.67 / 2.28 ms; 33 rows against 49 at 52 columns
// N = 500, s = 0, 60 slices, R = 1.75 N 1.27 / 1.41 ms; 8 x 8 tiles of 17 rows
// against 20, N = 160, s = 3, R = 2.25 N 95 / 109 us.
#define FDKOD_BP_SHAPES_ONE(X) \
    X(16, 16, 32, 25, 1, 100) X(16, 16, 32, 33, 1, 107) X(16, 16, 36, 35, 1, 119) X(16, 16, 32, 45, 1, 120) \
    X(16, 16, 32, 49, 1, 164) X(16, 16, 52, 33, 1, 163) X(16, 16, 52, 49, 1, 177) X(16, 16, 64, 63, 1, 337) \
    X(16, 8, 32, 17, 1, 110) X(16, 8, 32, 25, 1, 126) X(16, 8, 36, 23, 1, 134) X(16, 8, 44, 29, 1, 153) \
    X(16, 8, 32, 41, 1, 172) X(16, 8, 52, 33, 1, 249) X(16, 8, 60, 43, 1, 268) X(16, 8, 64, 57, 1, 525) \
    X(8, 8, 16, 17, 1, 150) X(8, 8, 20, 17, 1, 180) X(8, 8, 20, 20, 1, 200) X(8, 8, 28, 28, 1, 335)
#define FDKOD_BP_SHAPES(X) FDKOD_BP_SHAPES_ONE(X) \
    X(16, 8, 32, 17, 2, 110) X(16, 8, 32, 25, 2, 126) X(16, 8, 36, 23, 2, 134) X(16, 8, 44, 29, 2, 153) \
    X(8, 8, 16, 17, 4, 150) X(8, 8, 20, 20, 4, 200) \
    X(8, 4, 16, 13, 4, 190) X(8, 4, 20, 13, 4, 220) X(8, 4, 28, 20, 4, 400)

// Public tuning keys (z run, tile columns, tile rows, angles per stage).
#define FDKOD_BP_VARIANTS(X)  \
    X(64, 32, 96, 1) \
    X(32, 32, 48, 1) X(32, 32, 48, 2) X(32, 32, 48, 4) \
    X(32, 32, 64, 1) X(32, 32, 64, 2) \
    X(32, 64, 48, 1) X(32, 64, 48, 2) \
    X(32, 64, 64, 1) \
    X(16, 32, 48, 1) X(16, 32, 48, 2) X(16, 32, 48, 4) \
    X(16, 32, 64, 1) X(16, 32, 64, 2) \
    X(16, 64, 48, 1) X(16, 64, 48, 2) \
    X(16, 64, 64, 1)

bool backproject_variant_exists(const BpVariant& var) {
#define FDKOD_X(Z, W, H, GG) \
    if (var.zrun == Z && var.tile_w == W && var.tile_h == H && var.g == GG) return true;
    FDKOD_BP_VARIANTS(FDKOD_X)
#undef FDKOD_X
    return false;
}

bool backproject_shape_for(int bx, int zp, int ag, int need_c, int need_r, BpShape* out) {
    BpShape best{};
#define FDKOD_X(B, Z, W, H, A, C)                                                                    \
    if (B == bx && Z == zp && A == ag && W >= need_c && H >= need_r && (!best.zp || C < best.cost)) \
        best = BpShape{B, Z, W, H, A, C, bp_waves<B, W, H, A>()};
    FDKOD_BP_SHAPES(FDKOD_X)
#undef FDKOD_X
    *out = best;
    return best.zp != 0;
}

static bool same_shape(const BpShape& sh, int bx, int zp, int tw, int th, int ag) {
    return sh.bx == bx && sh.zp == zp && sh.tw == tw && sh.th == th && sh.ag == ag;
}

// K<..., STORE> for the run-time storage type
#define FDKOD_BP_LAUNCH(K, GRID, BLOCK, ...)                                                      \
    switch (store) {                                                                              \
        case 0: hipLaunchKernelGGL((K<__VA_ARGS__, 0>), GRID, dim3(BLOCK), 0, st, a); break;      \
        case 1: hipLaunchKernelGGL((K<__VA_ARGS__, 1>), GRID, dim3(BLOCK), 0, st, a); break;      \
        default: hipLaunchKernelGGL((K<__VA_ARGS__, 2>), GRID, dim3(BLOCK), 0, st, a); break;     \
    }                                                                                             \
    return hipGetLastError();

hipError_t launch_backproject(const BpArgs& a, const BpShape& sh, int store, hipStream_t st) {
    const dim3 grid(8 * a.chunk);
#define FDKOD_X(B, Z, W, H, A, C) \
    if (same_shape(sh, B, Z, W, H, A)) { FDKOD_BP_LAUNCH(k_backproject, grid, B * B * A, B, Z, W, H, A) }
    FDKOD_BP_SHAPES(FDKOD_X)
#undef FDKOD_X
    return hipErrorInvalidValue;
}

hipError_t launch_backproject_slab(const BpArgs& a, const BpShape& sh, int store, hipStream_t st) {
    const dim3 grid(8 * a.chunk);
#define FDKOD_X(B, Z, W, H, A, C) \
    if (same_shape(sh, B, Z, W, H, A)) { FDKOD_BP_LAUNCH(k_backproject_slab, grid, B * B * A, B, Z, W, H, A) }
    FDKOD_BP_SHAPES(FDKOD_X)
#undef FDKOD_X
    return hipErrorInvalidValue;
}

hipError_t launch_backproject_batch(const BpBatchArgs& a, const BpShape& sh, int store, int blocks, hipStream_t st) {
#define FDKOD_X(B, Z, W, H, A, C) \
    if (same_shape(sh, B, Z, W, H, A)) { FDKOD_BP_LAUNCH(k_backproject_batch, dim3(blocks), B * B, B, Z, W, H) }
    FDKOD_BP_SHAPES_ONE(FDKOD_X)
#undef FDKOD_X
    return hipErrorInvalidValue;
}

int backproject_batch_occupancy(const BpShape& sh, int store) {
    int nb = 0;
    hipError_t e = hipErrorInvalidValue;
#define FDKOD_X(B, Z, W, H, A, C)                                                                  \
    if (same_shape(sh, B, Z, W, H, A)) {                                                           \
        switch (store) {                                                                           \
            case 0: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_backproject_batch<B, Z, W, H, 0>, B * B, 0); break; \
            case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_backproject_batch<B, Z, W, H, 1>, B * B, 0); break; \
            default: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_backproject_batch<B, Z, W, H, 2>, B * B, 0); break; \
        }                                                                                          \
    }
    FDKOD_BP_SHAPES_ONE(FDKOD_X)
#undef FDKOD_X
    return e == hipSuccess ? nb : 0;
}

}  // namespace fdkod
