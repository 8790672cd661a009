// Decomposition of the filtered sinogram (Sec. 2.1; cost eq. (7)): for every
// square q, detector row v and local column j, crop the row part the square
// uses, shift it so the square's centre trajectory becomes one column (linear
// interpolation), and decimate it in angle with the triangle low-pass filter:
//
//   Y_q[m][v][j] = sum_p w[m][p] * Lin(q[p][v][.], a_c(beta_p) + u0_q + j)
//
// One wavefront per task (square, group of rows, columns, segment of the
// decimated angles).  The wavefront walks the projections once, in the order
// of a host-built schedule; with the triangle each projection feeds at most
// two open decimation windows, held in two accumulators per column, and a
// window is written out as soon as its last projection has been added.
//
// Bound by instruction issue: a step's scalar work (tables, resource) and its
// address arithmetic cost as much as its multiply-adds, and squares narrower
// than a wave leave lanes idle.  So
//  - narrow squares put several rows side by side into a wave (wider ones, in
//    one chunk, equal pieces of their columns): lanes idle by a tenth instead
//    of three quarters at 14 columns;
//  - every sample is loaded once: the taps to its right are the next lanes'
//    values, by a DPP shift folded into the difference (a chunk has as many
//    lanes more than columns), where each tap was a load of its own;
//  - one buffer resource spans a projection, so the row is part of a lane's
//    offset and a lane takes two rows with one more addition; the column's
//    range check is one compare and select per sample.  A resource per row
//    was rebuilt in scalar registers for each row and step, which bounded the
//    cone-corrected rows (46 cycles per row and step, scalar unit shared by
//    four SIMDs);
//  - a small volume's decimated angles go to several tasks (see DecimSeg).
// Before -> after: 256 volumes of 32^3..64^3, BF16 1000 -> 260 us; N = 64,
// s = 2 14 -> 8 us; N = 193, cone-corrected FP16 rows 249 -> 118 us; N = 384,
// windowed sinc and cubic 1113 -> 613 us; N = 1000, s = 5 18.4 (row-staged
// kernel) -> 10.6 ms.
//
// Cone-corrected rows (CONE): row v' of square q at angle beta_p is first
// resampled from detector row (v' - c_v) R / D_c(beta_p) + c_v, so each
// cropped sample is a bilinear one: the same column interpolation on the two
// detector rows that bracket the warped row, then a linear one between them.
//
// Quality knobs: a windowed-sinc decimation keeps `taps` windows open (each
// projection is added to all of them with its own weight; the schedule
// carries the extra weights), and the cubic shift weights four neighbouring
// samples with Keys' kernel of the step's fraction.
#include "internal.h"
#include "dtype.h"
#include "geom.h"
#include "offsets.h"

namespace fdkod {

// Read-only tables of the decimation (schedule, crop offsets, row scales,
// extra window weights), read word by word through the constant address
// space so that their lane-uniform loads are scalar.
typedef __attribute__((address_space(4))) const int* cword_ptr;
static_assert(sizeof(DecimStep) == 16 && sizeof(int2) == 8, "table layouts");

// Shape of one task's inner loop: CH column chunks, NW decimation windows open
// at once (2 for the triangle, `taps` for the windowed sinc), RPT output rows
// per lane, NR detector rows read for them (one each, or two for
// cone-corrected rows).  U steps are loaded per group and two groups are in
// flight (the next group's loads are issued before the current group's
// arithmetic), so U shrinks as a step's loads grow.
template <int CH, int NR, int NW>
struct DecimShape {
    static constexpr int LOADS = CH * NR;
    // at most 4 steps per group: the scalar state of 8 steps (schedule and
    // crop entries of two groups in flight) does not fit the scalar registers
    static constexpr int U0 = LOADS >= 8 ? 1 : 8 / LOADS;
    static constexpr int U = U0 > 4 ? 4 : U0;
    static constexpr int NX = NW > 2 ? NW - 2 : 1;     // extra weights per step (array size)
};

// the value of the next lane (zero in lane 63)
__device__ __forceinline__ float next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130 /* wave_shl:1 */, 0xf, 0xf, true));
}

// One task: square q, a group of rows, a group of columns and a segment of the
// decimated angles (SEG; else all of them), run by one wavefront.  Lanes form
// a.rw groups of a.gw (rows of the task side by side); each lane owns RPT rows,
// a.rw apart, and CH columns.
template <int CH, int STORE, bool CONE, int NW, bool CUBIC, int RPT, bool SEG>
__device__ __forceinline__ void decimate_task(const DecimVol& a, int task, int lane) {
    using S = Store<STORE>;
    using T = typename S::T;
    constexpr int NT = CUBIC ? 4 : 2;
    constexpr int NR = CONE ? 2 * RPT : RPT;                // detector rows loaded per step
    constexpr int CW = 64 - (NT - 1);                       // columns per chunk (CH > 1)
    using Sh = DecimShape<CH, NR, NW>;
    constexpr int U = Sh::U;
    constexpr int NX = Sh::NX;
    static_assert(kDecimUnroll % U == 0, "the schedule is padded to whole groups");
    // plain rows: the squares of one group of rows run together and share its
    // reads in L2.  CONE: the row groups of one square run together, since
    // squares read different detector rows for the same warped row.
    const int g = task % a.tasks_per_sq;
    const int sv = task / a.tasks_per_sq;
    const int seg = SEG ? sv / (a.nvb * a.nsq) : 0;
    const int vq = SEG ? sv % (a.nvb * a.nsq) : sv;
    const int q = CONE ? vq / a.nvb : vq % a.nsq;
    const int vb = CONE ? vq % a.nvb : vq / a.nsq;
    const int n = a.n;
    const int width = a.grid[q].y;
    const int lr = lane / a.gw, lc = lane - lr * a.gw;      // row group and column of the lane
    const int jbase = g * (CH > 1 ? CH * CW : a.gw - (NT - 1)) + lc;
    if (jbase - lc >= width) return;
    const int row0 = vb * a.rw * RPT + lr;                  // the lane's first row within the buffer

    T* ws = (T*)a.ws;
    // the segment: windows [m0, m1) written, of the steps [e0, e1) they are
    // open in, ms the window open at e0 (earlier windows' parts, from before
    // m0, are dropped)
    int e0 = 0, e1 = a.nsched, ms = 0, m0 = 0, m1 = a.pd;
    if (SEG && a.nseg > 1) {
        // (P' <= 32768 angles, at most kDecimWaves segments: below 2^31)
        m0 = (int)((unsigned)(a.pd * seg) / (unsigned)a.nseg);
        m1 = (int)((unsigned)(a.pd * (seg + 1)) / (unsigned)a.nseg);
        const cword_ptr first = (cword_ptr)(a.segs + m0), last = (cword_ptr)(a.segs + m1 - 1);
        e0 = first[0];
        ms = first[1];
        e1 = last[2];
    }
    cword_ptr sched = (cword_ptr)(a.sched + e0);                              // 4 words per step
    cword_ptr crop = (cword_ptr)(a.crop + (size_t)q * a.nsched + e0);         // 2 words per step
    cword_ptr rsc = (cword_ptr)(CONE ? a.rscale + (size_t)q * a.nsched + e0 : nullptr);
    cword_ptr wext = (cword_ptr)(NW > 2 ? a.wext + (size_t)(NW - 2) * e0 : nullptr);
    const int64_t yoff = a.squares[q].y_off_row * a.nv;
    const size_t plane = (size_t)a.nv * width;   // elements per decimated angle
    constexpr int ES = (int)sizeof(T);
    const int rowb = n * ES;                     // bytes per detector row
    const uint32_t planeb = (uint32_t)a.nv * (uint32_t)rowb;   // bytes per projection
    // the column of the lane's first sample relative to the crop offset (idle
    // lanes: outside any row), and its byte offset within the
    // projection less the crop's
    const int lcol = lr < a.rw ? jbase - (CUBIC ? 1 : 0) : 0x20000000;
    const int loff = (jbase - (CUBIC ? 1 : 0)) * ES + (CONE ? 0 : row0 * rowb);
    float vrel[RPT];                             // v' - c_v (CONE)
    if constexpr (CONE) {
#pragma unroll
        for (int r = 0; r < RPT; ++r) vrel[r] = (float)(row0 + r * a.rw) - a.cv;
    }

    // acc[i][r]: the i-th open window of output row r (acc[0] is written out next)
    float acc[NW][RPT][CH];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int r = 0; r < RPT; ++r)
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[i][r][c] = 0.0f;
    int m = ms;

    // Per-group state: the steps' close flags, weights and fractions, the row
    // fractions and the loaded samples x[row][step][chunk].
    struct Group {
        int emit[U];
        float w[U][NW > 2 ? NW : 2];
        float phi[U];
        float fv[RPT][U];
        float x[NR][U][CH];
    };
    // Each projection is read through a buffer resource spanning it, one
    // sample per lane; a column outside the detector moves the offset out of
    // range (it reads zero, the zero extension of the crop), as does a row
    // below or above it.
    auto issue = [&](cword_ptr sg, cword_ptr cg, cword_ptr rg, cword_ptr wg, Group& G) {
        int p[U], cx[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            p[u] = sg[4 * u];
            G.emit[u] = sg[4 * u + 1];
            G.w[u][0] = __int_as_float(sg[4 * u + 2]);
            G.w[u][1] = __int_as_float(sg[4 * u + 3]);
            cx[u] = cg[2 * u];
            G.phi[u] = __int_as_float(cg[2 * u + 1]);
            if constexpr (NW > 2) {
#pragma unroll
                for (int i = 0; i < NX; ++i) G.w[u][i + 2] = __int_as_float(wg[(NW - 2) * u + i]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                uniform_ptr((const char*)a.filt + (uint64_t)(uint32_t)p[u] * planeb), (short)0, (int)planeb,
                0x00020000);
            uint32_t coff[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c)
                coff[c] = column_offset((unsigned)(cx[u] + lcol + CW * c) < (unsigned)n, cx[u] * ES + loff + CW * ES * c);
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                if constexpr (CONE) {
                    // warped row -> detector row (v' - c_v) R / D_c + c_v
                    const float rr = fmaf(vrel[r], __int_as_float(rg[u]), a.cv);
                    const float rf = floorf(rr);
                    G.fv[r][u] = rr - rf;
                    const int r0 = min(max((int)rf, -2), n);    // both rows outside beyond these
                    const int ro = __mul24(r0, rowb);
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        G.x[2 * r][u][c] = S::raw(rs, (int)moved(coff[c], ro));
                        G.x[2 * r + 1][u][c] = S::raw(rs, (int)moved(coff[c], ro + rowb));
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < CH; ++c) G.x[r][u][c] = S::raw(rs, (int)moved(coff[c], r * a.rw * rowb));
                }
            }
        }
    };
    auto consume = [&](const Group& G) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float phi = G.phi[u];
            float cw[4];
            if constexpr (CUBIC) keys_weights(phi, cw);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                float rowv[NR];
#pragma unroll
                for (int rw = 0; rw < NR; ++rw) {
                    // the taps to the right are the next lanes' samples
                    const float x0 = G.x[rw][u][c];
                    const float x1 = next_lane(x0);
                    if constexpr (CUBIC) {
                        const float x2 = next_lane(x1);
                        const float x3 = next_lane(x2);
                        float t = cw[0] * x0;
                        t = fmaf(cw[1], x1, t);
                        t = fmaf(cw[2], x2, t);
                        rowv[rw] = fmaf(cw[3], x3, t);
                    } else {
                        rowv[rw] = fmaf(phi, x1 - x0, x0);
                    }
                }
#pragma unroll
                for (int r = 0; r < RPT; ++r) {
                    float val;
                    if constexpr (CONE) val = fmaf(G.fv[r][u], rowv[2 * r + 1] - rowv[2 * r], rowv[2 * r]);
                    else val = rowv[r];
#pragma unroll
                    for (int i = 0; i < NW; ++i) acc[i][r][c] = fmaf(G.w[u][i], val, acc[i][r][c]);
                }
            }
            if (G.emit[u]) {
                const bool mine = !SEG || (m >= m0 && m < m1);
#pragma unroll
                for (int r = 0; r < RPT; ++r) {
                    const int row = row0 + r * a.rw;
                    const size_t base = (size_t)yoff + (size_t)m * plane + (size_t)row * width;
                    const bool rok = mine && lr < a.rw && row < a.nv && lc < (CH > 1 ? CW : a.gw - (NT - 1));
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const int j = jbase + CW * c;
                        if (rok && j < width) S::put(ws, base + j, acc[0][r][c]);
#pragma unroll
                        for (int i = 0; i + 1 < NW; ++i) acc[i][r][c] = acc[i + 1][r][c];
                        acc[NW - 1][r][c] = 0.0f;
                    }
                }
                ++m;
            }
        }
    };
    // Two groups (ping, pong) per iteration; segments hold whole pairs.  Where
    // branches join after a group's loads, the wait is for every load in flight,
    // the next group's with them; four chunks of FP32 cone rows, 16 loads a step,
    // take the last pair after the loop instead, without branches (N = 2000, s = 4
    // 98.6 -> 83.5 ms, N = 1024, s = 3 4.73 -> 4.32).  It costs registers and code:
    // with 16-bit rows, the cubic shift, fewer loads a step or a short walk it is
    // slower (N = 2000, s = 4, BF16, 360 projections 22.4 / 23.0 ms; N = 193, s = 3,
    // cone 115 / 132 us, N = 100, s = 2 10.5 / 11.3).
    constexpr bool PEEL = CONE && CH == 4 && STORE == 0 && !CUBIC;
    static_assert(kDecimUnroll % (2 * U) == 0, "segments hold whole pairs of groups");
    Group ga, gb;
    issue(sched, crop, rsc, wext, ga);
    for (int t = PEEL ? e0 + 2 * U : e0; t < e1; t += 2 * U) {
        const bool b_ok = PEEL || t + U < e1;
        if (b_ok) issue(sched + 4 * U, crop + 2 * U, rsc + U, wext + (NW - 2) * U, gb);
        sched += 8 * U;
        crop += 4 * U;
        rsc += 2 * U;
        wext += 2 * (NW - 2) * U;
        consume(ga);
        if (PEEL || t + 2 * U < e1) issue(sched, crop, rsc, wext, ga);
        if (b_ok) consume(gb);
    }
    if constexpr (PEEL) {
        issue(sched + 4 * U, crop + 2 * U, rsc + U, wext + (NW - 2) * U, gb);
        consume(ga);
        consume(gb);
    }
}

template <int CH, int STORE, bool CONE, int NW, bool CUBIC, int RPT>
__global__ __launch_bounds__(256) void k_decimate(DecimVol a) {
    // XCD-aware order: consecutive logical blocks share an XCD (and its L2)
    const int nblk = gridDim.x;
    const int chunk = nblk / 8;
    const int b = blockIdx.x;
    const int lblk = (b & 7) * chunk + (b >> 3);
    // the wave index is uniform across the wave; say so, so that the task's
    // square, row and buffer resources live in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task = lblk * 4 + wave;
    if (task >= a.ntasks) return;         // no barriers in this kernel
    decimate_task<CH, STORE, CONE, NW, CUBIC, RPT, true>(a, task, threadIdx.x & 63);
}

// Many volumes in one launch (tasks concatenated volume after volume).  Each
// volume uses its own chunk count (at most CHMAX) and rows per wave, so the
// waves of a small volume do not carry idle columns.  Rows per lane of one chunk
// are the launch's: a kernel with both forms takes 15..18 % longer for two (its
// scalar registers hold fewer waves), and the code of segments, which a batch
// has none of, costs two chunks 14 % (4 volumes of 512^3, s = 3, BF16 4.05 / 3.55
// ms).  32 mixed volumes of 128^3..512^3, BF16: two rows 33.9 ms, four 21.8.
template <int CHMAX, int STORE, int RPT>
__global__ __launch_bounds__(256) void k_decimate_batch(DecimBatchArgs a) {
    const int nblk = gridDim.x;
    const int chunk = nblk / 8;
    const int b = blockIdx.x;
    const int lblk = (b & 7) * chunk + (b >> 3);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task = lblk * 4 + wave;
    if (task >= a.ntasks) return;
    const int2 bv = uniform_load(a.block_vol + lblk);   // (volume, first task of the volume)
    const DecimVol dv = uniform_load(a.vols + bv.x);    // wave-uniform: scalar registers
    const int t = task - bv.y;
    if (t >= dv.ntasks) return;                         // padding of the volume's range
    const int lane = threadIdx.x & 63;
    if (CHMAX >= 8 && dv.chunks >= 8) decimate_task<(CHMAX >= 8 ? 8 : 1), STORE, false, 2, false, 1, false>(dv, t, lane);
    else if (CHMAX >= 4 && dv.chunks >= 4) decimate_task<(CHMAX >= 4 ? 4 : 1), STORE, false, 2, false, 1, false>(dv, t, lane);
    else if (CHMAX >= 2 && dv.chunks >= 2) decimate_task<(CHMAX >= 2 ? 2 : 1), STORE, false, 2, false, 2, false>(dv, t, lane);
    else decimate_task<1, STORE, false, 2, false, RPT, false>(dv, t, lane);
}

template <int CH, bool CONE, int NW, bool CUBIC, int RPT>
static void launch_rows(const DecimVol& a, int store, dim3 grid, hipStream_t st) {
    switch (store) {
        case 0: hipLaunchKernelGGL((k_decimate<CH, 0, CONE, NW, CUBIC, RPT>), grid, dim3(256), 0, st, a); break;
        case 1: hipLaunchKernelGGL((k_decimate<CH, 1, CONE, NW, CUBIC, RPT>), grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_decimate<CH, 2, CONE, NW, CUBIC, RPT>), grid, dim3(256), 0, st, a); break;
    }
}

template <int CH, bool CONE, int NW, bool CUBIC>
static void launch_shape(const DecimVol& a, int store, dim3 grid, hipStream_t st) {
    if constexpr (CH > 1) {
        launch_rows<CH, CONE, NW, CUBIC, decim_rows_per_lane(CH, CONE)>(a, store, grid, st);
    } else {
        switch (a.rpt) {
            case 1: launch_rows<CH, CONE, NW, CUBIC, 1>(a, store, grid, st); break;
            case 2: launch_rows<CH, CONE, NW, CUBIC, 2>(a, store, grid, st); break;
            default: launch_rows<CH, CONE, NW, CUBIC, 4>(a, store, grid, st); break;
        }
    }
}

template <int CH, int NW>
static void launch_nw(const DecimVol& a, int store, dim3 grid, hipStream_t st) {
    if (a.cone) {
        if (a.cubic) launch_shape<CH, true, NW, true>(a, store, grid, st);
        else launch_shape<CH, true, NW, false>(a, store, grid, st);
    } else {
        if (a.cubic) launch_shape<CH, false, NW, true>(a, store, grid, st);
        else launch_shape<CH, false, NW, false>(a, store, grid, st);
    }
}

// false when no kernel exists for the chunk count and window count
template <int CH>
static bool launch_ch(const DecimVol& a, int store, dim3 grid, hipStream_t st) {
    switch (a.nw) {
        case 2: launch_nw<CH, 2>(a, store, grid, st); return true;
        case 4: if constexpr (CH <= kDecimMaxChunksWide) { launch_nw<CH, 4>(a, store, grid, st); return true; }
                return false;
        case 6: if constexpr (CH <= kDecimMaxChunksWide) { launch_nw<CH, 6>(a, store, grid, st); return true; }
                return false;
        default: return false;
    }
}

template <int CH, int RPT>
static void launch_rows_batch(const DecimBatchArgs& a, int store, dim3 grid, hipStream_t st) {
    switch (store) {
        case 0: hipLaunchKernelGGL((k_decimate_batch<CH, 0, RPT>), grid, dim3(256), 0, st, a); break;
        case 1: hipLaunchKernelGGL((k_decimate_batch<CH, 1, RPT>), grid, dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_decimate_batch<CH, 2, RPT>), grid, dim3(256), 0, st, a); break;
    }
}

template <int CH>
static void launch_ch_batch(const DecimBatchArgs& a, int store, dim3 grid, hipStream_t st) {
    if (a.rpt == 4) launch_rows_batch<CH, 4>(a, store, grid, st);
    else launch_rows_batch<CH, 2>(a, store, grid, st);
}

static dim3 decimate_grid(int ntasks) {
    const int blocks = (ntasks + 3) / 4;
    return dim3(((blocks + 7) / 8) * 8);   // a multiple of 8 for the XCD order
}

hipError_t launch_decimate(const DecimVol& a, int chunks, int store, hipStream_t st) {
    const dim3 grid = decimate_grid(a.ntasks);
    bool ok = false;
    switch (chunks) {
        case 1: ok = launch_ch<1>(a, store, grid, st); break;
        case 2: ok = launch_ch<2>(a, store, grid, st); break;
        case 4: ok = launch_ch<4>(a, store, grid, st); break;
        case 8: ok = launch_ch<8>(a, store, grid, st); break;
        default: break;
    }
    if (!ok) return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_decimate_batch(const DecimBatchArgs& a, int chunks, int store, hipStream_t st) {
    const dim3 grid = decimate_grid(a.ntasks);
    switch (chunks) {
        case 1: launch_ch_batch<1>(a, store, grid, st); break;
        case 2: launch_ch_batch<2>(a, store, grid, st); break;
        case 4: launch_ch_batch<4>(a, store, grid, st); break;
        case 8: launch_ch_batch<8>(a, store, grid, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace fdkod
