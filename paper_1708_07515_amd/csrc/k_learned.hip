// Learned angular decimation and its training kernels (gfx950).
//
// The paper leaves the low-pass filter of the angular decimation open (Sec. 2.1:
// quality depends on the low-pass filter's implementation).  The learned filter
// adds a correction R to the plain triangle decimation T of every square q and
// detector row v:
//
//   Y_q[m][v][j] = T[m][j] + R[m][j],   R = conv2(ReLU(conv1(S)))
//   conv1: H_k(p, j) = b1_k + sum_{a,b} W1[k][a][b] S((p + (a-2) d) mod P, j + b - 2)
//   R(m, j) = b2 + sum_{k,a,b} W2[k][a][b] A_k((c(m) + (a-2) d) mod P, j + b - 2)
//
// with S the cropped, shifted full-rate sub-sinogram (Sec. 2.1), A = ReLU(H)
// on the columns [0, W) and zero outside, c(m) the original angle nearest to
// the decimated angle m, d = max(1, D / 4), 16 channels, 5 x 5 taps.
//
// Matrix cores.  conv1 is a BF16 MFMA product per 16 columns,
//   H^T[16 ch][16 col] = W1[16 ch][32 taps] x X^T[32 taps][16 col]
// (X^T gathers S at the taps), FP32 accumulation.  Its output layout (lane l
// holds channels 4(l/16)..+3 of column l%16) is exactly the B-operand layout
// of a second MFMA, which contracts the channels of conv2:
//   Q[b][col] += W2_a[16 (b, 5 used)][16 ch] x A^T[16 ch][16 col]
// over the five dilated angles a; then R[j] = b2 + sum_b Q[b][j+b-2].  The
// forward pass uses the K = 32 product (one per conv1 angle, three for conv2
// with two angles per product), the training pass the K = 16 one.  The weight
// gradient of conv1 is an MFMA reduction over positions:
//   dW1^T[32 taps][16 ch] += X[taps][16 pos] x dH[16 pos][16 ch].
// Weights are BF16 (817 values: W1 [16][5][5], b1 [16], W2 [16][5][5], b2).
//
// One workgroup per (square, row) walks the decimated angles m.  The S values
// of the nine original angles c(m) + (t - 4) d, t = 0..8, are kept in LDS as
// BF16 (the precision conv1 multiplies them in).  The next angle's S values
// and output row are loaded into registers before the current angle's matrix
// products, so the global-memory latency of one angle overlaps the
// arithmetic of the previous one; when the decimated angles fall on original
// ones the forward pass fetches only the four rows that the next angle adds.
#include <algorithm>

#include "internal.h"
#include "dtype.h"
#include "geom.h"

namespace fdkod {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kSP = 16 * ((kLearnedMaxWidth + 15) / 16) + 4;  // LDS pitch of the Q rows (general forward)
constexpr int kOffW1 = 0, kOffB1 = 400, kOffW2 = 416, kOffB2 = 816;
constexpr int kThreads = 256;
static_assert(kLearnedMaxWidth + 4 <= kThreads, "one thread per staged column");

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// FP32 -> BF16, round to nearest even (hardware conversion)
__device__ __forceinline__ uint16_t f2bf(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

// c(m) = floor(m P / P' + 1/2) = floor((2 m P + P') / (2 P')), walked in m
// with an integer quotient and remainder (c(m) < P for m < P').
struct CentreWalk {
    int c, rem, dq, dr, den;
    __device__ CentreWalk(int p, int pd) {
        den = 2 * pd;
        dq = (2 * p) / den;
        dr = (2 * p) % den;
        c = pd / den;      // m = 0: floor(P' / 2P') = 0
        rem = pd % den;
    }
    __device__ void next() {
        c += dq;
        rem += dr;
        if (rem >= den) {
            rem -= den;
            ++c;
        }
    }
};

// One row of S at the thread's column: the detector samples of the crop's
// interpolation -- two for the linear shift, four (offsets -1 .. 2) for Keys'
// cubic convolution -- and the fraction; value() is S.
template <bool CUBIC>
struct SRow {
    float x[CUBIC ? 4 : 2];
    float ph;
    __device__ __forceinline__ float value() const {
        if constexpr (CUBIC) {
            float c[4];
            keys_weights(ph, c);
            float s = c[0] * x[0];
            s = fmaf(c[1], x[1], s);
            s = fmaf(c[2], x[2], s);
            return fmaf(c[3], x[3], s);
        } else {
            return fmaf(ph, x[1] - x[0], x[0]);
        }
    }
};

// The detector samples of row p at the crop offset o and local column jj,
// each through its own range-checked load (zero outside the row; a column
// outside [0, W) takes offsets left of the row and reads zero).
template <int STORE, bool CUBIC>
__device__ __forceinline__ void srow_load(const LearnedArgs& a, int v, int p, float o, int jj, bool valid,
                                          SRow<CUBIC>& r) {
    using S = Store<STORE>;
    using T = typename S::T;
    constexpr int ES = (int)sizeof(T);
    const float of = floorf(o);
    r.ph = o - of;
    const __amdgpu_buffer_rsrc_t rs = row_rsrc((const T*)a.filt + ((size_t)p * a.nv + v) * a.n, a.n);
    constexpr int K = CUBIC ? 4 : 2, LO = CUBIC ? -1 : 0;
    const int off0 = valid ? ((int)of + jj + LO) * ES : -(K + 2) * ES;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        int off = off0 + i * ES;
        if (i > 0) asm volatile("" : "+v"(off));   // separately range-checked loads, never one wider load
        r.x[i] = S::raw(rs, off);
    }
}

// The nine rows of S for centre angle c at the thread's column jj: detector
// samples x0, x1 and the (row-uniform) interpolation fraction.  offr[t]: the
// row offsets (t - 4) d mod P.  Rows are read through buffer resources that
// span exactly one detector row, so samples outside the detector, and every
// sample of a column outside [0, W) (given a negative offset), read zero.
template <int STORE, bool CUBIC>
__device__ __forceinline__ void s_fetch_rows(const LearnedArgs& a, const float* acq, float u0f, int v, int c,
                                             int jj, bool valid, const int offr[9], SRow<CUBIC> (&rows)[9]) {
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        int p = c + offr[t];
        if (p >= a.p) p -= a.p;
        srow_load<STORE, CUBIC>(a, v, p, const_load(acq + p) + u0f, jj, valid, rows[t]);
    }
}

// The forward pass keeps the nine S rows in a pair layout: entry x of row t
// holds the BF16 values of staged columns x (low half) and x + 1 (high half),
// so one 32-bit LDS load gives a lane two of its conv1 taps.  Its K order
// groups the taps in horizontal pairs: pair pi = 3 a + e (a = 0..4, e = 0..2)
// holds taps (a, 2e) and (a, 2e + 1), where tap (a, 5) has weight zero; pair
// (0, 3) pads the K dimension (weight zero; the entries beyond the staged
// columns stay at the zeros the tile was cleared to).
constexpr int kPP = 16 * ((kLearnedMaxWidth + 15) / 16) + 8;   // pitch in pairs (index 16 ntile + 5 read)
static_assert(kPP >= kThreads + 1, "every staged column has a pair entry");

struct FwdSmem {
    int off_tab[9];
    uint32_t sp[9 * kPP];
};

// Operands of the forward pass, which runs on the K = 32 BF16 MFMA
// (16x16x32: a lane of group g = lane / 16 holds eight K slots of its row or
// column; the product pairs A's and B's slots of the same lane group and
// element, so any K order common to both is valid).
//   conv1: lane group g holds two dominoes of pairs, a horizontal one (pairs
//          (a, e) and (a, e + 1), two entries apart) and a vertical one
//          ((a, e) and (a + 1, e), one row apart), so that each is one
//          two-address LDS load into consecutive registers.  The eight
//          dominoes cover the 15 pairs and one padding pair (0, 3), i.e.
//          taps (0, 6) and (0, 7), whose weights are zero like tap (a, 5).
//          Slot (g, i): pair k = i / 2 of the group (H first, H second,
//          V first, V second), half i % 2.
//   conv2: K = two dilated angles x 16 channels, three products t = 0..2;
//          slot (g, i) is channel 4 g + i % 4 of angle 2 t + i / 4 (angle 5:
//          weight zero), which is exactly how conv1's outputs for angles 2 t
//          and 2 t + 1 sit in the lane (channels 4 g .. 4 g + 3 of its column).
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

// first pairs (a, e) of each group's horizontal and vertical domino
__device__ constexpr int kDomH[4][2] = {{0, 0}, {0, 2}, {1, 1}, {4, 1}};
__device__ constexpr int kDomV[4][2] = {{1, 0}, {2, 1}, {2, 2}, {3, 0}};

struct FwdOperands {
    bf8v w1;          // A of conv1: row = channel lr
    bf8v w2[3];       // A of conv2: row = R offset b = lr (0..4 used)
    f4v b1;           // conv1 bias of the lane's output channels 4 g .. 4 g + 3
    int hoff, voff;   // the lane's dominoes in a tile of pitch PP (column lr)
};

template <int PP>
__device__ __forceinline__ FwdOperands load_fwd_operands(const uint16_t* w) {
    const int lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    FwdOperands op;
    s8v w1;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = i / 2;
        const int* dom = k < 2 ? kDomH[lg] : kDomV[lg];
        const int ta = dom[0] + (k == 3 ? 1 : 0), e = dom[1] + (k == 1 ? 1 : 0);
        const int tb = 2 * e + (i & 1);
        w1[i] = tb < 5 ? (short)w[kOffW1 + lr * 25 + ta * 5 + tb] : (short)0;
    }
    op.w1 = __builtin_bit_cast(bf8v, w1);
    op.hoff = kDomH[lg][0] * PP + 2 * kDomH[lg][1] + lr;
    op.voff = kDomV[lg][0] * PP + 2 * kDomV[lg][1] + lr;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        s8v w2;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int a2 = 2 * t + i / 4, ch = 4 * lg + i % 4;
            w2[i] = lr < 5 && a2 < 5 ? (short)w[kOffW2 + ch * 25 + a2 * 5 + lr] : (short)0;
        }
        op.w2[t] = __builtin_bit_cast(bf8v, w2);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) op.b1[i] = bf2f(w[kOffB1 + 4 * lg + i]);
    return op;
}

// Stage the thread's column x of the nine rows: the low half of pair x and
// the high half of pair x - 1.
template <bool CUBIC>
__device__ __forceinline__ void s_stage_pairs(uint32_t* sp, int x, const SRow<CUBIC> (&rows)[9]) {
    uint16_t* h = reinterpret_cast<uint16_t*>(sp);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const uint16_t v = f2bf(rows[t].value());
        h[2 * (t * kPP + x)] = v;
        if (x > 0) h[2 * (t * kPP + x - 1) + 1] = v;
    }
}

// ReLU of a conv1 output (FP32, bias included) as the BF16 B operand of
// conv2.  Rounding commutes with ReLU, so the values are rounded first and
// the negative BF16 codes (sign bit set: negative as 16-bit integers) are then
// cleared by a packed integer maximum with zero.
__device__ __forceinline__ s4v relu_bf16(f4v h) {
    typedef float f2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
    typedef short s2v __attribute__((ext_vector_type(2)));
    const s2v zero = {0, 0};
    const s2v lo = __builtin_elementwise_max(
        __builtin_bit_cast(s2v, __builtin_convertvector((f2v){h[0], h[1]}, bf2v)), zero);
    const s2v hi = __builtin_elementwise_max(
        __builtin_bit_cast(s2v, __builtin_convertvector((f2v){h[2], h[3]}, bf2v)), zero);
    return (s4v){lo[0], lo[1], hi[0], hi[1]};
}

// One 16-column tile of the forward pass for the nine S rows starting at sp
// (pair layout, row pitch PP): conv1 at the five dilated angles (five
// independent MFMAs, the bias as the initial accumulator), ReLU, conv2 (three
// MFMAs); Q rows 0..4 go to qt (row pitch QP, column c at index c + 2) for
// the columns inside [0, W) only: outside, A and hence Q are zero, and the Q
// tile keeps the zeros it was cleared to.
template <int PP, int QP>
__device__ __forceinline__ void fwd_tile(const uint32_t* sp, float* qt, int col0, int width,
                                         const FwdOperands& op) {
    typedef uint32_t u4v __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const uint32_t* ph = sp + col0 + op.hoff;
    const uint32_t* pv = sp + col0 + op.voff;
    f4v h[5];
#pragma unroll
    for (int a2 = 0; a2 < 5; ++a2) {
        const u4v d = {ph[a2 * PP], ph[a2 * PP + 2], pv[a2 * PP], pv[a2 * PP + PP]};
        h[a2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op.w1, __builtin_bit_cast(bf8v, d), op.b1, 0, 0, 0);
    }
    f4v qacc = {0.0f, 0.0f, 0.0f, 0.0f};
    const s4v zero = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const s4v lo = relu_bf16(h[2 * t]);
        const s4v hi = t < 2 ? relu_bf16(h[2 * t + 1]) : zero;
        const s8v act = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        qacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op.w2[t], __builtin_bit_cast(bf8v, act), qacc, 0, 0, 0);
    }
    if (col0 + lr < width) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int bb = 4 * lg + i;
            if (bb < 5) qt[bb * QP + col0 + lr + 2] = qacc[i];
        }
    }
}

// XCD-aware task order of the forward kernels.  Workgroups are dealt to the
// XCDs round-robin (workgroup b to XCD b mod 8), so the workgroups of XCD x
// take the detector rows v = x (mod 8), all squares of a row consecutively:
// the overlapping crops of one detector row read the same filtered rows, and
// that XCD's L2 then fetches them once.  Grid: nsq * 8 * ceil(N / 8); the
// workgroups with v >= N exit at once.
__device__ __forceinline__ bool fwd_task(const LearnedArgs& a, int& q, int& v) {
    const int x = (int)blockIdx.x % kXcds, i = (int)blockIdx.x / kXcds;
    q = i % a.nsq;
    v = (i / a.nsq) * kXcds + x;
    return v < a.nv;
}

__host__ __device__ inline unsigned fwd_grid(const LearnedArgs& a) {
    return (unsigned)a.nsq * kXcds * ((a.nv + kXcds - 1) / kXcds);
}

// Forward (inference): Y(m) += R(m) for every decimated angle of one
// (square, row).  Thread t stages column t - 2 of the tile and owns output
// column t; the waves share the 16-column tiles.  This form fetches the nine
// S rows of every angle; k_learned_fwd_ring below reuses them when the
// decimated angles fall on original ones.
template <int STORE, bool CUBIC>
__global__ __launch_bounds__(kThreads) void k_learned_fwd(LearnedArgs a) {
    using S = Store<STORE>;
    using T = typename S::T;
    __shared__ FwdSmem sm;
    __shared__ float q_tile[5 * kSP];
    int q, v;
    if (!fwd_task(a, q, v)) return;
    const int2 gd = a.grid[q];
    const int u0 = gd.x, width = gd.y;
    const int wave = threadIdx.x >> 6;
    const FwdOperands op = load_fwd_operands<kPP>(a.w);
    const float b2 = bf2f(a.w[kOffB2]);
    const int ntile = (width + 15) >> 4;
    // the crop offset of projection p is a_c(beta_p) + u0 (a_c from the
    // bounds, read through scalar loads where it is used)
    const float* acq = a.ac_p + (size_t)q * a.p;
    const float u0f = (float)u0;
    if (threadIdx.x < 9) {
        int off = ((int)threadIdx.x - 4) * a.d % a.p;
        sm.off_tab[threadIdx.x] = off < 0 ? off + a.p : off;
    }
    for (int e = threadIdx.x; e < 9 * kPP; e += kThreads) sm.sp[e] = 0u;
    for (int e = threadIdx.x; e < 5 * kSP; e += kThreads) q_tile[e] = 0.0f;
    const int col = threadIdx.x;               // staged column index (local column col - 2)
    const int jj = col - 2;
    const bool stager = col < width + 4;
    const bool valid = jj >= 0 && jj < width;
    T* ws = (T*)a.ws;
    const size_t yrow = (size_t)a.squares[q].y_off_row * a.nv + (size_t)v * width;   // + m n W + j
    const size_t yplane = (size_t)a.nv * width;
    const int j = threadIdx.x;                                           // output column
    CentreWalk cw(a.p, a.pd);
    __syncthreads();
    int offr[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) offr[t] = __builtin_amdgcn_readfirstlane(sm.off_tab[t]);

    SRow<CUBIC> rows[9];
    s_fetch_rows<STORE, CUBIC>(a, acq, u0f, v, cw.c, jj, valid, offr, rows);
    float y_cur = j < width ? S::load(ws, yrow + j) : 0.0f;
    if (stager) s_stage_pairs(sm.sp, col, rows);
    vmem_drain();
    __syncthreads();
    for (int m = 0; m < a.pd; ++m) {
        const bool more = m + 1 < a.pd;
        float y_next = 0.0f;
        if (more) {
            cw.next();
            s_fetch_rows<STORE, CUBIC>(a, acq, u0f, v, cw.c, jj, valid, offr, rows);
            if (j < width) y_next = S::load(ws, yrow + (size_t)(m + 1) * yplane + j);
        }
#pragma unroll
        for (int k = 0; k < kPP / 64; ++k) {
            const int tile = wave + 4 * k;
            if (tile < ntile) fwd_tile<kPP, kSP>(sm.sp, q_tile, tile * 16, width, op);
        }
        __syncthreads();
        if (j < width) {
            float r = b2;
#pragma unroll
            for (int bb = 0; bb < 5; ++bb) r += q_tile[bb * kSP + j + bb];
            S::put(ws, yrow + (size_t)m * yplane + j, y_cur + r);
        }
        if (more && stager) s_stage_pairs(sm.sp, col, rows);
        vmem_drain();
        y_cur = y_next;
        __syncthreads();
    }
}

// Row reuse.  When D divides P and D >= 4 (so d = D / 4), c(m) = m D and the
// nine S rows of angle m are the rows u = 4m .. 4m + 8 of the sequence
// p(u) = (u - 4) d mod P: consecutive angles share five rows.  The rows live
// in a ring of 16 LDS slots, row u in slot u mod 16; windows start at slots
// 0, 4, 8 and 12, so mirroring slots 0..4 at 16..20 makes every window of
// nine contiguous.  Each angle fetches
// its successor's four new rows and stages them while its own products run
// (their slots, and mirrors, lie outside its window), and the Q tile
// alternates between two buffers, so one barrier per angle orders the whole
// pipeline.  PW: the widest square's tiles (128, 224 or 256 columns; 224
// keeps five workgroups per compute unit within the LDS).
constexpr int kRing = 16;
constexpr int kRingMirror = 5;
constexpr int kRingSlots = kRing + kRingMirror;

template <int PW>
struct RingSmem {
    static constexpr int kPitch = PW + 8;   // pairs: a tile reads up to index 16 ntile + 5
    static constexpr int kQPitch = PW + 4;  // Q rows: columns -2 .. 16 ntile + 1
    uint32_t sp[kRingSlots * kPitch];
    float qb[2][5 * kQPitch];
};
// The ring kernel stages the crop offsets of all P projections in LDS beside
// its tile (64 KB per workgroup): up to this many projections; more take the
// general kernel, which reads each offset where it is used.
constexpr int kRingMaxP = (65536 - (int)sizeof(RingSmem<256>)) / 4;
static_assert(kRingMaxP >= 2048, "ring tile and offset table fit the LDS of a workgroup");

// Row p of S at the thread's staged column (local column jj): the two
// detector samples and the interpolation fraction (zero outside the row and
// for columns outside [0, W), as s_fetch_rows).
template <int STORE, bool CUBIC>
__device__ __forceinline__ void ring_fetch(const LearnedArgs& a, const float* o_tab, int v, int p, int jj,
                                           bool valid, SRow<CUBIC>& r) {
    srow_load<STORE, CUBIC>(a, v, p, o_tab[p], jj, valid, r);
}

// Stage the thread's column x of one row into ring slot `slot` (and its
// mirror): the low half of pair x and the high half of pair x - 1.
template <int PP, bool CUBIC>
__device__ __forceinline__ void ring_stage(uint32_t* sp, int slot, int x, const SRow<CUBIC>& r) {
    uint16_t* h = reinterpret_cast<uint16_t*>(sp);
    const uint16_t val = f2bf(r.value());
    h[2 * (slot * PP + x)] = val;
    if (x > 0) h[2 * (slot * PP + x - 1) + 1] = val;
    if (slot < kRingMirror) {
        h[2 * ((slot + kRing) * PP + x)] = val;
        if (x > 0) h[2 * ((slot + kRing) * PP + x - 1) + 1] = val;
    }
}

template <int STORE, int PW, bool CUBIC>
__global__ __launch_bounds__(kThreads) void k_learned_fwd_ring(LearnedArgs a) {
    using S = Store<STORE>;
    using T = typename S::T;
    using R = RingSmem<PW>;
    constexpr int PP = R::kPitch, QP = R::kQPitch;
    __shared__ R sm;
    extern __shared__ float o_tab[];     // [P]: a_c(beta_p) + u0
    int q, v;
    if (!fwd_task(a, q, v)) return;
    const int2 gd = a.grid[q];
    const int u0 = gd.x, width = gd.y;
    const int wave = threadIdx.x >> 6;
    const FwdOperands op = load_fwd_operands<PP>(a.w);
    const float b2 = bf2f(a.w[kOffB2]);
    const int ntile = (width + 15) >> 4;
    for (int p = threadIdx.x; p < a.p; p += kThreads) o_tab[p] = a.ac_p[(size_t)q * a.p + p] + (float)u0;
    for (int e = threadIdx.x; e < kRingSlots * PP; e += kThreads) sm.sp[e] = 0u;
    for (int e = threadIdx.x; e < 2 * 5 * QP; e += kThreads) (&sm.qb[0][0])[e] = 0.0f;
    const int x = threadIdx.x;                 // staged column index (local column x - 2)
    const int jj = x - 2;
    const bool stager = x < width + 4;
    const bool valid = jj >= 0 && jj < width;
    T* ws = (T*)a.ws;
    const size_t yrow = (size_t)a.squares[q].y_off_row * a.nv + (size_t)v * width;   // + m n W + j
    const size_t yplane = (size_t)a.nv * width;
    const int j = threadIdx.x;                                           // output column
    const int d = a.d;
    int pn = (a.p - (4 * d) % a.p) % a.p;      // p(0) = -4 d mod P
    __syncthreads();
    {
        SRow<CUBIC> rows[9];
#pragma unroll
        for (int u = 0; u < 9; ++u) {
            ring_fetch<STORE, CUBIC>(a, o_tab, v, pn, jj, valid, rows[u]);
            pn += d;
            if (pn >= a.p) pn -= a.p;
        }
        if (stager) {
#pragma unroll
            for (int u = 0; u < 9; ++u) ring_stage<PP, CUBIC>(sm.sp, u, x, rows[u]);
        }
        vmem_drain();
    }
    float y_cur = j < width ? S::load(ws, yrow + j) : 0.0f;
    __syncthreads();
    for (int m = 0; m < a.pd; ++m) {
        const bool more = m + 1 < a.pd;
        SRow<CUBIC> rows[4];
        float y_next = 0.0f;
        if (more) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ring_fetch<STORE, CUBIC>(a, o_tab, v, pn, jj, valid, rows[k]);
                pn += d;
                if (pn >= a.p) pn -= a.p;
            }
            if (j < width) y_next = S::load(ws, yrow + (size_t)(m + 1) * yplane + j);
        }
        const uint32_t* win = sm.sp + ((4 * m) & (kRing - 1)) * PP;
        float* qt = sm.qb[m & 1];
        // a fixed number of tile slots per wave (no inner loop: the prefetched
        // rows stay in flight across the products); PW / 16 tiles over four
        // waves, rounded up (PW = 224: 14 tiles, four slots per wave)
#pragma unroll
        for (int k = 0; k < (PW / 16 + 3) / 4; ++k) {
            const int tile = wave + 4 * k;
            if (tile < ntile) fwd_tile<PP, QP>(win, qt, tile * 16, width, op);
        }
        if (more && stager) {
#pragma unroll
            for (int k = 0; k < 4; ++k) ring_stage<PP, CUBIC>(sm.sp, (4 * m + 9 + k) & (kRing - 1), x, rows[k]);
        }
        vmem_drain();
        __syncthreads();
        if (j < width) {
            float r = b2;
#pragma unroll
            for (int bb = 0; bb < 5; ++bb) r += qt[bb * QP + j + bb];
            S::put(ws, yrow + (size_t)m * yplane + j, y_cur + r);
        }
        y_cur = y_next;
    }
}

// Backward (training): gradients of sum_{m,v,j} R[m][v][j] dY[m][v][j] with
// respect to the weights (dY = dL/dY in FP32, workspace layout), accumulated
// into grad.  A workgroup takes (square, row) tasks in the forward kernels'
// XCD-aware order with a grid stride, walks each task's decimated angles with
// the forward's staging and operands, and keeps its gradient partials in
// registers until all its tasks are done.
//
// conv1 runs in the transposed orientation, H[col][ch] = X[col][taps] x
// W1^T[taps][ch] (the forward's operands with their roles swapped), so a lane
// holds columns 4g .. 4g + 3 of channel lr.  That is the B-operand layout of a
// product over columns, so every reduction over positions is an MFMA:
//   dW2^T_a[b][ch] += G^T[b][col] x A_a[col][ch],   G[col][b] = dR[col - b + 2]
//   dA_a[col][ch]   = G[col][b] x W2_a^T[b][ch]      (b = 0..4)
//   dW1^T[tap][ch] += X^T[tap][col] x dH[col][ch]
// All are BF16 products with FP32 accumulation.  A, W2, S and the rounded dH
// are BF16 already; dR is FP32 and enters as the sum of three BF16 parts
// (8 significant bits each: 24, so the parts add up to dR exactly from |dR| =
// 2^-103 on, below which the third leaves BF16's normal range), which the
// row's staging splits once.  dA's three parts times five offsets fill
// one K = 16 product, dW2 takes two K = 32 ones (two parts, the third), and
// dW1 two angles in each K = 32 one: 26 matrix instructions per tile of 16
// columns, against 45 (30 of them FP32 ones of twice the time) before.
// Columns outside [0, W) have dR operands of zero.  db1 is a per-lane sum of
// dH, reduced over the lane groups at the end.
//
// RING: the forward's row reuse (its conditions): four new rows per angle,
// fetched while the current angle is computed and staged into the ring slots
// outside its window, dR in two buffers, one barrier per angle.  Otherwise
// the next angle's nine rows are fetched during the current one and staged
// after it.  Without the prefetch every angle waited for its rows: 32-slice
// slab at 2000^2, s = 4: 28.0 ms.
//
// Waves per SIMD: the linear shift is held to four, although the registers
// then spill 44 (ring) or 108 bytes per lane: the fourth wave is worth more
// (N = 300, s = 3: ring, 360 projections 2.53 ms against 2.97 without scratch
// at three; general, 362 projections 3.47 against 3.98; N = 2000, 36 rows 3.88
// against 4.63).  The cubic shift's rows hold four samples each, so its spills
// were three times those of the ring and cost more than the waves gave: two
// waves are asked for (ring 3.63 -> 3.20 ms; general 7.45 -> 4.64, and 6.55
// before the rows were fetched ahead).
constexpr int bwd_waves(bool cubic) { return cubic ? 2 : 4; }
constexpr int kDrPad = 4;                           // dR row: column c at index c + 4
constexpr int kDrLen = 16 * ((kLearnedMaxWidth + 15) / 16) + 16;

template <bool RING>
struct BwdSmem {
    uint32_t sp[(RING ? kRingSlots : 9) * kPP];
    uint32_t dr[RING ? 2 : 1][3][kDrLen];           // the parts in the pair layout (columns x and x + 1)
    int off_tab[9];
};

template <int STORE, bool CUBIC, bool RING>
__global__ __launch_bounds__(kThreads, bwd_waves(CUBIC)) void k_learned_bwd(LearnedArgs a) {
    // the task state, and after the last task the waves' partial gradients
    __shared__ union {
        BwdSmem<RING> s;
        float red[4 * kLearnedParams];
    } smu;
    BwdSmem<RING>& sm = smu.s;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const FwdOperands op = load_fwd_operands<kPP>(a.w);
    const float b1l = bf2f(a.w[kOffB1 + lr]);             // bias of the lane's channel
    // dA: K slot s = 4 g + i is part s / 5 of dR at offset b = s % 5 (slot 15:
    // weight zero); B operand W2[ch = lr][a2][b], A operand read at gco
    s4v w2op[5];
    int gco[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int sl = min(4 * lg + i, 14);
        gco[i] = 2 * ((sl / 5) * kDrLen + kDrPad + lr - sl % 5 + 2);       // in 16-bit halves
#pragma unroll
        for (int a2 = 0; a2 < 5; ++a2)
            w2op[a2][i] = 4 * lg + i < 15 ? (short)a.w[kOffW2 + lr * 25 + a2 * 5 + sl % 5] : (short)0;
    }
    const int gto = kDrPad + 4 * lg - min(lr, 4) + 2;       // dW2: columns 4 g .. of row b = lr (rows above 4 are discarded)
    // the lane's dW1 rows: taps lr and lr + 16 (taps >= 25 read a valid
    // tile entry and give discarded rows)
    int xoff[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int tap = lr + 16 * mt;
        xoff[mt] = tap < 25 ? (tap / 5) * kPP + tap % 5 + 4 * lg : 4 * lg;
    }
    f4v gw1[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
    f4v gw2[5];
#pragma unroll
    for (int a2 = 0; a2 < 5; ++a2) gw2[a2] = (f4v){0.0f, 0.0f, 0.0f, 0.0f};
    float gb1 = 0.0f, gb2 = 0.0f;

    typedef uint32_t u2v __attribute__((ext_vector_type(2)));
    typedef uint32_t u4v __attribute__((ext_vector_type(4)));
    // one tile of 16 columns: S rows at sp, dR parts at dr
    auto tile_grad = [&](const uint32_t* sp, const uint32_t* dr, int col0, int width) {
        u2v gt[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const uint32_t* g = dr + t * kDrLen + col0 + gto;
            gt[t] = (u2v){g[0], g[2]};
        }
        const uint16_t* dh16 = reinterpret_cast<const uint16_t*>(dr) + 2 * col0;
        s4v gc = {(short)dh16[gco[0]], (short)dh16[gco[1]], (short)dh16[gco[2]], (short)dh16[gco[3]]};
        if (col0 + 16 > width) {                           // uniform: the last tile
            const int left = width - (col0 + 4 * lg);      // columns of the lane's four inside [0, W)
            const uint32_t m0 = left >= 2 ? 0xFFFFFFFFu : (left == 1 ? 0xFFFFu : 0u);
            const uint32_t m1 = left >= 4 ? 0xFFFFFFFFu : (left == 3 ? 0xFFFFu : 0u);
#pragma unroll
            for (int t = 0; t < 3; ++t) gt[t] &= (u2v){m0, m1};
            if (col0 + lr >= width) gc = (s4v){0, 0, 0, 0};
        }
        const bf8v gt01 = __builtin_bit_cast(bf8v, (u4v){gt[0][0], gt[0][1], gt[1][0], gt[1][1]});
        const bf8v gt2 = __builtin_bit_cast(bf8v, (u4v){gt[2][0], gt[2][1], 0u, 0u});
        const uint32_t* ph = sp + col0 + op.hoff;
        const uint32_t* pv = sp + col0 + op.voff;
        u2v dhp = {0u, 0u}, xp[2];
#pragma unroll
        for (int a2 = 0; a2 < 5; ++a2) {
            const u4v d = {ph[a2 * kPP], ph[a2 * kPP + 2], pv[a2 * kPP], pv[a2 * kPP + kPP]};
            const f4v b1v = {b1l, b1l, b1l, b1l};
            // H[col0 + 4 g + i][ch = lr], bias included
            const f4v h =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, d), op.w1, b1v, 0, 0, 0);
            // A = ReLU(H) rounded to BF16 (the value conv2 multiplies)
            const s4v act = relu_bf16(h);
            const s8v act2 = {act[0], act[1], act[2], act[3], act[0], act[1], act[2], act[3]};
            gw2[a2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gt01, __builtin_bit_cast(bf8v, act2), gw2[a2], 0, 0, 0);
            // (the same K = 32 instruction for the third part: measured, a K = 16
            // product right behind the K = 32 one it accumulates onto read two of
            // its four sums before they were written)
            gw2[a2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gt2, __builtin_bit_cast(bf8v, act2), gw2[a2], 0, 0, 0);
            const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
            const f4v da = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(gc, w2op[a2], zero, 0, 0, 0);
            float dh[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dh[i] = h[i] > 0.0f ? da[i] : 0.0f;
                gb1 += dh[i];
            }
            // B operand of dW1: dH[col0 + 4 g + i][ch = lr] in BF16; A operand: S
            // of tap lr + 16 mt at columns col0 + 4 g .. + 3 (pair entries x and
            // x + 2 hold staged columns x .. x + 3)
            typedef float f2v __attribute__((ext_vector_type(2)));
            typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
            const u2v dhop = {__builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){dh[0], dh[1]}, bf2v)),
                              __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){dh[2], dh[3]}, bf2v))};
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const uint32_t* e = sp + a2 * kPP + col0 + xoff[mt];
                const u2v x = {e[0], e[2]};
                if (a2 == 4) {
                    gw1[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                        __builtin_bit_cast(s4v, x), __builtin_bit_cast(s4v, dhop), gw1[mt], 0, 0, 0);
                } else if (a2 & 1) {
                    gw1[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf8v, (u4v){xp[mt][0], xp[mt][1], x[0], x[1]}),
                        __builtin_bit_cast(bf8v, (u4v){dhp[0], dhp[1], dhop[0], dhop[1]}), gw1[mt], 0, 0, 0);
                } else {
                    xp[mt] = x;
                }
            }
            dhp = dhop;
            // (the next angle's operand loads stay behind: moved ahead of these
            // products they cost the fourth wave per SIMD its registers)
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const unsigned ntot = fwd_grid(a);
    for (unsigned task = blockIdx.x; task < ntot; task += gridDim.x) {
        const int x8 = (int)(task % kXcds), i8 = (int)(task / kXcds);
        const int q = i8 % a.nsq, v = (i8 / a.nsq) * kXcds + x8;
        if (v >= a.nv) continue;                           // uniform over the workgroup
        const int2 gd = a.grid[q];
        const int u0 = gd.x, width = gd.y;
        const int ntile = (width + 15) >> 4;
        __syncthreads();                                   // the previous task's reads are done
        const float* acq = a.ac_p + (size_t)q * a.p;   // crop offsets a_c(beta_p) + u0
        const float u0f = (float)u0;
        if (!RING && threadIdx.x < 9) {
            int off = ((int)threadIdx.x - 4) * a.d % a.p;
            sm.off_tab[threadIdx.x] = off < 0 ? off + a.p : off;
        }
        for (int e = threadIdx.x; e < (RING ? kRingSlots : 9) * kPP; e += kThreads) sm.sp[e] = 0u;
        for (int e = threadIdx.x; e < (RING ? 2 : 1) * 3 * kDrLen; e += kThreads) (&sm.dr[0][0][0])[e] = 0u;
        const int col = threadIdx.x;                        // staged column (local column col - 2)
        const int jj = col - 2;
        const bool stager = col < width + 4;
        const bool valid = jj >= 0 && jj < width;
        const size_t yrow = (size_t)a.squares[q].y_off_row * a.nv + (size_t)v * width;
        const size_t yplane = (size_t)a.nv * width;
        // the row of dR at the thread's column, and its three parts into buffer b
        auto load_dr = [&](int m) { return col < width ? a.dws[yrow + (size_t)m * yplane + col] : 0.0f; };
        auto stage_dr = [&](int b, float g) {
            gb2 += g;
            if (col >= width) return;
            // each part is the leading eight bits of what the ones before leave
            // (cut off, not rounded: a value near the largest stays finite)
            float part[3];
            part[0] = g;
#pragma unroll
            for (int t = 1; t < 3; ++t) part[t] = part[t - 1] - __uint_as_float(__float_as_uint(part[t - 1]) & 0xFFFF0000u);
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                uint16_t* h = reinterpret_cast<uint16_t*>(sm.dr[b][t]);
                const uint16_t val = (uint16_t)(__float_as_uint(part[t]) >> 16);
                h[2 * (kDrPad + col)] = val;
                h[2 * (kDrPad + col - 1) + 1] = val;
            }
        };
        __syncthreads();
        if constexpr (RING) {
            int pn = (a.p - (4 * a.d) % a.p) % a.p;        // p(0) = -4 d mod P
            auto fetch = [&](SRow<CUBIC>& r) {
                srow_load<STORE, CUBIC>(a, v, pn, const_load(acq + pn) + u0f, jj, valid, r);
                pn += a.d;
                if (pn >= a.p) pn -= a.p;
            };
            {
                SRow<CUBIC> rows[9];
#pragma unroll
                for (int u = 0; u < 9; ++u) fetch(rows[u]);
                const float g = load_dr(0);
                if (stager) {
#pragma unroll
                    for (int u = 0; u < 9; ++u) ring_stage<kPP, CUBIC>(sm.sp, u, col, rows[u]);
                }
                stage_dr(0, g);
                vmem_drain();
            }
            __syncthreads();
            for (int m = 0; m < a.pd; ++m) {
                const bool more = m + 1 < a.pd;
                SRow<CUBIC> rows[4];
                float g = 0.0f;
                if (more) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) fetch(rows[k]);
                    g = load_dr(m + 1);
                }
                const uint32_t* win = sm.sp + ((4 * m) & (kRing - 1)) * kPP;
#pragma unroll 1
                for (int tile = wave; tile < ntile; tile += kThreads / 64)
                    tile_grad(win, &sm.dr[m & 1][0][0], tile * 16, width);
                if (more) {
                    if (stager) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            ring_stage<kPP, CUBIC>(sm.sp, (4 * m + 9 + k) & (kRing - 1), col, rows[k]);
                    }
                    stage_dr((m + 1) & 1, g);
                }
                vmem_drain();
                __syncthreads();
            }
        } else {
            CentreWalk cw(a.p, a.pd);
            int offr[9];
#pragma unroll
            for (int t = 0; t < 9; ++t) offr[t] = __builtin_amdgcn_readfirstlane(sm.off_tab[t]);
            SRow<CUBIC> rows[9];
            s_fetch_rows<STORE, CUBIC>(a, acq, u0f, v, cw.c, jj, valid, offr, rows);
            float g = load_dr(0);
            for (int m = 0; m < a.pd; ++m) {
                if (stager) s_stage_pairs(sm.sp, col, rows);
                stage_dr(0, g);
                vmem_drain();
                __syncthreads();
                if (m + 1 < a.pd) {
                    cw.next();
                    s_fetch_rows<STORE, CUBIC>(a, acq, u0f, v, cw.c, jj, valid, offr, rows);
                    g = load_dr(m + 1);
                }
#pragma unroll 1
                for (int tile = wave; tile < ntile; tile += kThreads / 64)
                    tile_grad(sm.sp, &sm.dr[0][0][0], tile * 16, width);
                __syncthreads();
            }
        }
    }
    // the wave's partials: dW1^T[tap = 4 g + i + 16 mt][ch = lr],
    // dW2^T[b = 4 g + i][ch = lr] per angle, db1 of channel lr, db2 -- each
    // parameter held by exactly one lane of the wave.  They are summed over
    // the four waves in a fixed order and written as the workgroup's partial
    // gradient; k_grad_sum adds the workgroups' partials in a fixed order, so
    // the gradient does not depend on scheduling.
    __syncthreads();                                       // the last task's reads of sm are done
    float* red = smu.red;                                  // [4][kLearnedParams]
    float* mine = red + wave * kLearnedParams;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int tap = 16 * mt + 4 * lg + i;
            if (tap < 25) mine[kOffW1 + lr * 25 + tap] = gw1[mt][i];
        }
#pragma unroll
    for (int a2 = 0; a2 < 5; ++a2)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = 4 * lg + i;
            if (b < 5) mine[kOffW2 + lr * 25 + a2 * 5 + b] = gw2[a2][i];
        }
    gb1 += __shfl_xor(gb1, 16, 64);
    gb1 += __shfl_xor(gb1, 32, 64);
    if (lg == 0) mine[kOffB1 + lr] = gb1;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) gb2 += __shfl_xor(gb2, off, 64);
    if (lane == 0) mine[kOffB2] = gb2;
    __syncthreads();
    for (int e = threadIdx.x; e < kLearnedParams; e += kThreads)
        a.partials[(size_t)blockIdx.x * kLearnedParams + e] =
            ((red[e] + red[kLearnedParams + e]) + red[2 * kLearnedParams + e]) + red[3 * kLearnedParams + e];
}

// grad[e] = sum over the backward pass's workgroups of their partials, in a
// fixed order: sixteen threads take every sixteenth workgroup each, their
// sums are added in thread order.  (One thread per parameter walked all 1024
// workgroups, one dependent load after the other: 240-320 us.)
constexpr int kGradSeg = 16;
__global__ __launch_bounds__(16 * kGradSeg) void k_grad_sum(const float* partials, int nblocks, float* grad) {
    __shared__ float part[kGradSeg][16];
    const int i = threadIdx.x & 15, seg = threadIdx.x >> 4;
    const int e = blockIdx.x * 16 + i;
    float acc = 0.0f;
    if (e < kLearnedParams) {
#pragma unroll 8
        for (int b = seg; b < nblocks; b += kGradSeg) acc += partials[(size_t)b * kLearnedParams + e];
    }
    part[seg][i] = acc;
    __syncthreads();
    if (seg == 0 && e < kLearnedParams) {
        for (int k = 1; k < kGradSeg; ++k) acc += part[k][i];
        grad[e] = acc;
    }
}

// Transpose of the backprojection of decimated data (training): for every
// voxel and decimated angle, the residual is scattered with the bilinear
// weights and (pi / P') U^-2 into dY (workspace layout).  The sums are exact
// integer sums of the FP32 contributions rounded to multiples of 2^-e
// (fixed point in int64; e from a bound of the largest possible sum, so
// that no partial sum overflows), converted to FP32 at the end: the result
// does not depend on the order in which the atomics land.  One workgroup
// per 16 x 16 (x, y) tile of a square and slab of 32 slices (the
// backprojection's blocks).  Per angle, the block's contributions are summed
// in an LDS tile over its detector footprint, whose origin the block's
// corners bound (the column is linear-fractional in x and y, the row linear
// in z), and the tile is then added to dY with one int64 global atomic per
// non-zero entry.  A sample outside the tile (not expected) goes to dY
// directly, so the result does not depend on the bound.  The block's
// residuals sit in LDS, and in step k lane l takes slice (k + l) mod 32, so
// the lanes of one LDS atomic fall on different rows and columns of the tile
// (with one slice per step they would share a row and, several at a time, a
// column, and the atomics would serialize).  A thread sums each detector
// row of its column pair in registers and adds it once, about one row per
// slice instead of two.
constexpr int kAdjZR = 32, kAdjTW = 40, kAdjTH = 48;

// max |resid| over the voxels, as the bits of a non-negative float: one
// atomic per workgroup (one per wave of 1024 workgroups queued on the one
// address: 40 us for 2e5 voxels)
__global__ __launch_bounds__(256) void k_adj_absmax(const float* resid, int64_t count, AdjScale* qs) {
    __shared__ unsigned part[4];
    unsigned m = 0;
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        m = max(m, __float_as_uint(resid[i]) & 0x7FFFFFFFu);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) m = max(m, (unsigned)__shfl_xor((int)m, off, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = max(max(part[0], part[1]), max(part[2], part[3]));
        if (m) atomicMax(&qs->rmax, m);
    }
}

// clears the maximum and the sums' buffer (a fill kernel, no memset node)
__global__ void k_adj_clear(AdjScale* qs, unsigned long long* dq, int64_t count) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 == 0) qs->rmax = 0u;
    for (int64_t i = i0; i < count; i += (int64_t)gridDim.x * blockDim.x) dq[i] = 0ull;
}

// qscale = 2^e, the largest power of two with bound * max |resid| * qscale < 2^61
__global__ void k_adj_scale(AdjScale* qs, double bound) {
    const unsigned bits = qs->rmax;
    double q;
    if (bits >= 0x7F800000u) {
        q = 0.0;                                  // not finite: the result is NaN
    } else if (bits == 0u) {
        q = 1.0;                                  // all zero
    } else {
        int x;
        (void)frexp(bound * (double)__uint_as_float(bits), &x);   // the product < 2^x
        q = ldexp(1.0, 61 - x);
    }
    qs->qscale = q;
}

// dY = the int64 sums / qscale, rounded once to FP32
__global__ void k_adj_convert(const unsigned long long* dq, const AdjScale* qs, float* dws, int64_t count) {
    // qscale is a power of two: its reciprocal and the products are exact (a
    // 64-bit division per entry took 1.0 ms where the traffic takes 0.7)
    const double q = qs->qscale, rq = 1.0 / q;
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        dws[i] = q > 0.0 ? (float)((double)(long long)dq[i] * rq) : __builtin_nanf("");
}

__global__ __launch_bounds__(256) void k_bp_adjoint(AdjArgs a) {
    __shared__ unsigned long long acc[kAdjTH * kAdjTW];
    __shared__ float rs[kAdjZR][256];          // residual of slice l0 + k, voxel threadIdx.x
    const int tile = (int)(blockIdx.x % (unsigned)a.ntiles), zt = (int)(blockIdx.x / (unsigned)a.ntiles);
    const BpTile tl = a.tiles[tile];
    const SquareDesc sq = a.squares[tl.sq];
    const int2 gd = a.grid[tl.sq];
    const int u0 = gd.x, width = gd.y;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int ix1 = min(tl.x0 + 15, sq.x1 - 1), iy1 = min(tl.y0 + 15, sq.y1 - 1);
    const int i = tl.x0 + tx, j = tl.y0 + ty;
    const bool own = i <= ix1 && j <= iy1;
    const int l0 = zt * kAdjZR, l1 = min(l0 + kAdjZR, a.nz) - 1;
    const float dx = (float)min(i, ix1) - a.cu - sq.xc, dy = (float)min(j, iy1) - a.cu - sq.yc;
    const float bx[2] = {(float)tl.x0 - a.cu - sq.xc, (float)ix1 - a.cu - sq.xc};
    const float by[2] = {(float)tl.y0 - a.cu - sq.yc, (float)iy1 - a.cu - sq.yc};
    const float z0 = (float)(a.zbase + l0) - a.cz, z1 = (float)(a.zbase + l1) - a.cz;
    // the block's residuals (slices l0 .. l0 + 31; zero outside the square or volume)
#pragma unroll 8
    for (int k = 0; k < kAdjZR; ++k) {
        const int l = l0 + k;
        rs[k][threadIdx.x] = own && l <= l1 ? a.resid[((size_t)l * a.n + j) * a.n + i] : 0.0f;
    }
    const int skew = threadIdx.x & 63;
    const double qscale = a.qs->qscale;
    // a contribution as an integer multiple of 1 / qscale (qscale is a power
    // of two: the product is exact, the conversion rounds to nearest)
    auto fixed = [&](float v) { return (unsigned long long)__double2ll_rn((double)v * qscale); };
    for (int m = 0; m < a.pd; ++m) {
        const float2 t = a.trig[m];
        const float dc = a.r + sq.xc * t.x + sq.yc * t.y;
        const float lc = sq.yc * t.x - sq.xc * t.y;
        const float rdc = 1.0f / dc;
        // footprint origin: the least column and row over the block's corners, less a margin
        float tlo = INFINITY, vlo = INFINITY;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float cx = bx[c & 1], cy = by[c >> 1];
            tlo = fminf(tlo, rel_column(cx, cy, t.x, t.y, a.r, dc, lc, rdc) + a.cu - (float)u0);
            const float iuc = a.r / (dc + cx * t.x + cy * t.y);
            vlo = fminf(vlo, fminf(z0 * iuc, z1 * iuc) + a.cv);
        }
        const int c0 = (int)floorf(tlo) - 1, r0 = (int)floorf(vlo) - 1;
        const size_t plane = (size_t)sq.y_off_row * a.nv + (size_t)m * a.nv * width;
        for (int e = threadIdx.x; e < kAdjTH * kAdjTW; e += 256) acc[e] = 0ull;
        __syncthreads();
        if (own) {
            const float tau = rel_column(dx, dy, t.x, t.y, a.r, dc, lc, rdc) + a.cu - (float)u0;
            const float d = dc + dx * t.x + dy * t.y;
            const float invu = a.r / d;
            const float wgt = a.scale * invu * invu;
            const float tf = floorf(tau), fu = tau - tf;
            const int iu = min(max((int)tf, 0), width - 2);
            const int cl = iu - c0;
            const bool cin = cl >= 0 && cl + 1 < kAdjTW;
            // one detector row's sum (columns iu and iu + 1 by the fixed split
            // 1 - fu, fu) into the tile, or into dY when outside it; rows
            // outside the detector are dropped
            auto flush_row = [&](int row, float val) {
                if (val == 0.0f || (unsigned)(row - a.v0) >= (unsigned)a.nv) return;
                const int rl = row - r0;
                const unsigned long long q0 = fixed(val * (1.0f - fu)), q1 = fixed(val * fu);
                if (cin && rl >= 0 && rl < kAdjTH) {
                    atomicAdd(&acc[rl * kAdjTW + cl], q0);
                    atomicAdd(&acc[rl * kAdjTW + cl + 1], q1);
                } else {
                    unsigned long long* p = a.dq + plane + (size_t)(row - a.v0) * width + iu;
                    atomicAdd(p, q0);
                    atomicAdd(p + 1, q1);
                }
            };
            // the slices in order (from the lane's skew, wrapping once) move
            // the row down monotonically: rows rc and rc + 1 are summed in
            // registers and written once the slices have passed them
            int rc = INT_MIN / 2;
            float s0 = 0.0f, s1 = 0.0f;
            for (int k = 0; k < kAdjZR; ++k) {
                const int sl = (k + skew) & (kAdjZR - 1);
                if (sl == 0 && k > 0) {              // the wrap back to slice 0
                    flush_row(rc, s0);
                    flush_row(rc + 1, s1);
                    s0 = s1 = 0.0f;
                    rc = INT_MIN / 2;
                }
                const float rv = rs[sl][threadIdx.x];
                if (rv == 0.0f) continue;
                const float vv = fmaf((float)(a.zbase + l0 + sl) - a.cz, invu, a.cv);
                const float vf = floorf(vv), fv = vv - vf;
                const int iv = (int)vf;
                if (iv != rc) {
                    flush_row(rc, s0);
                    if (iv == rc + 1) {
                        s0 = s1;
                    } else {
                        flush_row(rc + 1, s1);
                        s0 = 0.0f;
                    }
                    s1 = 0.0f;
                    rc = iv;
                }
                const float w = wgt * rv;
                s0 = fmaf(w, 1.0f - fv, s0);
                s1 = fmaf(w, fv, s1);
            }
            flush_row(rc, s0);
            flush_row(rc + 1, s1);
        }
        __syncthreads();
        // non-zero entries lie at rows in [v0, v0 + nv) and columns in
        // [0, W): only such samples were added
        for (int e = threadIdx.x; e < kAdjTH * kAdjTW; e += 256) {
            const unsigned long long val = acc[e];
            if (val != 0ull)
                atomicAdd(&a.dq[plane + (size_t)(r0 - a.v0 + e / kAdjTW) * width + (c0 + e % kAdjTW)], val);
        }
        __syncthreads();
    }
}

// The transpose in two separable steps, for blocks whose footprint fits 32 x
// 32 samples (every source not close to the volume).  Workgroup = a 16 x 16
// tile, a run of zr slices and a part of the angles.  Per angle:
//
//  1. rows: every voxel column (x, y) sums its residuals onto the detector rows
//     they lie between, weighted by (pi / P') U^-2 -- a scan along z in
//     registers, each row stored once -- into H[voxel][row] in LDS.
//  2. columns: entry (row, column) gathers w(tau - column) H[voxel][row] over the
//     voxels within one column.  Those lie between two rays, i.e. between two
//     straight lines of the tile, so along the axis that the column changes
//     faster with, each of the 16 voxel lines has them in a run of at most four,
//     whose start is linear in the line's index.  A thread owns one column and
//     four rows (one 128-bit LDS read per voxel).
//
// A line's at most four terms are added in FP32 (as the rows' are), the lines
// in FP64, and the block's sum is rounded once to a multiple of 1 / qscale and
// added to the int64 sums: the result depends on no order.  Against 64-bit sums
// the error measured 1.3 to 7 times below the scatter's over ten geometries of
// N = 32..320 (relative RMS, random residuals: N = 320 1.09e-5 / 1.69e-6, N = 96
// 2.92e-6 / 1.31e-6; smooth ones, N = 96 4.8e-7 / 2.0e-7).  No LDS atomics: the scatter form
// above spends its time on their conflicts and on a 64-bit conversion for
// each term (2600 VALU instructions per thread and angle); bound here: VALU
// issue (about 900 per thread and angle), then the LDS.
// 32-slice slab at 2000^2, s = 4: 22.3 ms scattered, 8.75 gathered; 96 x 96 x 24
// voxels, 32 angles: 648 us, 29.
constexpr int kGatZ = kAdjGatherZ, kGatRows = kAdjGatherRows;
static_assert(kGatRows == 32 && kAdjGatherCols == 32, "thread = one column and four rows");
constexpr int kGatPitch = kGatRows + 4;    // words of a voxel's rows
constexpr int kGatLine = 16 * kGatPitch + 4;   // words of a line of 16 voxels
constexpr int kGatChunk = 16;              // angles whose constants are computed together
constexpr float kGatMargin = 0.01f;        // of a sample: far above the coordinates' rounding

struct GatAngle {
    float ax, ay, cs, sn;       // R (dL Dc - Lc dD) / Dc = ax dx + ay dy; cos, sin
    float dc, kc, kr;           // Dc, c_u - u0 - c0, c_v - r0
    int c0, r0, nrows, xdom;    // footprint's first column and row, rows; 1: the column changes faster along x
};

__global__ __launch_bounds__(256, 4) void k_bp_adjoint_gather(AdjArgs a) {
    __shared__ float4 hbuf[16 * kGatLine / 4];
    __shared__ float taus[256 + 16];
    __shared__ GatAngle ang[kGatChunk];
    float* H = (float*)hbuf;
    const int tid = threadIdx.x;
    // XCD-aware order: each XCD runs a contiguous range (neighbouring tiles add to the same rows)
    const int lblk = (int)(blockIdx.x & 7) * a.chunk + (int)(blockIdx.x >> 3);
    if (lblk >= a.nlogical) return;
    const int tile = lblk % a.ntiles, rest = lblk / a.ntiles;
    const int run = rest % a.nruns, part = rest / a.nruns;
    const int per = (a.pd + a.parts - 1) / a.parts;
    const int m0 = part * per, m1 = min(m0 + per, a.pd);
    const BpTile tl = a.tiles[tile];
    const SquareDesc sq = a.squares[tl.sq];
    const int2 gd = a.grid[tl.sq];
    const int u0 = gd.x, width = gd.y;
    const int tx = tid & 15, ty = tid >> 4;
    const int ix1 = min(tl.x0 + 15, sq.x1 - 1), iy1 = min(tl.y0 + 15, sq.y1 - 1);
    const int i = tl.x0 + tx, j = tl.y0 + ty;
    const bool own = i <= ix1 && j <= iy1;
    const int l0 = run * a.zr, nz = min(a.zr, a.nz - l0);
    const float bx0 = (float)tl.x0 - a.cu - sq.xc, by0 = (float)tl.y0 - a.cu - sq.yc;
    const float bx1 = (float)ix1 - a.cu - sq.xc, by1 = (float)iy1 - a.cu - sq.yc;
    const float dx = (float)min(i, ix1) - a.cu - sq.xc, dy = (float)min(j, iy1) - a.cu - sq.yc;
    const float z0 = (float)(a.zbase + l0) - a.cz, z1 = (float)(a.zbase + l0 + nz - 1) - a.cz;
    const float kq = a.cu - (float)u0;
    // the voxel column's residuals (zero outside the square)
    float rz[kGatZ];
#pragma unroll
    for (int k = 0; k < kGatZ; ++k)
        rz[k] = own && k < nz ? a.resid[((size_t)(l0 + k) * a.n + j) * a.n + i] : 0.0f;
    const double qscale = a.qs->qscale;
    const float sr2 = a.scale * a.r * a.r;
    const int c = tid & 31, rg = tid >> 5;         // step 2: the thread's column and rows 4 rg ..

    for (int m = m0; m < m1; ++m) {
        const int ci = (m - m0) & (kGatChunk - 1);
        if (ci == 0) {
            // the chunk's angles, one lane each: the footprint from the block's corners
            __syncthreads();
            if (tid < kGatChunk && m + tid < m1) {
                const float2 t = a.trig[m + tid];
                const float dc = a.r + sq.xc * t.x + sq.yc * t.y;
                const float lc = sq.yc * t.x - sq.xc * t.y;
                const float rdc = 1.0f / dc;
                const float lr = a.r * lc * rdc;
                GatAngle g;
                g.ax = -(a.r * t.y + lr * t.x);
                g.ay = a.r * t.x - lr * t.y;
                g.cs = t.x;
                g.sn = t.y;
                g.dc = dc;
                float tlo = INFINITY, vlo = INFINITY, vhi = -INFINITY;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float cx = (k & 1) ? bx1 : bx0, cy = (k & 2) ? by1 : by0;
                    const float rd = 1.0f / (dc + (cx * t.x + cy * t.y));
                    tlo = fminf(tlo, (cx * g.ax + cy * g.ay) * rd + kq);
                    const float va = z0 * a.r * rd + a.cv, vb = z1 * a.r * rd + a.cv;
                    vlo = fminf(vlo, fminf(va, vb));
                    vhi = fmaxf(vhi, fmaxf(va, vb));
                }
                g.c0 = (int)floorf(tlo - kGatMargin);
                g.r0 = (int)floorf(vlo - kGatMargin);
                g.nrows = min((int)floorf(vhi + kGatMargin) + 2 - g.r0, kGatRows);
                g.kc = kq - (float)g.c0;
                g.kr = a.cv - (float)g.r0;
                // d tau / dx and d tau / dy at the block's centre, up to a common factor
                const float mx = 0.5f * (bx0 + bx1), my = 0.5f * (by0 + by1);
                const float num = mx * g.ax + my * g.ay, d = dc + (mx * t.x + my * t.y);
                g.xdom = fabsf(g.ax * d - num * t.x) >= fabsf(g.ay * d - num * t.y);
                ang[tid] = g;
            }
            __syncthreads();
        }
        const GatAngle& g = ang[ci];
        const bool xdom = __builtin_amdgcn_readfirstlane(g.xdom) != 0;
        const int nrows = __builtin_amdgcn_readfirstlane(g.nrows);
        {
            // step 1: the voxel column's rows
            const int line = xdom ? ty : tx, pos = xdom ? tx : ty;
            float* h = H + line * kGatLine + pos * kGatPitch;
            const float d = g.dc + fmaf(dx, g.cs, dy * g.sn);
            const float rd = 1.0f / d;
            taus[line * 16 + pos] = fmaf(fmaf(dx, g.ax, dy * g.ay), rd, g.kc);
            const float w = sr2 * rd * rd, vstep = a.r * rd;
            // the whole run lies in [0, nrows - 1): the clamp only keeps the rows of
            // a block that the planner has not bounded inside H
            const float v0 = fminf(fmaxf(fmaf(z0, vstep, g.kr), 0.0f),
                                   fmaf(-(float)(nz - 1), vstep, (float)(kGatRows - 1) - kGatMargin));
#pragma unroll
            for (int e = 0; e < kGatRows / 4; ++e)
                if (4 * e < nrows) *(float4*)(h + 4 * e) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            int rc = (int)v0;
            float s0 = 0.0f, s1 = 0.0f;            // rows rc and rc + 1
#pragma unroll
            for (int k = 0; k < kGatZ; ++k) {
                if (k >= nz) break;                // uniform
                const float vv = fmaf((float)k, vstep, v0);
                const int iv = (int)vv;
                const float fv = __builtin_amdgcn_fractf(vv);
                const int adv = iv - rc;           // 0, 1 or 2: one slice moves by R / D < 2 rows
                if (adv > 0) h[rc] = s0;
                if (adv > 1) h[rc + 1] = s1;
                s0 = adv == 0 ? s0 : (adv == 1 ? s1 : 0.0f);
                s1 = adv == 0 ? s1 : 0.0f;
                rc = iv;
                const float wr = w * rz[k];
                s0 = fmaf(wr, 1.0f - fv, s0);
                s1 = fmaf(wr, fv, s1);
            }
            h[rc] = s0;
            h[rc + 1] = s1;
        }
        __syncthreads();
        if (4 * rg < nrows) {
            // step 2: P(l) = the position where line l crosses the column T:
            // tau = T where p (A1 - q C1) = q Dc + l (q C2 - A2), q = T - kc, in
            // offsets p along and l across the lines
            const float A1 = xdom ? g.ax : g.ay, A2 = xdom ? g.ay : g.ax;
            const float C1 = xdom ? g.cs : g.sn, C2 = xdom ? g.sn : g.cs;
            const float p0 = xdom ? bx0 : by0, q0 = xdom ? by0 : bx0;
            const float col = (float)c;
            float lo = 0.0f, dlo = 0.0f;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float q = (e ? col + 1.0f : col - 1.0f) - g.kc;
                const float rden = 1.0f / (A1 - q * C1);
                const float slope = (q * C2 - A2) * rden;
                const float at = fmaf(q0, slope, q * g.dc * rden) - p0;
                if (e == 0 || at < lo) {
                    lo = at;
                    dlo = slope;
                }
            }
            lo -= kGatMargin;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            const float* hrow = H + 4 * rg;
#pragma unroll 2
            for (int line = 0; line < 16; ++line) {
                const int pi = (int)fminf(fmaxf(ceilf(fmaf((float)line, dlo, lo)), 0.0f), 12.0f);
                const float* tp = taus + line * 16 + pi;
                const float* hp = hrow + line * kGatLine + pi * kGatPitch;
                float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float wt = __builtin_amdgcn_fmed3f(1.0f - fabsf(tp[k] - col), 0.0f, 1.0f);
                    const float4 hv = *(const float4*)(hp + k * kGatPitch);
                    s[0] = fmaf(wt, hv.x, s[0]);
                    s[1] = fmaf(wt, hv.y, s[1]);
                    s[2] = fmaf(wt, hv.z, s[2]);
                    s[3] = fmaf(wt, hv.w, s[3]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] += (double)s[r];
            }
            // rows outside the band and columns outside [0, W) are dropped; the
            // product is exact (qscale is a power of two), the conversion rounds
            const int oc = g.c0 + c;
            const size_t plane = (size_t)sq.y_off_row * a.nv + (size_t)m * a.nv * width;
            if (oc >= 0 && oc < width) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = g.r0 + 4 * rg + r - a.v0;
                    if (4 * rg + r < nrows && row >= 0 && row < a.nv && acc[r] != 0.0)
                        atomicAdd(a.dq + plane + (size_t)row * width + oc,
                                  (unsigned long long)__double2ll_rn(acc[r] * qscale));
                }
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_residual(const float* f, const float* ref, float* r, double* loss,
                                                   int64_t count, float weight) {
    __shared__ double part[4];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float dlt = f[i] - ref[i];
        r[i] = (2.0f * weight) * dlt;
        acc += (double)dlt * (double)dlt;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(loss, (double)weight * (part[0] + part[1] + part[2] + part[3]));
}

__global__ void k_fill_d(double* p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.0;
}

// AdamW on the FP32 master weights; writes their BF16 copy.
__global__ void k_adamw(AdamArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    const float g = a.grad[i];
    float m1 = a.m1[i] = a.beta1 * a.m1[i] + (1.0f - a.beta1) * g;
    float m2 = a.m2[i] = a.beta2 * a.m2[i] + (1.0f - a.beta2) * g * g;
    const float mh = m1 / (1.0f - powf(a.beta1, (float)a.step));
    const float vh = m2 / (1.0f - powf(a.beta2, (float)a.step));
    float w = a.master[i];
    w -= a.lr * (mh / (sqrtf(vh) + a.eps) + a.weight_decay * w);
    a.master[i] = w;
    a.w_bf16[i] = (uint16_t)f2bf(w);
}

template <int STORE, bool CUBIC>
void launch_fwd_ring(const LearnedArgs& a, int max_width, hipStream_t st) {
    const size_t dyn = sizeof(float) * (size_t)a.p;
    if (max_width <= 128)
        hipLaunchKernelGGL((k_learned_fwd_ring<STORE, 128, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), dyn, st, a);
    else if (max_width <= 224)
        hipLaunchKernelGGL((k_learned_fwd_ring<STORE, 224, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), dyn, st, a);
    else
        hipLaunchKernelGGL((k_learned_fwd_ring<STORE, 256, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), dyn, st, a);
}

template <bool CUBIC>
void launch_fwd_store(const LearnedArgs& a, int max_width, bool ring, int store, hipStream_t st) {
    if (ring) {
        switch (store) {
            case 0: launch_fwd_ring<0, CUBIC>(a, max_width, st); break;
            case 1: launch_fwd_ring<1, CUBIC>(a, max_width, st); break;
            default: launch_fwd_ring<2, CUBIC>(a, max_width, st); break;
        }
        return;
    }
    switch (store) {
        case 0: hipLaunchKernelGGL((k_learned_fwd<0, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), 0, st, a); break;
        case 1: hipLaunchKernelGGL((k_learned_fwd<1, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), 0, st, a); break;
        default: hipLaunchKernelGGL((k_learned_fwd<2, CUBIC>), dim3(fwd_grid(a)), dim3(kThreads), 0, st, a); break;
    }
}

// consecutive decimated angles share five of their nine S rows (see above)
bool ring_rows(const LearnedArgs& a, int dfac) {
    return dfac >= 4 && a.p % dfac == 0 && a.pd * dfac == a.p && a.d * 4 == dfac;
}

hipError_t launch_learned_fwd(const LearnedArgs& a, int max_width, int dfac, int store, hipStream_t st) {
    if (max_width > kLearnedMaxWidth) return hipErrorInvalidValue;
    const bool ring = ring_rows(a, dfac) && a.p <= kRingMaxP;
    if (a.cubic) launch_fwd_store<true>(a, max_width, ring, store, st);
    else launch_fwd_store<false>(a, max_width, ring, store, st);
    return hipGetLastError();
}

// Workgroups of the backward pass: a grid stride over the tasks, a multiple of
// the XCD count (so a workgroup's tasks stay on its XCD's rows), about four
// per compute unit.
constexpr unsigned kBwdGrid = kLearnedBwdGrid;

template <int STORE>
void launch_bwd(const LearnedArgs& a, bool ring, dim3 grid, hipStream_t st) {
    if (ring) {
        if (a.cubic) hipLaunchKernelGGL((k_learned_bwd<STORE, true, true>), grid, dim3(kThreads), 0, st, a);
        else hipLaunchKernelGGL((k_learned_bwd<STORE, false, true>), grid, dim3(kThreads), 0, st, a);
    } else {
        if (a.cubic) hipLaunchKernelGGL((k_learned_bwd<STORE, true, false>), grid, dim3(kThreads), 0, st, a);
        else hipLaunchKernelGGL((k_learned_bwd<STORE, false, false>), grid, dim3(kThreads), 0, st, a);
    }
}

hipError_t launch_learned_bwd(const LearnedArgs& a, int dfac, int store, hipStream_t st) {
    if (!a.partials) return hipErrorInvalidValue;
    const bool ring = ring_rows(a, dfac);
    const unsigned ntot = fwd_grid(a);
    const dim3 grid(ntot < kBwdGrid ? ntot : kBwdGrid);
    switch (store) {
        case 0: launch_bwd<0>(a, ring, grid, st); break;
        case 1: launch_bwd<1>(a, ring, grid, st); break;
        default: launch_bwd<2>(a, ring, grid, st); break;
    }
    hipLaunchKernelGGL(k_grad_sum, dim3((kLearnedParams + 15) / 16), dim3(16 * kGradSeg), 0, st, a.partials,
                       (int)grid.x, a.grad);
    return hipGetLastError();
}

hipError_t launch_bp_adjoint(const AdjArgs& a, hipStream_t st) {
    const int64_t nblk = (int64_t)a.ntiles * ((a.nz + kAdjZR - 1) / kAdjZR);
    if (nblk <= 0 || nblk > (int64_t)1 << 31) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_adj_clear, dim3(1024), dim3(256), 0, st, a.qs, a.dq, a.ws_elems);
    const unsigned nmax = (unsigned)std::min<int64_t>(1024, (a.nvox + 4095) / 4096);
    hipLaunchKernelGGL(k_adj_absmax, dim3(nmax), dim3(256), 0, st, a.resid, a.nvox, a.qs);
    hipLaunchKernelGGL(k_adj_scale, dim3(1), dim3(1), 0, st, a.qs, a.bound);
    if (a.zr > 0)
        hipLaunchKernelGGL(k_bp_adjoint_gather, dim3(8u * (unsigned)a.chunk), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(k_bp_adjoint, dim3((unsigned)nblk), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_adj_convert, dim3(1024), dim3(256), 0, st, (const unsigned long long*)a.dq,
                       (const AdjScale*)a.qs, a.dws, a.ws_elems);
    return hipGetLastError();
}

hipError_t launch_residual(const float* f, const float* ref, float* r, double* loss, int64_t count, float weight,
                           hipStream_t st) {
    hipLaunchKernelGGL(k_fill_d, dim3(1), dim3(64), 0, st, loss, (int64_t)1);
    hipLaunchKernelGGL(k_residual, dim3(1024), dim3(256), 0, st, f, ref, r, loss, count, weight);
    return hipGetLastError();
}

hipError_t launch_adamw(const AdamArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(k_adamw, dim3((a.count + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace fdkod
