// loss.hip -- the float region of a segmentation training step on gfx950.
//
// The int8 logits [N,h,w,K] (one power-of-two exponent) are upsampled
// bilinearly to the label size [N,H,W] (half-pixel centres: source coordinate
// (o + 1/2) n_in / n_out - 1/2 clamped at 0, upper neighbour clamped at the
// edge), scored by the pixel-wise softmax cross-entropy (mean over the N H W
// pixels), differentiated, taken back through the adjoint of the upsampling,
// and quantized by SQ to the int8 error E1 at the logits (Eq. 4 / Eq. 16: the
// one float -> integer crossing of the dataflow).
//
// Float64 throughout, so that the integer codes decided at the end agree with
// a float64 reference except where a value sits very close to a rounding
// boundary.  A class's x-step ratio is multiplied down the rows of a cell and
// applied once per column, and both factors carry an exp's error (up to 1.35e-16)
// and a rounding (1.1e-16), so the relative error of an exp is below 2.5e-16 times
// the cell's rows times its columns, plus as much per row and column.  Measured
// in the gradient, against its largest element: 1e-15 at cells of 16 x 16, 1e-12 at
// 256 x 256, 2.5e-12 at 600 x 200.  Deterministic: every sum runs in a fixed order.
//   k_ce_cells8   one block per bilinear cell (a run of output rows that read
//   / k_ce_cells  the same two source rows x a run of columns): softmax of each
//                 pixel with lanes over classes, the gradient folded into the
//                 cell's four source corners, the cell's loss
//   k_ce_combine  one thread per low-res element: the corner sums of every cell
//                 touching it, in a fixed order -> gradient
//   k_ce_quant    SQ codes and exponent; block 0 also forms the mean loss
#include <math.h>

#include "iseg_common.h"

namespace {

// the logit exponents the region accepts: |logit| < 128, so every exp() of a
// difference of (bilinear mixes of) logits stays a normal finite double
constexpr int kLogitExpMin = -1000, kLogitExpMax = 0;
__device__ __forceinline__ bool logit_exp_ok(int32_t e) { return e >= kLogitExpMin && e <= kLogitExpMax; }


// 64-bit value moved across lanes by a DPP control (both 32-bit halves)
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double readlane_f64(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wave-wide sum, the same value in every lane: within each row of 16
// lanes by DPP steps whose pairs are symmetric (quad swaps, half-row and row
// mirrors), then the four row results added in a fixed order.
__device__ __forceinline__ double wave_sum_f64(double v)
{
    v += dpp_f64<0xB1>(v);      // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);      // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);     // row_half_mirror
    v += dpp_f64<0x140>(v);     // row_mirror
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// ---------------------------------------------------------------------------
// Runs: maximal ranges of output coordinates that read the same two source
// positions (i0, i1) with the same clamping, so that the interpolation weight
// is affine in the coordinate inside a run.  A cell is (row run) x (column
// run): its logits are bilinear in (x, y), so exp(l - m) follows a 2-D
// multiplicative recurrence: exp at one corner, the x-step ratio, the y-step
// ratio and the change of the x-step per row (4 exps per class and cell).
// ---------------------------------------------------------------------------
constexpr int kMaxRuns = 136;

struct Run {
    int16_t start, len, i0, i1;
};

struct CeCellArgs {
    const int8_t* logits;
    const int32_t* logit_exp;
    const uint8_t* labels;
    int32_t N, h, w, K, H, W;
    int32_t nry, nrx;
    Run ry[kMaxRuns];
    Run rx[kMaxRuns];
    // per low-res row / column: the (run << 1 | corner) pairs that touch it, in run
    // order, -1 past the last.  A run's corners are i0 and i1 = min(i0 + 1, n - 1),
    // and only i0 = 0 has a second (clamped) run, so there are at most four
    int16_t ey[64][4], ex[64][4];
    double* cell;        // [N][nry][nrx][4][K]: corner sums (i0,j0),(i0,j1),(i1,j0),(i1,j1)
    double* cell_loss;   // [N][nry][nrx]
    double* grad;        // [N][h][w][K]
    uint64_t* part;      // |grad| max partials, one per combine block
    int32_t* status;
};

__host__ __device__ __forceinline__ void src_coord_hd(int o, int n_in, int n_out, int& i0, int& i1, double& lam,
                                                       bool& clamped)
{
    double src = ((double)o + 0.5) * (double)n_in / (double)n_out - 0.5;
    clamped = src < 0.0;
    if (clamped) src = 0.0;
    i0 = (int)floor(src);
    i1 = i0 + 1 < n_in ? i0 + 1 : n_in - 1;
    lam = src - (double)i0;
}

// host: run table of one axis; returns the count, or -1 above kMaxRuns
static int make_runs(int n_in, int n_out, Run* runs)
{
    int n = 0, pi0 = -1, pi1 = -1;
    bool pcl = false;
    for (int o = 0; o < n_out; o++) {
        int i0, i1;
        double lam;
        bool cl;
        src_coord_hd(o, n_in, n_out, i0, i1, lam, cl);
        if (o == 0 || i0 != pi0 || i1 != pi1 || cl != pcl) {
            if (n == kMaxRuns) return -1;
            runs[n].start = (int16_t)o;
            runs[n].len = 0;
            runs[n].i0 = (int16_t)i0;
            runs[n].i1 = (int16_t)i1;
            n++;
        }
        runs[n - 1].len++;
        pi0 = i0;
        pi1 = i1;
        pcl = cl;
    }
    return n;
}

__device__ __forceinline__ double interp(double a00, double a01, double a10, double a11, double wx0, double wx1,
                                         double wy0, double wy1, double scale)
{
    const double top = wx0 * a00 + wx1 * a01;
    const double bot = wx0 * a10 + wx1 * a11;
    return (wy0 * top + wy1 * bot) * scale;
}

// One block per cell (three per CU: occupancy hides the latency of each
// cell's loads and barriers).  A wave takes P = 64 / L rows of the cell at a time, one
// row per group of L lanes; lane l of a group holds the classes l + L t
// (t < KT).  Along a row the exps follow the cell's multiplicative recurrence
// (one multiply per pixel and class), the softmax denominator is a group-wide
// sum (DPP steps within a row of 16 lanes, no readlane) and one reciprocal per
// pixel scales the gradient; two pixels of a row are in flight per step.  The
// cell's per-class constants (the exp at its first pixel, the x- and y-step
// ratios, the change of the x-step per row) are computed once per block; a
// row's starting values are integer powers of them.  The one-hot part of the
// gradient collects in LDS (one region per wave and group, added to by the
// lane that owns the pixel's label with no-return LDS atomics, so no wait),
// the corner sums of the groups are added in group order, then those of the
// waves in wave order.
constexpr int kCellWaves = 4;
constexpr int kMaxRunLen = 256;
constexpr int kLabPre = 4;        // label bytes per lane loaded ahead (a pass of up to 256 pixels)

// v + v[lane ^ O] (O = 16, 32) by gfx950's cross-row swaps; the pair comes
// back in a lane-dependent order, and the sum is the same bits either way
template <int O>
__device__ __forceinline__ double swap_sum_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    uint32_t l0, l1, h0, h1;
    if constexpr (O == 16) {
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        l0 = rl[0]; l1 = rl[1]; h0 = rh[0]; h1 = rh[1];
    } else {
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        l0 = rl[0]; l1 = rl[1]; h0 = rh[0]; h1 = rh[1];
    }
    const double x = __longlong_as_double((long long)(((uint64_t)h0 << 32) | l0));
    const double y = __longlong_as_double((long long)(((uint64_t)h1 << 32) | l1));
    return x + y;
}

template <int O>
__device__ __forceinline__ double swap_max_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    uint32_t l1, h1;
    if constexpr (O == 16) {
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        l1 = rl[0] == lo && rh[0] == hi ? rl[1] : rl[0];
        h1 = rl[0] == lo && rh[0] == hi ? rh[1] : rh[0];
    } else {
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        l1 = rl[0] == lo && rh[0] == hi ? rl[1] : rl[0];
        h1 = rl[0] == lo && rh[0] == hi ? rh[1] : rh[0];
    }
    return fmax(v, __longlong_as_double((long long)(((uint64_t)h1 << 32) | l1)));
}

// group-wide (L = 8: half a DPP row, L = 32: two) sum / max of a double, by
// steps whose partner pairs are symmetric: every lane of the group ends with
// the same bits
template <int L>
__device__ __forceinline__ double group_sum_f64(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    if constexpr (L == 32) v = swap_sum_f64<16>(v + dpp_f64<0x140>(v));
    return v;
}

template <int L>
__device__ __forceinline__ double group_max_f64(double v)
{
    v = fmax(v, dpp_f64<0xB1>(v));
    v = fmax(v, dpp_f64<0x4E>(v));
    v = fmax(v, dpp_f64<0x141>(v));
    v = fmax(v, dpp_f64<0x140>(v));
    if constexpr (L == 32) v = swap_max_f64<16>(v);
    return v;
}

// sum of a value over the P groups of a wave (lanes l, l + L, ...), the same
// bits in every lane: pairs of groups first, then pairs of pairs
template <int L>
__device__ __forceinline__ double groups_sum_f64(double v)
{
    static_assert(L == 32, "group width");
    return swap_sum_f64<32>(v);
}

// b^e, e >= 0, by squaring
__device__ __forceinline__ double pow_int(double b, int e)
{
    double r = 1.0;
    while (e) {
        if (e & 1) r *= b;
        b *= b;
        e >>= 1;
    }
    return r;
}

// pairwise sum of KT values
template <int KT>
__device__ __forceinline__ double tree_sum(const double* v)
{
    double t[KT];
#pragma unroll
    for (int i = 0; i < KT; i++) t[i] = v[i];
#pragma unroll
    for (int w = 1; w < KT; w *= 2)
#pragma unroll
        for (int i = 0; i + w < KT; i += 2 * w) t[i] += t[i + w];
    return t[0];
}

// a / s for s > 0 (a normal double, here at least exp(-256)): hardware
// reciprocal, two Newton steps and one correction of the quotient
__device__ __forceinline__ double div_pos(double a, double s)
{
    double r = __builtin_amdgcn_rcp(s);
    r = fma(fma(-s, r, 1.0), r, r);
    r = fma(fma(-s, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-s, q, a), r, q);
}

__device__ __forceinline__ void lds_add_f64(double* p, double v)
{
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// exp(x) for |x| below 2^20 (here |x| <= 256 unless the logit exponent is out of
// range, where nothing is used): x = k ln 2 + r with ln 2 in two parts (Cody and
// Waite), |r| <= ln 2 / 2, the Taylor polynomial of degree 13 (its remainder is
// below 5e-18) by Horner's rule, scaled by 2^k.  Straight-line: a fifth of the
// library call's instructions.
__device__ __forceinline__ double exp_small(double x)
{
    const double k = rint(x * 1.44269504088896340736);
    double r = fma(k, -0x1.62e42fefap-1, x);             // ln 2 to 36 bits: k times it is exact
    r = fma(k, -(0.69314718055994530942 - 0x1.62e42fefap-1 + 2.3190468138462996e-17), r);
    double p = 1.0 / 6227020800.0;
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)k);
}

// Up to 176 classes: groups of eight lanes, KT classes per lane, so a wave
// takes eight rows of the cell at once and what a pixel costs besides its
// four operations per class (the denominator's cross-lane sum, the division,
// the label) is shared by eight pixels.  Two waves per block, 16 rows per
// pass; four blocks fit a CU (40 KB of LDS at 150 classes).  One LDS region
// [row][2][8 KT] serves a pass three times: the rows' starting exps and x-step
// ratios (one thread per class multiplies them down the rows; zero past the
// last row and class, so no later step has a condition), then the one-hot sums
// (added to by the lane that owns a pixel's label, each row its own region),
// then the rows' two column sums, which one thread per class folds into the
// cell's four corners in row order.  The loss takes log(s) of a row as the log
// of the product of the mantissas plus the exponents, and the label logits from
// eight threads per row.  Bound by instruction issue, float64 at 4.5 clocks per
// wave: 1.3 G lane operations of the four per class, 41 us of 132 at 8 x 512 x
// 512 pixels and 150 classes; 313 us for rows of 32-lane groups.
constexpr int kCell8Waves = 2, kCell8Rows = kCell8Waves * 8;

template <int KT>
__global__ __launch_bounds__(64 * kCell8Waves, 2) void k_ce_cells8(const CeCellArgs a, int maxlen)
{
    constexpr int NT = 64 * kCell8Waves, RW = kCell8Rows, KP = 8 * KT, KR = (KP + NT - 1) / NT;
    constexpr bool TWO = KT <= 16;                     // two pixels in flight (registers)
    extern __shared__ __align__(16) char smem[];
    __shared__ double wl[kCell8Waves], wys[RW];
    __shared__ int smax[kCell8Waves];
    const int n = blockIdx.z, sy = blockIdx.y, sx = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lig = lane & 7, row = t >> 3;
    const int K = a.K, wk = a.w * a.K;
    const Run ry = a.ry[sy], rx = a.rx[sx];
    const int j0 = rx.i0, j1 = rx.i1, len = rx.len;
    double* reg = (double*)smem;                       // [RW][2][KP]
    double* wxs = reg + RW * 2 * KP;                   // column weight lambda_x per pixel of the run
    int8_t* C0 = (int8_t*)(wxs + maxlen);              // corner codes [4][KP]
    uint8_t* labs = (uint8_t*)(C0 + 4 * KP);           // [RW][maxlen]
    const uint8_t* lab_base = a.labels + ((int64_t)n * a.H + ry.start) * a.W + rx.start;
    const int8_t* r0 = a.logits + ((int64_t)n * a.h + ry.i0) * wk;
    const int8_t* r1 = a.logits + ((int64_t)n * a.h + ry.i1) * wk;
    const int32_t le = *a.logit_exp;
    // this thread's classes t, t + NT: corner codes to registers and LDS
    int c4[KR][4], mxc = -128;
#pragma unroll
    for (int r = 0; r < KR; r++) {
        const int k = t + r * NT, kk = k < K ? k : 0;
        c4[r][0] = r0[j0 * K + kk]; c4[r][1] = r0[j1 * K + kk];
        c4[r][2] = r1[j0 * K + kk]; c4[r][3] = r1[j1 * K + kk];
    }
    for (int c = t; c < len; c += NT) {
        int e0, e1;
        bool ecl;
        double lx;
        src_coord_hd(rx.start + c, a.w, a.W, e0, e1, lx, ecl);
        wxs[c] = lx;
    }
#pragma unroll
    for (int r = 0; r < KR; r++) {
        const int k = t + r * NT;
        mxc = max(mxc, max(max(c4[r][0], c4[r][1]), max(c4[r][2], c4[r][3])));
        if (k < KP) {
#pragma unroll
            for (int q = 0; q < 4; q++) C0[q * KP + k] = (int8_t)c4[r][q];
        }
    }
    for (int o = 32; o > 0; o >>= 1) mxc = max(mxc, __shfl_xor(mxc, o, 64));
    if (lane == 0) smax[wv] = mxc;
    __syncthreads();
    // outside the documented range the outputs are discarded (k_ce_quant)
    const double scale = logit_exp_ok(le) ? ldexp(1.0, le) : 0.0;
    const double invP = 1.0 / ((double)a.N * (double)a.H * (double)a.W);
    int mi = smax[0];
#pragma unroll
    for (int v = 1; v < kCell8Waves; v++) mi = max(mi, smax[v]);
    const double m = (double)mi * scale;               // the cell's max logit
    // per class: the current row's exp at the first pixel and x-step ratio, and
    // the factors that take them to the next row
    double e0r[KR], x0r[KR], ys[KR], xs[KR], g4[KR][4];
    {
        int d0, d1;
        bool dcl;
        double ly0, ly1;
        src_coord_hd(ry.start, a.h, a.H, d0, d1, ly0, dcl);
        src_coord_hd(ry.start + (ry.len > 1 ? 1 : 0), a.h, a.H, d0, d1, ly1, dcl);
        const double lx0 = wxs[0], lx1 = wxs[len > 1 ? 1 : 0];
#pragma unroll
        for (int r = 0; r < KR; r++) {
            const double c00 = c4[r][0], c01 = c4[r][1], c10 = c4[r][2], c11 = c4[r][3];
            const double l00 = interp(c00, c01, c10, c11, 1.0 - lx0, lx0, 1.0 - ly0, ly0, scale);
            const double l10 = interp(c00, c01, c10, c11, 1.0 - lx1, lx1, 1.0 - ly0, ly0, scale);
            const double l01 = interp(c00, c01, c10, c11, 1.0 - lx0, lx0, 1.0 - ly1, ly1, scale);
            const double l11 = interp(c00, c01, c10, c11, 1.0 - lx1, lx1, 1.0 - ly1, ly1, scale);
            e0r[r] = t + r * NT < K ? exp_small(l00 - m) : 0.0;
            x0r[r] = exp_small(l10 - l00);
            ys[r] = exp_small(l01 - l00);
            xs[r] = exp_small((l11 - l01) - (l10 - l00));
            g4[r][0] = g4[r][1] = g4[r][2] = g4[r][3] = 0.0;
        }
    }
    double lsum = 0.0;
    bool bad = false;
    for (int base = 0; base < ry.len; base += RW) {
        const int rows = min(RW, ry.len - base);
        if (base) __syncthreads();                     // the last pass's column sums are read
        const bool live = row < rows;
        // labels and row weights (eight threads per row), the rows' starting values
        for (int c = lig; c < len; c += 8)
            labs[row * maxlen + c] = live ? lab_base[(int64_t)(base + row) * a.W + c] : (uint8_t)0;
        double ly;
        {
            int q0, q1;
            bool qcl;
            src_coord_hd(ry.start + base + (live ? row : 0), a.h, a.H, q0, q1, ly, qcl);
            if (lig == 0) wys[row] = ly;
        }
#pragma unroll
        for (int r = 0; r < KR; r++) {
            const int k = t + r * NT;
            if (k < KP) {
                double* d = reg + k;
#pragma unroll 4
                for (int q = 0; q < RW; q++, d += 2 * KP) {
                    d[0] = q < rows ? e0r[r] : 0.0;
                    d[KP] = x0r[r];
                    if (q < rows) { e0r[r] *= ys[r]; x0r[r] *= xs[r]; }
                }
            }
        }
        __syncthreads();
        // label logits
        for (int c = lig; c < len; c += 8) {
            const int lab = labs[row * maxlen + c], lc = lab < K ? lab : 0;
            const double lx = wxs[c];
            const double l = interp((double)C0[lc], (double)C0[KP + lc], (double)C0[2 * KP + lc],
                                    (double)C0[3 * KP + lc], 1.0 - lx, lx, 1.0 - ly, ly, scale);
            lsum -= live && lab < K ? l : 0.0;
            bad |= lab >= K;
        }
        double* rg = reg + row * 2 * KP;
        double E[KT], R[KT], alo[KT], ahi[KT];
#pragma unroll
        for (int q = 0; q < KT; q++) {                 // read and cleared by the same lane
            E[q] = rg[lig + 8 * q];
            R[q] = rg[KP + lig + 8 * q];
            rg[lig + 8 * q] = 0.0;
            rg[KP + lig + 8 * q] = 0.0;
            alo[q] = ahi[q] = 0.0;
        }
        __builtin_amdgcn_wave_barrier();
        double prod = 1.0;
        int pexp = 0;
        const uint8_t* lab_row = labs + row * maxlen;
        // a row past the last has E = 0: its quotients are not finite and its
        // sums are not used
        auto pixel = [&](const double* Ev, double s, double lx, int lab) {
            const double cp = div_pos(invP, s);
            const double c1 = lx * cp, c0 = (1.0 - lx) * cp;
#pragma unroll
            for (int q = 0; q < KT; q++) {
                alo[q] = fma(c0, Ev[q], alo[q]);
                ahi[q] = fma(c1, Ev[q], ahi[q]);
            }
            if (lab < K && lig == (lab & 7)) {
                lds_add_f64(&rg[lab], 1.0 - lx);
                lds_add_f64(&rg[KP + lab], lx);
            }
            // mantissas in [1/2, 1): at most 256 factors stay above 2^-256
            prod *= __builtin_amdgcn_frexp_mant(s);
            pexp += __builtin_amdgcn_frexp_exp(s);
        };
        int c = 0;
        if constexpr (TWO) {
            for (; c + 1 < len; c += 2) {
                double E1[KT];
#pragma unroll
                for (int q = 0; q < KT; q++) E1[q] = E[q] * R[q];
                const double sa = group_sum_f64<8>(tree_sum<KT>(E)), sb = group_sum_f64<8>(tree_sum<KT>(E1));
                pixel(E, sa, wxs[c], lab_row[c]);
                pixel(E1, sb, wxs[c + 1], lab_row[c + 1]);
#pragma unroll
                for (int q = 0; q < KT; q++) E[q] = E1[q] * R[q];
            }
        }
        for (; c < len; c++) {
            const double sa = group_sum_f64<8>(tree_sum<KT>(E));
            pixel(E, sa, wxs[c], lab_row[c]);
#pragma unroll
            for (int q = 0; q < KT; q++) E[q] *= R[q];
        }
        const double ls = log(prod) + (double)pexp * 0.69314718055994530942;
        lsum += live && lig == 0 ? ls : 0.0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < KT; q++) {
            double* d = rg + lig + 8 * q;
            d[0] = alo[q] - d[0] * invP;
            d[KP] = ahi[q] - d[KP] * invP;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KR; r++) {
            const int k = t + r * NT;
            if (k < K) {
                const double* d = reg + k;
#pragma unroll 4
                for (int q = 0; q < rows; q++, d += 2 * KP) {
                    const double wy = wys[q], glo = d[0], ghi = d[KP];
                    g4[r][0] = fma(1.0 - wy, glo, g4[r][0]);
                    g4[r][1] = fma(1.0 - wy, ghi, g4[r][1]);
                    g4[r][2] = fma(wy, glo, g4[r][2]);
                    g4[r][3] = fma(wy, ghi, g4[r][3]);
                }
            }
        }
    }
    const int64_t cid = ((int64_t)n * a.nry + sy) * a.nrx + sx;
    double* out = a.cell + cid * 4 * K;
#pragma unroll
    for (int r = 0; r < KR; r++) {
        const int k = t + r * NT;
        if (k < K) {
#pragma unroll
            for (int q = 0; q < 4; q++) out[q * K + k] = g4[r][q];
        }
    }
    lsum = wave_sum_f64(lsum);
    if (lane == 0) wl[wv] = lsum;
    if (__any(bad) && lane == 0) set_status(a.status, ISEG_DEV_RANGE);
    __syncthreads();
    if (t == 0) {
        double ls = wl[0];
#pragma unroll
        for (int v = 1; v < kCell8Waves; v++) ls += wl[v];
        a.cell_loss[cid] = ls + m * ((double)ry.len * (double)len);
    }
}

// More classes: groups of 32 lanes.
template <int L, int KT>
__global__ __launch_bounds__(256, 3) void k_ce_cells(const CeCellArgs a)
{
    constexpr int P = 64 / L;
    static_assert(L == 32, "group width");
    extern __shared__ __align__(16) char smem[];
    __shared__ double wxs[kMaxRunLen];                     // column weight lambda_x per pixel of the run
    __shared__ double wl[kCellWaves];
    __shared__ uint8_t labs[kCellWaves][P][kMaxRunLen];    // labels of the rows a wave has in flight
    const int n = blockIdx.z, sy = blockIdx.y, sx = blockIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int grp = lane / L, lig = lane % L;
    const int K = a.K, wk = a.w * a.K;
    const Run ry = a.ry[sy], rx = a.rx[sx];
    const int j0 = rx.i0, j1 = rx.i1, len = rx.len;
    // LDS: the four corner columns of both source rows [4][K] (codes), the
    // per-class constants [4][K], and per wave P one-hot regions [2][K]
    // (reused for the wave's corner sums [4][K] at the end)
    int8_t* C0 = (int8_t*)smem;
    double* cst = (double*)(smem + ((4 * K + 15) & ~15));
    double* oh = cst + 4 * K;
    // labels of a pass (rows base .. base + P - 1 of the run): up to kLabPre
    // bytes per lane through registers, so a pass's loads can be issued early
    const uint8_t* lab_base = a.labels + ((int64_t)n * a.H + ry.start) * a.W + rx.start;
    auto lab_load = [&](int base, uint32_t* v) {
#pragma unroll
        for (int q = 0; q < kLabPre; q++) {
            const int t = lane + 64 * q, rr = base + t / len;
            v[q] = t < P * len && rr < ry.len ? lab_base[(int64_t)rr * a.W + t % len] : 0u;
        }
    };
    auto lab_store = [&](int base, const uint32_t* v) {
#pragma unroll
        for (int q = 0; q < kLabPre; q++) {
            const int t = lane + 64 * q;
            if (t < P * len) labs[wv][t / len][t % len] = (uint8_t)v[q];
        }
        for (int t = lane + 64 * kLabPre; t < P * len; t += 64) {
            const int rr = base + t / len;
            labs[wv][t / len][t % len] = rr < ry.len ? lab_base[(int64_t)rr * a.W + t % len] : (uint8_t)0;
        }
    };
    uint32_t lpre[kLabPre];
    lab_load(wv * P, lpre);
    const int8_t* r0 = a.logits + ((int64_t)n * a.h + ry.i0) * wk;
    const int8_t* r1 = a.logits + ((int64_t)n * a.h + ry.i1) * wk;
    for (int t = threadIdx.x; t < K; t += blockDim.x) {
        C0[t] = r0[j0 * K + t];
        C0[K + t] = r0[j1 * K + t];
        C0[2 * K + t] = r1[j0 * K + t];
        C0[3 * K + t] = r1[j1 * K + t];
    }
    for (int c = threadIdx.x; c < len; c += blockDim.x) {
        int e0, e1;
        bool ecl;
        double lx;
        src_coord_hd(rx.start + c, a.w, a.W, e0, e1, lx, ecl);
        wxs[c] = lx;
    }
    for (int t = threadIdx.x; t < kCellWaves * P * 2 * K; t += blockDim.x) oh[t] = 0.0;
    __syncthreads();
    // outside the documented range the outputs are discarded (k_ce_quant)
    const double scale = logit_exp_ok(*a.logit_exp) ? ldexp(1.0, *a.logit_exp) : 0.0;
    const double invP = 1.0 / ((double)a.N * (double)a.H * (double)a.W);

    // the cell's max logit (each group covers every class: the same m everywhere)
    double m = -INFINITY;
#pragma unroll
    for (int t = 0; t < KT; t++) {
        const int k = lig + L * t;
        if (k < K) m = fmax(m, fmax(fmax((double)C0[k], (double)C0[K + k]),
                                    fmax((double)C0[2 * K + k], (double)C0[3 * K + k])) * scale);
    }
    m = group_max_f64<L>(m);

    // per class: exp at the first pixel, x-step and y-step ratios, and the
    // factor by which the x-step changes from row to row
    {
        int d0, d1;
        bool dcl;
        double ly0, ly1;
        src_coord_hd(ry.start, a.h, a.H, d0, d1, ly0, dcl);
        src_coord_hd(ry.start + (ry.len > 1 ? 1 : 0), a.h, a.H, d0, d1, ly1, dcl);
        const double lx0 = wxs[0], lx1 = wxs[len > 1 ? 1 : 0];
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            const double c00 = C0[k], c01 = C0[K + k], c10 = C0[2 * K + k], c11 = C0[3 * K + k];
            const double l00 = interp(c00, c01, c10, c11, 1.0 - lx0, lx0, 1.0 - ly0, ly0, scale);
            const double l10 = interp(c00, c01, c10, c11, 1.0 - lx1, lx1, 1.0 - ly0, ly0, scale);
            const double l01 = interp(c00, c01, c10, c11, 1.0 - lx0, lx0, 1.0 - ly1, ly1, scale);
            const double l11 = interp(c00, c01, c10, c11, 1.0 - lx1, lx1, 1.0 - ly1, ly1, scale);
            cst[k] = exp(l00 - m);
            cst[K + k] = exp(l10 - l00);
            cst[2 * K + k] = exp(l01 - l00);
            cst[3 * K + k] = exp((l11 - l01) - (l10 - l00));
        }
    }
    lab_store(wv * P, lpre);
    __syncthreads();

    double G00[KT], G01[KT], G10[KT], G11[KT];
#pragma unroll
    for (int t = 0; t < KT; t++) G00[t] = G01[t] = G10[t] = G11[t] = 0.0;
    double lsum = 0.0, llab = 0.0, sv = 1.0;
    int pc = 0;
    bool bad = false;
    double* ohg = oh + (int64_t)((wv * P + grp) * 2) * K;
    const uint8_t* lab_row = labs[wv][grp];
    for (int base = wv * P; base < ry.len; base += kCellWaves * P) {
        const int row = base + grp;
        const bool live = row < ry.len;
        const bool more = base + kCellWaves * P < ry.len;
        if (more) lab_load(base + kCellWaves * P, lpre);     // the next pass's labels, in flight meanwhile
        int e0, e1;
        bool ecl;
        double ly;
        src_coord_hd(ry.start + (live ? row : 0), a.h, a.H, e0, e1, ly, ecl);
        const double wy0 = 1.0 - ly, wy1 = ly;
        double E[KT], R[KT], alo[KT], ahi[KT];
#pragma unroll
        for (int t = 0; t < KT; t++) {
            const int k = lig + L * t;
            const bool on = k < K;
            E[t] = on && live ? cst[k] * pow_int(cst[2 * K + k], row) : 0.0;
            R[t] = on ? cst[K + k] * pow_int(cst[3 * K + k], live ? row : 0) : 1.0;
            alo[t] = ahi[t] = 0.0;
        }
        // one pixel of the row: softmax part of the gradient E / s / P folded
        // into the row's two columns; one-hot part by the label's lane; the
        // loss log(s) + m - l(label), logs taken L pixels at a time and the
        // label logits at the end of the row from the one-hot weights
        auto pixel = [&](const double* Ev, double s, double lx, int lab, bool on) {
            const double cp = on ? div_pos(invP, s) : 0.0;
            const double c0 = (1.0 - lx) * cp, c1 = lx * cp;
#pragma unroll
            for (int t = 0; t < KT; t++) {
                alo[t] = fma(c0, Ev[t], alo[t]);
                ahi[t] = fma(c1, Ev[t], ahi[t]);
            }
            if (on) {
                bad |= lab >= K;
                if (lab < K && lig == lab % L) {
                    lds_add_f64(&ohg[lab], 1.0 - lx);
                    lds_add_f64(&ohg[K + lab], lx);
                }
                if ((pc % L) == lig) sv = s;
                pc++;
                if (pc % L == 0) lsum += log(sv);
            }
        };
        for (int c = 0; c < len; c += 2) {
            const bool two = c + 1 < len;
            const double lxa = wxs[c], lxb = wxs[two ? c + 1 : c];
            const int laba = lab_row[c], labb = lab_row[two ? c + 1 : c];
            double E1[KT];
#pragma unroll
            for (int t = 0; t < KT; t++) E1[t] = E[t] * R[t];
            const double sa = group_sum_f64<L>(tree_sum<KT>(E));
            const double sb = group_sum_f64<L>(tree_sum<KT>(E1));
            pixel(E, sa, lxa, laba, live);
            pixel(E1, sb, lxb, labb, live && two);
#pragma unroll
            for (int t = 0; t < KT; t++) E[t] = E1[t] * R[t];
        }
        if (live) {
#pragma unroll
            for (int t = 0; t < KT; t++) {
                const int k = lig + L * t;
                if (k < K) {
                    const double olo = ohg[k], ohi = ohg[K + k];
                    ohg[k] = 0.0;
                    ohg[K + k] = 0.0;
                    const double glo = alo[t] - olo * invP, ghi = ahi[t] - ohi * invP;
                    G00[t] += wy0 * glo;
                    G01[t] += wy0 * ghi;
                    G10[t] += wy1 * glo;
                    G11[t] += wy1 * ghi;
                    // sum over the row's pixels labelled k of l_k = the corners' bilinear mix
                    llab += (wy0 * ((double)C0[k] * olo + (double)C0[K + k] * ohi) +
                             wy1 * ((double)C0[2 * K + k] * olo + (double)C0[3 * K + k] * ohi)) * scale;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (more) lab_store(base + kCellWaves * P, lpre);
        __builtin_amdgcn_wave_barrier();
    }
    if (lig < (pc % L)) lsum += log(sv);
    lsum = wave_sum_f64(lsum - llab);
    const bool anybad = __any(bad);
    // the groups' corner sums, then this wave's into its own LDS region
    double* red = oh + (int64_t)wv * P * 2 * K;             // [4][K], within the wave's one-hot regions
#pragma unroll
    for (int t = 0; t < KT; t++) {
        const double g00 = groups_sum_f64<L>(G00[t]), g01 = groups_sum_f64<L>(G01[t]);
        const double g10 = groups_sum_f64<L>(G10[t]), g11 = groups_sum_f64<L>(G11[t]);
        const int k = lig + L * t;
        if (grp == 0 && k < K) {
            red[k] = g00;
            red[K + k] = g01;
            red[2 * K + k] = g10;
            red[3 * K + k] = g11;
        }
    }
    if (lane == 0) {
        wl[wv] = lsum;
        if (anybad) set_status(a.status, ISEG_DEV_RANGE);
    }
    __syncthreads();
    const int64_t cid = ((int64_t)n * a.nry + sy) * a.nrx + sx;
    double* out = a.cell + cid * 4 * K;
    const int64_t ws = (int64_t)P * 2 * K;
    for (int t = threadIdx.x; t < 4 * K; t += blockDim.x)
        out[t] = ((oh[t] + oh[ws + t]) + oh[2 * ws + t]) + oh[3 * ws + t];
    if (threadIdx.x == 0)
        a.cell_loss[cid] = (((wl[0] + wl[1]) + wl[2]) + wl[3]) + m * ((double)ry.len * (double)len);
}

// grad[n,i,j,k]: sum over the cells with a corner at (i, j), in the order of
// the row entries, then of the column entries; one thread per element, a block
// per 256 elements of one low-res row.  The loads of the (usually 2 x 2) first
// entries go out together (behind the branch of each cell they took a round
// trip each: 20.6 -> 12.2 us at 8 x 32 x 32 x 150).
__global__ __launch_bounds__(256) void k_ce_combine(const CeCellArgs a)
{
    const int n = blockIdx.z, i = blockIdx.y;
    const int wk = a.w * a.K;
    const int e = blockIdx.x * 256 + threadIdx.x;
    uint64_t mx = 0;
    if (e < wk) {
        const int j = e / a.K, k = e - j * a.K;
        const double* cell = a.cell + (int64_t)n * a.nry * a.nrx * 4 * a.K + k;
        auto at = [&](int y, int x) {
            const int64_t cid = (int64_t)(y >> 1) * a.nrx + (x >> 1);
            return cell[(cid * 4 + 2 * (y & 1) + (x & 1)) * a.K];
        };
        int ey[4], ex[4];
#pragma unroll
        for (int q = 0; q < 4; q++) { ey[q] = a.ey[i][q]; ex[q] = a.ex[j][q]; }
        // every low-res index is touched by at least one run
        const int y1 = ey[1] >= 0 ? ey[1] : ey[0], x1 = ex[1] >= 0 ? ex[1] : ex[0];
        const double v00 = at(ey[0], ex[0]), v01 = at(ey[0], x1), v10 = at(y1, ex[0]), v11 = at(y1, x1);
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            if (ey[q] < 0) break;
            if (q < 2) {
                acc += q ? v10 : v00;
                if (ex[1] >= 0) acc += q ? v11 : v01;
            } else {
                acc += at(ey[q], ex[0]);
                if (ex[1] >= 0) acc += at(ey[q], ex[1]);
            }
            if (ex[2] >= 0) acc += at(ey[q], ex[2]);
            if (ex[3] >= 0) acc += at(ey[q], ex[3]);
        }
        a.grad[((int64_t)n * a.h + i) * wk + e] = acc;
        mx = (uint64_t)__double_as_longlong(acc) & 0x7fffffffffffffffull;
    }
    mx = block_max_u64(mx);
    if (threadIdx.x == 0) a.part[((int64_t)n * a.h + i) * gridDim.x + blockIdx.x] = mx;
}

// smallest e with |v| < 2^e for the positive double with bits mb (frexp's exponent)
__device__ __forceinline__ int frexp_exp_bits64(uint64_t mb)
{
    const int E = (int)(mb >> 52);
    const uint64_t man = mb & 0xfffffffffffffull;
    if (E == 0) return bitlen_u64(man) - 1074;
    return E - 1022;
}

__global__ __launch_bounds__(256) void k_ce_quant(const CeCellArgs a, int64_t nparts, int bits,
                                                  int8_t* __restrict__ err, int32_t* err_exp, double* loss)
{
    const uint64_t mb = reduce_partials_u64(a.part, nparts);
    const int64_t total = (int64_t)a.N * a.h * a.w * a.K;
    const bool range_ok = logit_exp_ok(*a.logit_exp);
    if (!range_ok || mb >= 0x7ff0000000000000ull) {
        // logits outside the region's domain, or a NaN / infinite gradient:
        // flag it, zero codes, NaN loss
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            set_status(a.status, range_ok ? ISEG_DEV_NONFINITE : ISEG_DEV_RANGE);
            *err_exp = 1 - bits;
            if (loss) *loss = __longlong_as_double(0x7ff8000000000000ll);
        }
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
             e += (int64_t)gridDim.x * blockDim.x)
            err[e] = 0;
        return;
    }
    const int b = mb ? frexp_exp_bits64(mb) : 0;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) *err_exp = b + 1 - bits;
        // mean loss: cell losses summed in a fixed tree order
        __shared__ double red[256];
        double s = 0.0;
        const int64_t cells = (int64_t)a.N * a.nry * a.nrx;
        // eight loads in flight (one at a time they set the kernel's time: 17.8 -> 10.3 us)
        for (int64_t r = threadIdx.x; r < cells; r += 8 * (int64_t)blockDim.x) {
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const int64_t x = r + q * (int64_t)blockDim.x;
                v[q] = a.cell_loss[x < cells ? x : r];
            }
#pragma unroll
            for (int q = 0; q < 8; q++) s += r + q * (int64_t)blockDim.x < cells ? v[q] : 0.0;
        }
        red[threadIdx.x] = s;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0 && loss) *loss = red[0] / ((double)a.N * (double)a.H * (double)a.W);
    }
    const int sh = bits - 1 - b;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const double v = ldexp(a.grad[e], sh);      // a power-of-two scale: exact
        const double fl = floor(v);
        const double nf = fl + (v - fl >= 0.5 ? 1.0 : 0.0);
        err[e] = (int8_t)clamp_k((int64_t)nf, bits);
    }
}

template <int L, int KT>
int launch_cells(const CeCellArgs& a, hipStream_t s)
{
    const size_t lds = (size_t)((4 * a.K + 15) & ~15) + (size_t)(4 * a.K) * 8 +
                       (size_t)(kCellWaves * (64 / L) * 2 * a.K) * 8;
    if (!lds_limit((const void*)k_ce_cells<L, KT>, lds))
        return ISEG_ERR_DEVICE;
    hipLaunchKernelGGL((k_ce_cells<L, KT>), dim3((unsigned)a.nrx, (unsigned)a.nry, (unsigned)a.N), dim3(256), lds,
                       s, a);
    return launch_ok();
}

template <int KT>
int launch_cells8(const CeCellArgs& a, hipStream_t s)
{
    int maxlen = 1;
    for (int i = 0; i < a.nrx; i++) maxlen = a.rx[i].len > maxlen ? a.rx[i].len : maxlen;
    maxlen = (maxlen + 3) & ~3;
    const size_t lds = (size_t)kCell8Rows * 2 * 8 * KT * 8 + (size_t)maxlen * 8 + (size_t)4 * 8 * KT +
                       (size_t)kCell8Rows * maxlen;
    if (!lds_limit((const void*)k_ce_cells8<KT>, lds)) return ISEG_ERR_DEVICE;
    hipLaunchKernelGGL(k_ce_cells8<KT>, dim3((unsigned)a.nrx, (unsigned)a.nry, (unsigned)a.N),
                       dim3(64 * kCell8Waves), lds, s, a, maxlen);
    return launch_ok();
}

// the (run << 1 | corner) entries touching each low-res index, in run order;
// false if an index has more than four (it cannot) or none
bool run_entries(const Run* runs, int nr, int n_low, int16_t (*ent)[4])
{
    for (int i = 0; i < n_low; i++) {
        int n = 0;
        for (int q = 0; q < 4; q++) ent[i][q] = -1;
        for (int s = 0; s < nr; s++)
            for (int c = 0; c < 2; c++)
                if ((c ? runs[s].i1 : runs[s].i0) == i) {
                    if (n == 4) return false;
                    ent[i][n++] = (int16_t)(s << 1 | c);
                }
        if (!n) return false;
    }
    return true;
}

// max |grad| partials: one per combine block
int64_t ce_nparts(int64_t N, int64_t h, int64_t w, int64_t K) { return N * h * ceil_div64(w * K, 256); }

}  // namespace

// workspace: [max][cells][cell losses][grad (if not given)][max partials]
static size_t ce_cell_bytes(int64_t N, int64_t nry, int64_t nrx, int64_t K)
{
    return align256((size_t)(N * nry * nrx * 4 * K) * 8);
}

extern "C" size_t iseg_softmax_ce_ws(int64_t N, int64_t h, int64_t w, int64_t K, int64_t H, int64_t W)
{
    if (N < 1 || h < 1 || w < 1 || K < 1 || H < h || W < w || h > 64 || w > 64 || H > 32767 || W > 32767)
        return 0;
    Run tmp[kMaxRuns];
    const int nry = make_runs((int)h, (int)H, tmp), nrx = make_runs((int)w, (int)W, tmp);
    if (nry < 0 || nrx < 0) return 0;
    return 256 + ce_cell_bytes(N, nry, nrx, K) +
           align256((size_t)(N * nry * nrx) * 8) + align256((size_t)(N * h * w * K) * 8) +
           align256((size_t)ce_nparts(N, h, w, K) * 8);
}

extern "C" int iseg_softmax_ce(const int8_t* logits, const int32_t* logit_exp, const uint8_t* labels, int64_t N,
                               int64_t h, int64_t w, int64_t K, int64_t H, int64_t W, int32_t bits, double* loss,
                               double* grad, int8_t* err, int32_t* err_exp, void* ws, size_t ws_bytes,
                               int32_t* dev_status, hipStream_t stream)
{
    if (N < 1 || h < 1 || w < 1 || K < 1 || H < h || W < w || bits < 2 || bits > 8) return ISEG_ERR_ARG;
    if (!logits || !logit_exp || !labels || !err || !err_exp) return ISEG_ERR_ARG;
    if (K > 256 || h > 64 || w > 64 || H > 32767 || W > 32767 || N > 65535) return ISEG_ERR_UNSUPPORTED;
    const size_t need = iseg_softmax_ce_ws(N, h, w, K, H, W);
    if (need == 0) return ISEG_ERR_UNSUPPORTED;
    if (!ws || ws_bytes < need) return ISEG_ERR_WORKSPACE;
    CeCellArgs a{};
    a.logits = logits; a.logit_exp = logit_exp; a.labels = labels;
    a.N = (int32_t)N; a.h = (int32_t)h; a.w = (int32_t)w; a.K = (int32_t)K; a.H = (int32_t)H; a.W = (int32_t)W;
    a.nry = make_runs((int)h, (int)H, a.ry);
    a.nrx = make_runs((int)w, (int)W, a.rx);
    for (int i = 0; i < a.nrx; i++)
        if (a.rx[i].len > kMaxRunLen) return ISEG_ERR_UNSUPPORTED;
    if (!run_entries(a.ry, a.nry, (int)h, a.ey) || !run_entries(a.rx, a.nrx, (int)w, a.ex))
        return ISEG_ERR_UNSUPPORTED;
    a.status = dev_status;
    char* p = (char*)ws;
    p += 256;
    a.cell = (double*)p;
    p += ce_cell_bytes(N, a.nry, a.nrx, K);
    a.cell_loss = (double*)p;
    p += align256((size_t)(N * a.nry * a.nrx) * 8);
    double* gws = (double*)p;
    p += align256((size_t)(N * h * w * K) * 8);
    a.part = (uint64_t*)p;
    a.grad = grad ? grad : gws;
    int rc;
    // groups of 8 lanes up to 176 classes, else 32.  A class count runs at the cost
    // of its width, so the widths step by a quarter to a half, more finely where
    // the time is: 24 (four waves per SIMD), 48 and 64 (three) and 96 to 176 classes
    // (two).  22 classes per lane already spill 16 registers of two waves per SIMD;
    // still 118 us at 176 classes and 4 x 512 x 512 pixels against 218 at 177
    const int kt8 = (int)((K + 7) / 8);
    rc = kt8 <= 3    ? launch_cells8<3>(a, stream)
       : kt8 <= 6    ? launch_cells8<6>(a, stream)
       : kt8 <= 8    ? launch_cells8<8>(a, stream)
       : kt8 <= 12   ? launch_cells8<12>(a, stream)
       : kt8 <= 16   ? launch_cells8<16>(a, stream)
       : kt8 <= 19   ? launch_cells8<19>(a, stream)
       : kt8 <= 22   ? launch_cells8<22>(a, stream)
       : K <= 192    ? launch_cells<32, 6>(a, stream)
                     : launch_cells<32, 8>(a, stream);
    if (rc) return rc;
    const unsigned cx = (unsigned)ceil_div64(w * K, 256);
    hipLaunchKernelGGL(k_ce_combine, dim3(cx, (unsigned)h, (unsigned)N), dim3(256), 0, stream, a);
    if ((rc = launch_ok())) return rc;
    const int64_t nlow = N * h * w * K;
    hipLaunchKernelGGL(k_ce_quant, dim3(grid_for(nlow, 256 * 4, 512)), dim3(256), 0, stream, a,
                       ce_nparts(N, h, w, K), (int)bits, err, err_exp, loss);
    return launch_ok();
}

// ---------------------------------------------------------------------------
// MSE loss against one-hot labels (the FCN8s loss): L = mean over the N H W K
// elements of (y - t)^2, t = [k == label], and E1 = SQ(2 (y - t) / (N H W K))
// (Eq. 4 / 16) decided exactly.  With g = min(y_exp, 0), every y - t is an
// integer V on the grid 2^g: V = c 2^(y_exp - g) - t 2^-g.  The gradient is
// V 2^(g+1) / D (D = N H W K), its scale 2^u the smallest power of two above
// max|V| 2^(g+1) / D, and a code floor(V 2^(k-1-ce) / D + 1/2) with ce the
// smallest e with max|V| < D 2^e (u = ce + g + 1).  The loss is summed per
// block in float64 and the partials in a fixed order.
// ---------------------------------------------------------------------------
namespace {
struct MseArgs {
    const int8_t* y;
    const int32_t* y_exp;
    const uint8_t* labels;
    int64_t n;               // N H W K
    int32_t K;
    uint64_t* pmax;          // [gridDim.x] max |V|
    double* psum;            // [gridDim.x] sum V^2
    int32_t* status;
};

__device__ __forceinline__ int64_t mse_v(const MseArgs& a, int64_t i, int g, int ye)
{
    const int64_t pix = i / a.K;
    const int k = (int)(i - pix * a.K);
    const int lab = a.labels[pix];
    const int64_t t = lab == k ? 1 : 0;
    return (int64_t)a.y[i] * ((int64_t)1 << (ye - g)) - t * ((int64_t)1 << (-g));
}

__device__ __forceinline__ bool mse_exp_ok(int32_t e) { return e >= -60 && e <= 40; }

__global__ __launch_bounds__(256) void k_mse_part(MseArgs a)
{
    __shared__ double sd[256];
    const int32_t ye = *a.y_exp;
    const bool ok = mse_exp_ok(ye);
    if (!ok && blockIdx.x == 0 && threadIdx.x == 0) set_status(a.status, ISEG_DEV_RANGE);
    const int g = ye < 0 ? ye : 0;
    uint64_t m = 0;
    double s = 0.0;
    bool bad = false;
    if (ok)
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n;
             i += (int64_t)gridDim.x * blockDim.x) {
            bad |= a.labels[i / a.K] >= a.K;
            const int64_t v = mse_v(a, i, g, ye);
            const uint64_t av = (uint64_t)(v < 0 ? -v : v);
            m = av > m ? av : m;
            s += (double)v * (double)v;
        }
    if (bad) set_status(a.status, ISEG_DEV_RANGE);
    block_store_max_u64(m, a.pmax);
    sd[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sd[threadIdx.x] += sd[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.psum[blockIdx.x] = sd[0];
}

__global__ __launch_bounds__(256) void k_mse_codes(MseArgs a, int nparts, int bits, int8_t* __restrict__ err,
                                                   int32_t* err_exp, double* loss)
{
    const int32_t ye = *a.y_exp;
    const bool ok = mse_exp_ok(ye);
    const int g = ye < 0 ? ye : 0;
    const uint64_t M = reduce_partials_u64(a.pmax, nparts);
    const i128 D = (i128)a.n;
    const int ce = M ? ceil_pow2_exp128((i128)M, D) : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (M) {
            *err_exp = ce + g + 2 - bits;
        } else {
            int lg = 0;                              // ceil(log2 D)
            while (((int64_t)1 << lg) < a.n) lg++;
            *err_exp = g + 1 - lg;
        }
        double s = 0.0;
        for (int b = 0; b < nparts; b++) s += a.psum[b];
        if (loss) *loss = ok ? ldexp(s, 2 * g) / (double)a.n : __longlong_as_double(0x7ff8000000000000ll);
    }
    const int sh = bits - 1 - ce;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int8_t code = 0;
        if (ok && M) code = (int8_t)clamp_k128(rhu128((i128)mse_v(a, i, g, ye), sh, D), bits);
        err[i] = code;
    }
}
}  // namespace

extern "C" size_t iseg_mse_onehot_ws(int64_t n) { return n > 0 ? 256 + 2 * align256(2048 * 8) : 0; }

extern "C" int iseg_mse_onehot(const int8_t* y, const int32_t* y_exp, const uint8_t* labels, int64_t N, int64_t H,
                               int64_t W, int64_t K, int32_t bits, double* loss, int8_t* err, int32_t* err_exp,
                               void* ws, size_t ws_bytes, int32_t* dev_status, hipStream_t stream)
{
    if (N < 1 || H < 1 || W < 1 || K < 1 || bits < 2 || bits > 8) return ISEG_ERR_ARG;
    if (!y || !y_exp || !labels || !err || !err_exp) return ISEG_ERR_ARG;
    if (K > 256 || N * H * W * K > ((int64_t)1 << 40)) return ISEG_ERR_UNSUPPORTED;
    const int64_t n = N * H * W * K;
    if (!ws || ws_bytes < iseg_mse_onehot_ws(n)) return ISEG_ERR_WORKSPACE;
    MseArgs a{};
    a.y = y; a.y_exp = y_exp; a.labels = labels; a.n = n; a.K = (int32_t)K; a.status = dev_status;
    a.pmax = (uint64_t*)((char*)ws + 256);
    a.psum = (double*)((char*)ws + 256 + align256(2048 * 8));
    const unsigned grid = grid_for(n, 256 * 8, 2048);
    hipLaunchKernelGGL(k_mse_part, dim3(grid), dim3(256), 0, stream, a);
    int rc = launch_ok();
    if (rc) return rc;
    hipLaunchKernelGGL(k_mse_codes, dim3(grid_for(n, 256 * 4, 4096)), dim3(256), 0, stream, a, (int)grid,
                       (int)bits, err, err_exp, loss);
    return launch_ok();
}
