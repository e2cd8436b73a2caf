// bn.hip -- L1 batch normalization (Eq. 12-15) and its backward on gfx950.
//
// Because the input of BN is an int8 code tensor, every per-element quantity
// of the forward (xhat_q, y, the ReLU mask, sgn(x - mu_q), the output code A)
// is a function of (channel, input code) only, and the backward's dx code is
// a function of (channel, sgn class, masked error code).  The work therefore
// splits into
//   * streaming passes over [M, C]: coalesced dword loads (four channels per
//     lane), four rows in flight per lane, per-channel sums reduced in LDS and
//     written as one partial per block and channel (no global atomics, so no
//     same-address serialization across blocks);
//   * finalize steps that reduce the partials and do the exact rational
//     arithmetic once per channel or per table entry, in kernels of their own
//     (rounding E2: in the tails of the streaming passes, in the last block of
//     each channel slice to finish; an arrival counter picks it, no block
//     waits).
// sgn(x - mu_q) and the ReLU mask are monotone in the input code, so the
// streaming passes get them from two thresholds per channel instead of a
// table.
//
// Forward:  stats1 (block partials of sum q, min q, max q) -> stats2 (each
//           block first forms n_mu and the occupied code range of its slice
//           from them; the sums that give sum |x - mu_q|) -> fin2 (n_sigma,
//           den, b; xhat codes, y, thresholds, max|y|, y staged at each
//           channel's own Q_A shift) -> apply (Q_A's shift from the channels'
//           maxima; A codes; table gather).
// Backward: exact E2 (k_E2 >= 15): stats (block partials of sum delta, sum
//           delta*xhat, sum sgn and the per-class extremes of delta) ->
//           per-channel kernel (dgamma, dbeta, the channel's bound on E1's
//           exponent, its dx values staged at that bound) -> apply (E1's
//           exponent from the channels' bounds; staged values rounded into
//           the gather table).  k_E2 < 15 adds a second streaming pass: stats
//           tails give each slice's max|gamma delta| (E2's scale is the
//           largest), stats2 sums the rounded E2 terms and its tails give the
//           slices' bounds on E1's exponent; a table kernel, then apply.
#include <mutex>
#include <type_traits>

#include "iseg_common.h"

namespace {

constexpr int kSentinelLo = -(1 << 30);
typedef short short2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));

// launch geometry of the streaming passes (compile-time tuning knobs)
#ifndef ISEG_BN_NT
#define ISEG_BN_NT 1024          // threads per streaming block
#endif
#ifndef ISEG_BN_BLOCKS
#define ISEG_BN_BLOCKS 256       // streaming blocks per call, all channel slices
#endif
#ifndef ISEG_BNB_ROWS
#define ISEG_BNB_ROWS 2          // row groups per lane that size the backward statistics grid
#endif
constexpr int kMaxBlocks = ISEG_BN_BLOCKS;

// ---------------------------------------------------------------------------
// saved-state layout (documented in iseg.h)
// ---------------------------------------------------------------------------
struct Saved {
    int32_t* hdr;
    int32_t *n_mu, *n_sigma, *den, *qmin, *qmax;
    int32_t *t0, *p0, *mlo, *mhi;   // sgn/mask thresholds
    int16_t* xcode;                  // [C][256]
    uint8_t* flags;                  // [C][256]
    int8_t* acode;                   // [C][256]
    uint32_t* btab;                  // [C][256] by q & 0xff: y > 0, sgn, |sgn|, xhat code
    int16_t* ystg;                   // [C][256] ReLU(y) >> t_c (the output pass's staged A values)
};

size_t saved_bytes(int64_t C)
{
    return 256 + 9 * align256((size_t)C * 4) + align256((size_t)C * 512) +
           2 * align256((size_t)C * 256) + align256((size_t)C * 1024) + align256((size_t)C * 512);
}

Saved saved_map(void* base, int64_t C)
{
    char* p = (char*)base;
    Saved s;
    size_t v = align256((size_t)C * 4);
    s.hdr = (int32_t*)p; p += 256;
    s.n_mu = (int32_t*)p; p += v;
    s.n_sigma = (int32_t*)p; p += v;
    s.den = (int32_t*)p; p += v;
    s.qmin = (int32_t*)p; p += v;
    s.qmax = (int32_t*)p; p += v;
    s.t0 = (int32_t*)p; p += v;
    s.p0 = (int32_t*)p; p += v;
    s.mlo = (int32_t*)p; p += v;
    s.mhi = (int32_t*)p; p += v;
    s.xcode = (int16_t*)p; p += align256((size_t)C * 512);
    s.flags = (uint8_t*)p; p += align256((size_t)C * 256);
    s.acode = (int8_t*)p; p += align256((size_t)C * 256);
    s.btab = (uint32_t*)p; p += align256((size_t)C * 1024);
    s.ystg = (int16_t*)p;
    return s;
}

// ---------------------------------------------------------------------------
// streaming geometry: a block covers one channel slice of CS channels (CS % 4
// == 0, CS divides C); lane g of a row handles channels 4g..4g+3 of the slice;
// rpi rows are in flight per block step.
// ---------------------------------------------------------------------------
struct Stream {
    int64_t M;
    int32_t C, CS, G, rpi, gx;
};

int pick_cs(int64_t C, int csmax)
{
    for (int cs = csmax; cs >= 4; cs -= 4)
        if (C % cs == 0) return cs;
    return 0;
}

constexpr int kNT = ISEG_BN_NT;
constexpr int kWaves = kNT / 64;       // waves per streaming block

Stream make_stream(int64_t M, int64_t C, int cs, int cpl, int unroll, int max_blocks)
{
    Stream s;
    s.M = M; s.C = (int32_t)C; s.CS = cs; s.G = cs / cpl; s.rpi = kNT / s.G;
    int nsl = (int)(C / cs);
    int64_t want = max_blocks / nsl;
    if (want < 1) want = 1;
    int64_t rows = ceil_div64(M, (int64_t)s.rpi * unroll);
    s.gx = (int32_t)(rows < want ? rows : want);
    if (s.gx < 1) s.gx = 1;
    return s;
}

dim3 stream_grid(const Stream& s) { return dim3((unsigned)s.gx, (unsigned)(s.C / s.CS)); }

__device__ __forceinline__ bool stream_lane(const Stream& st, int& g, int& rsub)
{
    g = threadIdx.x % st.G;
    rsub = threadIdx.x / st.G;
    return rsub < st.rpi;
}

// Iterate the rows of this lane with U rows in flight; a lane covers CPL
// channels (4: one dword, 16: one 16-byte vector).  f(row, words[CPL/4]).
template <int CPL>
struct Vec { uint32_t w[CPL / 4]; };

template <int CPL>
__device__ __forceinline__ Vec<CPL> vload(const int8_t* p)
{
    Vec<CPL> v;
    if (CPL == 16) {
        uint4 t = *(const uint4*)p;
        v.w[0] = t.x; v.w[CPL / 4 > 1 ? 1 : 0] = t.y;
        if (CPL == 16) { v.w[2 % (CPL / 4)] = t.z; v.w[3 % (CPL / 4)] = t.w; }
    } else {
        v.w[0] = *(const uint32_t*)p;
    }
    return v;
}

template <int CPL>
__device__ __forceinline__ void vstore(int8_t* p, const Vec<CPL>& v)
{
    if (CPL == 16) *(uint4*)p = make_uint4(v.w[0], v.w[1 % (CPL / 4)], v.w[2 % (CPL / 4)], v.w[3 % (CPL / 4)]);
    else *(uint32_t*)p = v.w[0];
}

template <int CPL, int U, typename F>
__device__ __forceinline__ void stream_rows(const Stream& st, const int8_t* __restrict__ a, int c0,
                                            int rsub, F f)
{
    const int64_t step = (int64_t)gridDim.x * st.rpi;
    for (int64_t r = (int64_t)blockIdx.x * st.rpi + rsub; r < st.M; r += step * U) {
        Vec<CPL> v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            int64_t rr = r + u * step;
            if (rr < st.M) v[u] = vload<CPL>(a + rr * st.C + c0);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            int64_t rr = r + u * step;
            if (rr < st.M) f(rr, v[u]);
        }
    }
}

// two-input variant
template <int CPL, int U, typename F>
__device__ __forceinline__ void stream_rows2(const Stream& st, const int8_t* __restrict__ a,
                                             const int8_t* __restrict__ b, int c0, int rsub, F f)
{
    const int64_t step = (int64_t)gridDim.x * st.rpi;
    for (int64_t r = (int64_t)blockIdx.x * st.rpi + rsub; r < st.M; r += step * U) {
        Vec<CPL> va[U], vb[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            int64_t rr = r + u * step;
            if (rr < st.M) {
                va[u] = vload<CPL>(a + rr * st.C + c0);
                vb[u] = vload<CPL>(b + rr * st.C + c0);
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            int64_t rr = r + u * step;
            if (rr < st.M) f(rr, va[u], vb[u]);
        }
    }
}

__device__ __forceinline__ int sbyte(uint32_t w, int i) { return (int)(int8_t)(w >> (8 * i)); }

__device__ __forceinline__ bool sx_ok(int32_t s_x) { return s_x >= -40 && s_x <= 16; }

// D = (x - mu_q) / 2^g for code q; g = min(s_x, e_mu)
__device__ __forceinline__ int64_t bn_D(int q, int32_t s_x, int32_t n_mu, int e_mu)
{
    int g = s_x < e_mu ? s_x : e_mu;
    return (int64_t)q * ((int64_t)1 << (s_x - g)) - (int64_t)n_mu * ((int64_t)1 << (e_mu - g));
}

struct BnCfg {
    int32_t k_mu, k_sigma, k_xhat, k_gamma, k_beta, k_A, k_E1, k_E2, eps_code, relu;
};

BnCfg to_cfg(const iseg_bn_cfg* c)
{
    BnCfg b;
    b.k_mu = c->k_mu; b.k_sigma = c->k_sigma; b.k_xhat = c->k_xhat; b.k_gamma = c->k_gamma;
    b.k_beta = c->k_beta; b.k_A = c->k_A; b.k_E1 = c->k_E1; b.k_E2 = c->k_E2;
    b.eps_code = c->eps_code; b.relu = c->relu;
    return b;
}

// block-wide reduction of one value per thread (256 threads): xor-shuffles
// within each wave, then the four wave results through LDS (two barriers)
template <typename T, typename Op>
__device__ __forceinline__ T block_reduce(T v, Op op, T* sh)
{
    for (int o = 32; o > 0; o >>= 1) v = op(v, (T)__shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    T r = sh[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); k++) r = op(r, sh[k]);
    __syncthreads();
    return r;
}

struct OpAdd { template <typename T> __device__ T operator()(T a, T b) const { return a + b; } };
struct OpMin { template <typename T> __device__ T operator()(T a, T b) const { return a < b ? a : b; } };
struct OpMax { template <typename T> __device__ T operator()(T a, T b) const { return a > b ? a : b; } };

// v op v[lane ^ O]: for O = 16 or 32 with gfx950's cross-row swaps (VALU, no
// LDS traffic): v_permlane16_swap / v_permlane32_swap with both operands v
// leave v and its partner's value in the two results (which is which depends
// on the lane, so only commutative ops are folded); other O: an xor-shuffle.
template <int O>
__device__ __forceinline__ uint32_t lane_x32(uint32_t v, uint32_t* partner)
{
    if constexpr (O == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        *partner = r[1];
        return r[0];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        *partner = r[1];
        return r[0];
    }
}

template <int O, typename T, typename Op>
__device__ __forceinline__ T xor_fold(T v, Op op)
{
    if constexpr (O != 16 && O != 32) {
        return op(v, (T)__shfl_xor(v, O, 64));
    } else if constexpr (sizeof(T) == 8) {
        const uint64_t u = (uint64_t)v;
        uint32_t lp, hp;
        const uint32_t la = lane_x32<O>((uint32_t)u, &lp);
        const uint32_t ha = lane_x32<O>((uint32_t)(u >> 32), &hp);
        return op((T)((uint64_t)la | ((uint64_t)ha << 32)), (T)((uint64_t)lp | ((uint64_t)hp << 32)));
    } else {
        uint32_t p;
        const uint32_t a = lane_x32<O>((uint32_t)v, &p);
        return op((T)a, (T)p);
    }
}

// Lanes of a wave that hold the same channels are G apart (G a power of two
// dividing 64): fold them so that every lane holds the total over the wave's
// lanes of its channels (straight-line code for a compile-time G; G = 0 or 64:
// nothing to fold).  Every lane of the wave must be active.
template <int G, typename T, typename Op>
__device__ __forceinline__ T fold_g(T v, Op op)
{
    if constexpr (G >= 1 && G < 64) return fold_g<2 * G>(xor_fold<G>(v, op), op);
    else return v;
}

// f(std::integral_constant<int, G>) for a slice whose row has G lanes: G
// itself when it is a power of two up to 64 (compile-time folds), else 0.
template <typename F>
__device__ __forceinline__ void with_g(int G, F f)
{
    switch (G) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 8: f(std::integral_constant<int, 8>()); break;
    case 16: f(std::integral_constant<int, 16>()); break;
    case 32: f(std::integral_constant<int, 32>()); break;
    case 64: f(std::integral_constant<int, 64>()); break;
    default: f(std::integral_constant<int, 0>()); break;
    }
}

__device__ __forceinline__ bool group_leader(int G)
{
    return ((G & (G - 1)) != 0 || G > 64) || (int)(threadIdx.x & 63) < G;
}

// Copy n 16-byte pieces (n <= V * kNT) from global memory into LDS, every load
// of a thread issued before its first store.
template <int V>
__device__ __forceinline__ void copy_to_lds(uint4* dst, const uint4* __restrict__ src, int n)
{
    uint4 v[V];
#pragma unroll
    for (int k = 0; k < V; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < n) v[k] = src[i];
    }
#pragma unroll
    for (int k = 0; k < V; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < n) dst[i] = v[k];
    }
}

// LDS tables are kept one dword longer per row than in global memory: a
// table row is 256 entries (a multiple of the bank count), so without the skew
// every channel's entry for the same input code would sit in the same bank,
// and real activations concentrate on a few codes.
constexpr int kRowB = 256 + 4;      // bytes per row of a byte table in LDS
constexpr int kRowW = 256 + 1;      // dwords per row of a dword table in LDS

// Copy `rows` rows of 256 bytes (global, contiguous) into LDS rows of kRowB
// bytes; every load of a thread is issued before its first store.
template <int V>
__device__ __forceinline__ void copy_rows_to_lds(int8_t* dst, const int8_t* __restrict__ src, int rows)
{
    const int n = rows * 16;
    uint4 v[V];
#pragma unroll
    for (int k = 0; k < V; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < n) v[k] = ((const uint4*)src)[i];
    }
#pragma unroll
    for (int k = 0; k < V; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < n) {
            uint32_t* d = (uint32_t*)(dst + (i >> 4) * kRowB + (i & 15) * 16);
            d[0] = v[k].x; d[1] = v[k].y; d[2] = v[k].z; d[3] = v[k].w;
        }
    }
}

// ---------------------------------------------------------------------------
// arrival counters.  The backward workspace starts with ctr_bytes(C) bytes of
// uint32 counters: ctr[0] counts the channel slices whose partials are final,
// ctr[1 + y] the blocks of slice y that have published theirs.  atomicInc
// with limit n - 1 hands n - 1 to the n-th arrival and wraps the counter to
// zero there, so each kernel leaves the counters as it found them (zero); no
// block ever waits for another.
// ---------------------------------------------------------------------------
size_t ctr_bytes(int64_t C) { return ISEG_BN_WS_ZERO(C); }   // >= 4 (1 + C / 4)

// Values that cross blocks inside one kernel (partials, per-channel results
// a later tail reads) are stored and loaded as relaxed agent-scope atomics:
// write-through stores and loads that are coherent across the XCDs' L2
// caches.  Device-scope fences would give the same ordering by writing back
// and invalidating each whole L2, far too costly once per block.
template <typename T>
__device__ __forceinline__ void st_x(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T ld_x(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Called by every thread of a block after its st_x stores: true in all
// threads of the block that arrives last of n.  Each thread waits for its
// stores to complete (vmcnt 0) before the barrier, and the counter update
// follows the barrier, so every earlier arrival's stores precede the last
// block's ld_x loads.
__device__ __forceinline__ bool arrive_last(uint32_t* ctr, unsigned n)
{
    __shared__ int s_last;
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicInc(ctr, n - 1) == n - 1;
    __syncthreads();
    return s_last != 0;
}

// max over the kNT threads of a block (every thread gets it)
template <typename T>
__device__ __forceinline__ T block_max_nt(T v, T* sh)
{
    for (int o = 32; o > 0; o >>= 1) { const T u = __shfl_xor(v, o, 64); v = u > v ? u : v; }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    T m = sh[0];
    for (int k = 1; k < kNT / 64; k++) m = sh[k] > m ? sh[k] : m;
    __syncthreads();
    return m;
}

// ---------------------------------------------------------------------------
// forward statistics geometry: a block covers one slice of CS = CPL * G
// channels (the last slice of a C that CS does not divide leaves lanes idle)
// and walks row tiles of 4 * kNT / G rows, four rows of CPL channels per lane
// in flight.  Slices are 64 channels wide (16 or 32 for narrower tensors):
// each block of the second pass reads the first one's partials of its whole
// slice, gx * CS of them, and gx shrinks with the number of slices, so that
// read is a quarter of what 128-channel slices need (C = 256: 32 KB instead
// of 131 KB per block).
// ---------------------------------------------------------------------------
struct FStat {
    int64_t M;
    int32_t C, nsl, gx, ntiles;
    int32_t pad;                     // row slots past M in the tiles
};

template <int CPL, int G>
FStat make_fstat(int64_t M, int64_t C)
{
    constexpr int CS = CPL * G, TR = 4 * kNT / G;
    FStat f;
    f.M = M; f.C = (int32_t)C;
    f.nsl = (int32_t)ceil_div64(C, CS);
    f.ntiles = (int32_t)ceil_div64(M, TR);
    f.pad = (int32_t)((int64_t)f.ntiles * TR - M);
    int64_t gx = kMaxBlocks / f.nsl;
    if (gx > f.ntiles) gx = f.ntiles;
    if (gx < 1) gx = 1;
    f.gx = (int32_t)gx;
    return f;
}

// lanes per row of the 16-channel-lane variant
int fstat_g16(int64_t C) { return C <= 16 ? 1 : (C <= 32 ? 2 : 4); }

// ---------------------------------------------------------------------------
// forward workspace.  It starts, like the backward's, with ctr_bytes(C)
// bytes of arrival counters, which the forward leaves alone.
// ---------------------------------------------------------------------------
struct FwdWs {
    int32_t* b_glob;                 // exponent of Q_xhat's scale (fin2, block 0)
    int2* part;                      // [slice][gx][CS] sum q; (min q + 128) | (max q + 128) << 16
    unsigned long long* acc;         // [C] sum |q - T| (low half) and sum |q - T - 1| (high half)
    int32_t* sumq;                   // [C] sum q
    unsigned long long* maxYc;       // [C] max |ReLU(y)| of channel c over its occupied codes (fin2)
};

// partial entries of either variant: at most max(kMaxBlocks, slices) blocks of
// CS <= 64 channels
size_t fwd_part_entries(int64_t C)
{
    const int64_t n64 = ceil_div64(C, 64);
    return (size_t)(n64 > kMaxBlocks ? n64 : kMaxBlocks) * 64;
}

size_t fwd_ws_bytes(int64_t C)
{
    const size_t c = (size_t)C;
    return ctr_bytes(C) + 256 + align256(fwd_part_entries(C) * 8) + align256(c * 8) + align256(c * 4) +
           align256(c * 8);
}

FwdWs fwd_ws_map(void* base, int64_t C)
{
    char* p = (char*)base;
    const size_t c = (size_t)C;
    FwdWs w;
    p += ctr_bytes(C);
    w.b_glob = (int32_t*)p; p += 256;
    w.part = (int2*)p; p += align256(fwd_part_entries(C) * 8);
    w.acc = (unsigned long long*)p; p += align256(c * 8);
    w.sumq = (int32_t*)p; p += align256(c * 4);
    w.maxYc = (unsigned long long*)p;
    return w;
}

// ---------------------------------------------------------------------------
// forward kernels
//
// stats1 | block partials of sum q, min q, max q
// stats2 | prologue: n_mu and the occupied code range of the slice's channels
//          from stats1's partials | the channel sums of |q - T| and |q - T - 1|
//          added to the channel's accumulator
// fin2   (four channels per block, one thread per code): every block forms
//          all channels' sigma, denominator and bound on b (Q_xhat's scale);
//          xhat codes, y, sgn / ReLU thresholds, the backward's entries, the
//          channel's max|ReLU(y)| and ReLU(y) staged at the channel's own Q_A
//          shift
// apply  Q_A's shift r from the channels' maxima; the saved A codes; the
//          gather table from the staged values; table gather
//
// No pass ends in a tail: a kernel boundary costs less than the arrival,
// the reload and the serial arithmetic of a last block.
// ---------------------------------------------------------------------------
constexpr uint32_t kSign4 = 0x80808080u;

// lanes l and l ^ 32 (l ^ 16) exchange: bit clear lanes get op(a, a of the
// partner), bit set lanes op(b of the partner, b)
template <int O, typename T, typename Op>
__device__ __forceinline__ T swap_fold(T a, T b, Op op)
{
    if constexpr (O == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                        __builtin_bit_cast(uint32_t, b), false, false);
        const uint32_t u = r[0], v = r[1];
        return op(__builtin_bit_cast(T, u), __builtin_bit_cast(T, v));
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                        __builtin_bit_cast(uint32_t, b), false, false);
        const uint32_t u = r[0], v = r[1];
        return op(__builtin_bit_cast(T, u), __builtin_bit_cast(T, v));
    }
}

// v folded over the lanes of a 16-lane row that are multiples of G apart
// (rotations by DPP: every lane gets the total)
template <int G, typename T, typename Op>
__device__ __forceinline__ T row_fold(T v, Op op)
{
    auto ror = [&](auto n) {
        constexpr int N = decltype(n)::value;
        const int u = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, false);
        v = op(v, __builtin_bit_cast(T, u));
    };
    if constexpr (G <= 8) ror(std::integral_constant<int, 8>());
    if constexpr (G <= 4) ror(std::integral_constant<int, 4>());
    if constexpr (G <= 2) ror(std::integral_constant<int, 2>());
    if constexpr (G <= 1) ror(std::integral_constant<int, 1>());
    return v;
}

// Fold N = CPL values (channel i of the lane) over the wave's rows.  CPL = 16
// (G <= 4): the lane ends with channels fold_ch(l) + 0..3 in v[0..3]; CPL = 4
// (G = 16): with channel fold_ch(l) in v[0].  Two reduce-scatter steps halve
// the channels a lane holds, so 16 channels cost 12 swaps instead of 32.
template <int CPL, int G, typename T, typename Op>
__device__ __forceinline__ void wave_fold(T (&v)[CPL], Op op)
{
#pragma unroll
    for (int i = 0; i < CPL / 2; i++) v[i] = swap_fold<32>(v[i], v[i + CPL / 2], op);
#pragma unroll
    for (int i = 0; i < CPL / 4; i++) v[i] = swap_fold<16>(v[i], v[i + CPL / 4], op);
    if constexpr (CPL == 16) {
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = row_fold<G>(v[i], op);
    }
}

// first channel (of the lane's CPL) that a lane holds after wave_fold
template <int CPL>
__device__ __forceinline__ int fold_ch(int lane)
{
    return ((lane >> 5) & 1) * (CPL / 2) + ((lane >> 4) & 1) * (CPL / 4);
}

// four dwords of four channels (rows a, b, c, d) -> four dwords of four rows
__device__ __forceinline__ void transpose4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&o)[4])
{
    const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u);    // a0 b0 a1 b1
    const uint32_t ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);    // a2 b2 a3 b3
    const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u);
    const uint32_t cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
}

// Walk the block's row tiles: f(rows[4], valid[4]) with the lane's four rows of
// CPL channels; rows past M repeat the last one and are not valid.  The next
// tile's loads are issued before f runs on the current one.
template <int CPL, int G, typename F>
__device__ __forceinline__ void fstat_rows(const FStat& st, const int8_t* __restrict__ x, int c0, F f)
{
    constexpr int RPI = kNT / G;
    const int64_t rsub = threadIdx.x / G, last = st.M - 1;
    const int8_t* base = x + c0;
    Vec<CPL> cur[4], nxt[4];
    auto load = [&](int tile, Vec<CPL>* v) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int64_t r = (int64_t)tile * (4 * RPI) + u * RPI + rsub;
            v[u] = vload<CPL>(base + (r < last ? r : last) * st.C);
        }
    };
    int tile = blockIdx.x;
    if (tile < st.ntiles) load(tile, cur);
    while (tile < st.ntiles) {
        const int tn = tile + st.gx;
        if (tn < st.ntiles) load(tn, nxt);
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; u++) ok[u] = (int64_t)tile * (4 * RPI) + u * RPI + rsub <= last;
        f(cur, ok);
#pragma unroll
        for (int u = 0; u < 4; u++) cur[u] = nxt[u];
        tile = tn;
    }
}

// Bound by memory on the large tensors and by latency on the small ones; a
// lane's 16-byte loads keep 64 KB per CU in flight (131072 x 256 codes: 10.2 ->
// 8.5 us).  Sums by v_dot4 against a
// selector byte, minima and maxima as packed 16-bit operations on the bytes in
// the high halves (the low byte below them cannot change which high byte wins).
template <int CPL, int G>
__global__ __launch_bounds__(1024) void k_bnf_stats1(const int8_t* __restrict__ x, FStat st, FwdWs w)
{
    constexpr int CS = CPL * G, DW = CPL / 4;
    __shared__ int32_t sS[kWaves * CS];
    __shared__ int32_t sMm[kWaves * CS];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = t % G;
    const int c0 = blockIdx.y * CS + g * CPL;
    int s[CPL];
    short2v mnh[DW], mnl[DW], mxh[DW], mxl[DW];
#pragma unroll
    for (int i = 0; i < CPL; i++) s[i] = 0;
#pragma unroll
    for (int j = 0; j < DW; j++) { mnh[j] = mnl[j] = (short)0x7fff; mxh[j] = mxl[j] = (short)-0x8000; }
    fstat_rows<CPL, G>(st, x, c0 < st.C ? c0 : 0, [&](const Vec<CPL>* v, const bool* ok) {
#pragma unroll
        for (int u = 0; u < 4; u++)
#pragma unroll
            for (int j = 0; j < DW; j++) {
                const uint32_t q = v[u].w[j], qs = ok[u] ? q : 0u;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    s[4 * j + i] = __builtin_amdgcn_sdot4((int)qs, 1 << (8 * i), s[4 * j + i], false);
                const short2v h = __builtin_bit_cast(short2v, q), l = __builtin_bit_cast(short2v, q << 8);
                mnh[j] = __builtin_elementwise_min(mnh[j], h);
                mxh[j] = __builtin_elementwise_max(mxh[j], h);
                mnl[j] = __builtin_elementwise_min(mnl[j], l);
                mxl[j] = __builtin_elementwise_max(mxl[j], l);
            }
    });
    // (min + 128) | (max + 128) << 16 by channel; the halves' high bytes
    int mn[CPL], mx[CPL];
#pragma unroll
    for (int j = 0; j < DW; j++) {
        mn[4 * j] = mnl[j].x >> 8; mn[4 * j + 1] = mnh[j].x >> 8;
        mn[4 * j + 2] = mnl[j].y >> 8; mn[4 * j + 3] = mnh[j].y >> 8;
        mx[4 * j] = mxl[j].x >> 8; mx[4 * j + 1] = mxh[j].x >> 8;
        mx[4 * j + 2] = mxl[j].y >> 8; mx[4 * j + 3] = mxh[j].y >> 8;
    }
    wave_fold<CPL, G>(s, OpAdd());
    wave_fold<CPL, G>(mn, OpMin());
    wave_fold<CPL, G>(mx, OpMax());
    if ((lane & 15) < G) {
        constexpr int NV = CPL == 16 ? 4 : 1;
        const int cl = g * CPL + fold_ch<CPL>(lane);
#pragma unroll
        for (int i = 0; i < NV; i++) {
            sS[wv * CS + cl + i] = s[i];
            sMm[wv * CS + cl + i] = (mn[i] + 128) | ((mx[i] + 128) << 16);
        }
    }
    __syncthreads();
    const int c = blockIdx.y * CS + t;
    if (t < CS) {
        int bs = 0, lo = 255, hi = 0;
#pragma unroll
        for (int v = 0; v < kWaves; v++) {
            const int m = sMm[v * CS + t];
            bs += sS[v * CS + t];
            lo = min(lo, m & 0xffff);
            hi = max(hi, m >> 16);
        }
        // one contiguous row of partials per block, reduced by every block of
        // the next pass for its slice; the next pass's accumulators start at zero
        w.part[((int64_t)blockIdx.y * st.gx + blockIdx.x) * CS + t] = make_int2(bs, lo | (hi << 16));
        if (blockIdx.x == 0 && c < st.C) w.acc[c] = 0;
    }
}

// y on the grid 2^e_y of a channel's code q (before ReLU), and x-hat's code
struct FwdExps {
    int e_mu, e_sig, gg, e_g, e_b, e_xh, e_y, kx;
};

__device__ __forceinline__ FwdExps fwd_exps(int32_t s_x, int b, const BnCfg& cf)
{
    FwdExps e;
    e.e_mu = 2 - cf.k_mu; e.e_sig = 2 - cf.k_sigma;
    e.gg = s_x < e.e_mu ? s_x : e.e_mu;
    e.e_g = 2 - cf.k_gamma; e.e_b = 2 - cf.k_beta;
    e.kx = cf.k_xhat;
    e.e_xh = b - (cf.k_xhat - 1);
    e.e_y = (e.e_g + e.e_xh) < e.e_b ? (e.e_g + e.e_xh) : e.e_b;
    return e;
}

__device__ __forceinline__ i128 fwd_xcode(int64_t D, int32_t den, int b, const FwdExps& e)
{
    return clamp_k128(rhu128((i128)D, e.gg - e.e_sig + (e.kx - 1) - b, (i128)den), e.kx);
}

__device__ __forceinline__ i128 fwd_y(i128 nx, int gq, int bq, const FwdExps& e)
{
    return (i128)gq * nx * pow2_128(e.e_g + e.e_xh - e.e_y) + (i128)bq * pow2_128(e.e_b - e.e_y);
}

// The channel's offset off = n_mu 2^(e_mu - g) on the grid of its centred values
// D = q 2^(s_x - g) - off (g = min(s_x, e_mu)) and T = floor(off / 2^(s_x - g)),
// the largest code whose D is not positive.
__device__ __forceinline__ int64_t bn_off(int32_t s_x, int32_t n_mu, int e_mu)
{
    const int g = s_x < e_mu ? s_x : e_mu;
    return (int64_t)n_mu * ((int64_t)1 << (e_mu - g));
}
__device__ __forceinline__ int bn_T(int64_t off, int32_t s_x, int e_mu)
{
    const int g = s_x < e_mu ? s_x : e_mu;
    const int64_t t = off >> (s_x - g);
    return (int)(t < -129 ? -129 : (t > 127 ? 127 : t));
}
// reference byte (code + 128) of the first sum of absolute differences
__device__ __forceinline__ int bn_ref(int T) { return min(max(T + 128, 0), 254); }

// |D| is linear in q on either side of T .. T + 1, so sum |D| follows exactly
// from the two sums of absolute differences A0 = sum |q - T| and A1 = sum
// |q - T - 1| (see bnf_sigma).  Both come from v_sad_u8 on dwords of four rows
// of one channel (a 4x4 byte transpose per 16 elements): one VALU operation
// per element where a compare, select and two adds per element took five
// (the pass on 131072 x 256 codes: 23.8 -> 8.5 us, 3.9 TB/s; on 1024 x 16: 12.8 ->
// 4.5 us, with the slice tail gone; what is left there is the launch and the
// two round trips of the prologue and the rows).
template <int CPL, int G>
__global__ __launch_bounds__(1024) void k_bnf_stats2(const int8_t* __restrict__ x, const int32_t* x_exp,
                                                    FStat st, FwdWs w, Saved sv, BnCfg cf, int32_t* dev_status)
{
    constexpr int CS = CPL * G, DW = CPL / 4, NG = kNT / CS;
    __shared__ int32_t sS[kNT], sMm[kNT];          // prologue sums; then the wave totals of A0 and A1
    __shared__ int32_t sRef[CS];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = t % G;
    const int32_t s_in = *x_exp;
    const int32_t s_x = sx_ok(s_in) ? s_in : -14;     // keeps shifts defined; outputs are unspecified
    const int e_mu = 2 - cf.k_mu;
    {
        // n_mu (Eq. 12) and the occupied code range of the slice's channels from
        // stats1's partial rows: every block of the slice forms them, its first
        // block stores them.  All loads of a thread go out together; a row past
        // the last repeats the thread's first one, whose extremes change nothing.
        const int ch = t % CS, grp = t / CS;
        const int2* ps = w.part + (int64_t)blockIdx.y * st.gx * CS;
        int sum = 0, lo = 255, hi = 0;
        for (int b0 = grp; b0 < st.gx; b0 += 4 * NG) {
            int2 v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int b = b0 + u * NG;
                v[u] = ps[(int64_t)(b < st.gx ? b : b0) * CS + ch];
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (b0 + u * NG < st.gx) sum += v[u].x;      // |sum q| <= 2^29
                lo = min(lo, v[u].y & 0xffff);
                hi = max(hi, v[u].y >> 16);
            }
        }
        sS[t] = sum;
        sMm[t] = lo | (hi << 16);
        __syncthreads();
        if (t < CS) {
            const int ng = st.gx < NG ? st.gx : NG;
            for (int g2 = 1; g2 < ng; g2++) {
                const int m = sMm[g2 * CS + t];
                sum += sS[g2 * CS + t];
                lo = min(lo, m & 0xffff);
                hi = max(hi, m >> 16);
            }
            // mu/2 = S1 2^(s_x - 1) / M, code floor(mu/2 2^(k_mu-1) + 1/2); the mean
            // code is at most 128, so shifts below -24 give 0 like -24 does
            const int32_t nm = (int32_t)clamp_k(rhu64(sum, max(s_x - 1 + (cf.k_mu - 1), -24), st.M), cf.k_mu);
            sRef[t] = bn_ref(bn_T(bn_off(s_x, nm, e_mu), s_x, e_mu));
            const int c = blockIdx.y * CS + t;
            if (blockIdx.x == 0 && c < st.C) {
                sv.n_mu[c] = nm;
                sv.qmin[c] = lo - 128;
                sv.qmax[c] = hi - 128;
                w.sumq[c] = sum;
            }
        }
        __syncthreads();
    }
    const int c0 = blockIdx.y * CS + g * CPL;
    uint32_t a0[CPL], a1[CPL], r0[CPL];
#pragma unroll
    for (int i = 0; i < CPL; i++) {
        a0[i] = a1[i] = 0;
        r0[i] = (uint32_t)sRef[g * CPL + i] * 0x01010101u;
    }
    fstat_rows<CPL, G>(st, x, c0 < st.C ? c0 : 0, [&](const Vec<CPL>* v, const bool* ok) {
#pragma unroll
        for (int j = 0; j < DW; j++) {
            uint32_t u[4], o[4];
            // rows past M count as byte 0; their known share is taken out in bnf_sigma
#pragma unroll
            for (int k = 0; k < 4; k++) u[k] = ok[k] ? v[k].w[j] ^ kSign4 : 0u;
            transpose4(u[0], u[1], u[2], u[3], o);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                a0[4 * j + i] = __builtin_amdgcn_sad_u8(o[i], r0[4 * j + i], a0[4 * j + i]);
                a1[4 * j + i] = __builtin_amdgcn_sad_u8(o[i], r0[4 * j + i] + 0x01010101u, a1[4 * j + i]);
            }
        }
    });
    wave_fold<CPL, G>(a0, OpAdd());
    wave_fold<CPL, G>(a1, OpAdd());
    if ((lane & 15) < G) {
        constexpr int NV = CPL == 16 ? 4 : 1;
        const int cl = g * CPL + fold_ch<CPL>(lane);
#pragma unroll
        for (int i = 0; i < NV; i++) {
            sS[wv * CS + cl + i] = (int32_t)a0[i];
            sMm[wv * CS + cl + i] = (int32_t)a1[i];
        }
    }
    __syncthreads();
    const int c = blockIdx.y * CS + t;
    if (!sx_ok(s_in) && blockIdx.x == 0 && blockIdx.y == 0 && t == 0) set_status(dev_status, ISEG_DEV_RANGE);
    if (t < CS && c < st.C) {
        uint32_t b0 = 0, b1 = 0;
#pragma unroll
        for (int v = 0; v < kWaves; v++) {
            b0 += (uint32_t)sS[v * CS + t];
            b1 += (uint32_t)sMm[v * CS + t];
        }
        // each total stays below 255 (2^22 + 4096) < 2^31, so the halves of the
        // 64-bit addition never carry into each other
        atomicAdd(&w.acc[c], (unsigned long long)b0 | ((unsigned long long)b1 << 32));
    }
}

// n_sigma (Eq. 13-14) from the channel's sums.  With diff = A1 - A0 = M - 2
// N(q > T): sum |D| = 2^(s_x - g) (A0 - T diff) + off diff for T in [-128, 126];
// beyond, every D has one sign.  Magnitudes: either s_x <= e_mu and the power
// is 1 with |off| <= 255, or |off| < 2^15 and the power is at most 2^30: below 2^61.
__device__ __forceinline__ int32_t bnf_sigma(unsigned long long acc, int32_t sumq, const FStat& st, int32_t s_x,
                                             int32_t n_mu, int e_mu, const BnCfg& cf)
{
    const int g = s_x < e_mu ? s_x : e_mu;
    const int64_t off = bn_off(s_x, n_mu, e_mu), mul = (int64_t)1 << (s_x - g);
    const int T = bn_T(off, s_x, e_mu);
    int64_t sabs;
    if (T > 126) sabs = off * st.M - mul * sumq;
    else if (T < -128) sabs = mul * sumq - off * st.M;
    else {
        const int64_t ref = bn_ref(T);
        const int64_t A0 = (int64_t)(uint32_t)acc - (int64_t)st.pad * ref;
        const int64_t A1 = (int64_t)(uint32_t)(acc >> 32) - (int64_t)st.pad * (ref + 1);
        const int64_t diff = A1 - A0;
        sabs = mul * (A0 - T * diff) + off * diff;
    }
    // sigma/2 = sumabs 2^(g-1) / M ; n_sigma = floor(sigma/2 2^(k_sigma-1) + 1/2).
    // A shift below -24 needs g = s_x < e_mu, hence sumabs / M <= 512: 0 as with -24
    return (int32_t)clamp_k(rhu64(sabs, max(g - 1 + (cf.k_sigma - 1), -24), st.M), cf.k_sigma);
}

// max of n per-slice values, by every thread of the block (kSentinelLo if n = 0)
__device__ __forceinline__ int32_t slices_max(const int32_t* a, int n, int32_t* sh)
{
    int32_t m = kSentinelLo;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = max(m, a[i]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    m = sh[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); k++) m = max(m, sh[k]);
    return m;
}

// shift of a channel's staged A values: max(0, r_c - 1), r_c = bitlen(max) -
// (k_A - 1) the Q_A shift of the channel's own max |ReLU(y)|
__device__ __forceinline__ int ystg_shift(uint64_t maxy, int kA)
{
    const int rc = maxy ? bitlen_u64(maxy) - (kA - 1) : 0;
    return rc > 1 ? rc - 1 : 0;
}

// x-hat code of D and its y: 64-bit arithmetic where the operands fit (always
// for the occupied codes of ordinary layers), 128-bit otherwise
__device__ __forceinline__ int32_t fwd_xcode_any(int64_t D, int32_t den, int b, const FwdExps& e)
{
    const int sh = e.gg - e.e_sig + (e.kx - 1) - b;
    const uint64_t aD = (uint64_t)(D < 0 ? -D : D);
    const int lb = bitlen_u64(aD) + (sh > 0 ? sh : 0), ld = bitlen_u64((uint64_t)den) + (sh < 0 ? -sh : 0);
    if (lb <= 60 && ld <= 60 && lb - ld < 46) return (int32_t)clamp_k(rhu64(D, sh, den), e.kx);
    return (int32_t)fwd_xcode(D, den, b, e);
}

// Per (channel, code): xhat code, y, flags and the backward's entry; per
// channel: the sgn and ReLU thresholds and max |ReLU(y)| over the occupied
// codes (y is monotone in q, so over qmin and qmax).  Every block forms all
// channels' denominators and bounds on b itself (a few values per thread; C
// is at most a few thousand): the arrival, reload and arithmetic of a tail in
// the statistics pass took longer.  Bound by latency: the loads, two exact
// divisions and three barriers.
constexpr int kFinCh = kNT / 256;              // channels per block
__global__ __launch_bounds__(1024) void k_bnf_fin2(const int32_t* x_exp, FStat st, FwdWs w, Saved sv, BnCfg cf,
                                                  const int8_t* gamma_q, const int8_t* beta_q)
{
    __shared__ int32_t rsh[kWaves], sNs[kFinCh], sDen[kFinCh];
    __shared__ uint64_t sBal[kWaves][3], sAy[kFinCh][2];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lc = t >> 8;
    const int c = blockIdx.x * kFinCh + lc;
    const int q = (t & 255) - 128;
    const bool own = c < st.C;
    // every load of the first round goes out before the first wait (no branch on
    // a loaded value in between)
    const int32_t s_in = *x_exp;
    const int cs = own ? c : 0, k0 = t < st.C ? t : 0;
    const int32_t nmu = sv.n_mu[cs], qlo = sv.qmin[cs], qhi = sv.qmax[cs];
    const int gq = gamma_q[cs], bq = beta_q[cs];
    int32_t nm = sv.n_mu[k0], lo = sv.qmin[k0], hi = sv.qmax[k0], sumq = w.sumq[k0];
    unsigned long long acc = w.acc[k0];
    const int e_mu = 2 - cf.k_mu, e_sig = 2 - cf.k_sigma;
    const int32_t s_x = sx_ok(s_in) ? s_in : -14;     // outputs unspecified, shifts defined
    int best = kSentinelLo;
    for (int k = t; k < st.C; k += kNT) {
        if (k != t) { nm = sv.n_mu[k]; lo = sv.qmin[k]; hi = sv.qmax[k]; sumq = w.sumq[k]; acc = w.acc[k]; }
        const int32_t ns = bnf_sigma(acc, sumq, st, s_x, nm, e_mu, cf);
        const int32_t den = max(ns + cf.eps_code, 1);
        if (k / kFinCh == (int)blockIdx.x) { sNs[k % kFinCh] = ns; sDen[k % kFinCh] = den; }
        // xhat is linear in q: its largest magnitude is at qmin or qmax
        const int64_t D0 = bn_D(lo, s_x, nm, e_mu), D1 = bn_D(hi, s_x, nm, e_mu);
        const uint64_t m0 = (uint64_t)(D0 < 0 ? -D0 : D0), m1 = (uint64_t)(D1 < 0 ? -D1 : D1);
        const uint64_t m = m0 > m1 ? m0 : m1;
        if (m) best = max(best, ceil_pow2_exp64(m, (uint64_t)den) + min(s_x, e_mu) - e_sig);
    }
    for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
    if (lane == 0) rsh[wv] = best;
    __syncthreads();
    int b = rsh[0];
#pragma unroll
    for (int k = 1; k < kWaves; k++) b = max(b, rsh[k]);
    if (b == kSentinelLo) b = 0;
    const int32_t den = sDen[lc];
    if (blockIdx.x == 0 && t == 0) *w.b_glob = b;
    const FwdExps e = fwd_exps(s_x, b, cf);
    const int64_t D = bn_D(q, s_x, nmu, e.e_mu);
    const int32_t nx = own ? fwd_xcode_any(D, den, b, e) : 0;
    // y on its grid: one of the two shifts is zero; |y| < 2^62 for gaps up to 48
    const int gx = e.e_g + e.e_xh - e.e_y, gb = e.e_b - e.e_y;
    const bool wide = gx > 38 || gb > 48;          // uniform over the grid
    int64_t Yr = 0;
    bool pos;
    i128 Yw = 0;
    if (wide) {
        Yw = fwd_y(nx, gq, bq, e);
        pos = Yw > 0;
        if (cf.relu && Yw < 0) Yw = 0;
    } else {
        Yr = (int64_t)(gq * nx) * ((int64_t)1 << gx) + (int64_t)bq * ((int64_t)1 << gb);
        pos = Yr > 0;
        if (cf.relu && Yr < 0) Yr = 0;
    }
    const int idx = c * 256 + (t & 255);
    const int sg = (D > 0) - (D < 0);
    if (own) {
        sv.xcode[idx] = (int16_t)nx;
        sv.flags[idx] = (uint8_t)((pos ? 1 : 0) | ((sg + 1) << 1));
        sv.btab[c * 256 + (q & 255)] = ((uint32_t)(uint16_t)(int16_t)nx << 16) | ((uint32_t)(sg & 3) << 8) |
                                       ((uint32_t)(sg != 0) << 10) | (pos ? 1u : 0u);
    }
    // thresholds (least code with D >= 0, least with D > 0, code range with y >
    // 0) from the waves' ballots
    const uint64_t m0 = __ballot(D >= 0), m1 = __ballot(D > 0), m2 = __ballot(pos);
    if (lane == 0) { sBal[wv][0] = m0; sBal[wv][1] = m1; sBal[wv][2] = m2; }
    const uint64_t ay = wide ? (uint64_t)abs128(Yw) : (uint64_t)(Yr < 0 ? -Yr : Yr);
    if (q == qlo) sAy[lc][0] = ay;
    if (q == qhi) sAy[lc][1] = ay;
    __syncthreads();
    const uint64_t mx = sAy[lc][0] > sAy[lc][1] ? sAy[lc][0] : sAy[lc][1];
    if (own && (t & 255) == 0) {
        int v[4] = {128, 128, 128, -129};
#pragma unroll
        for (int k = 3; k >= 0; k--)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const uint64_t bm = sBal[wv + k][j];
                if (bm) v[j] = -128 + 64 * k + __builtin_ctzll(bm);
            }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint64_t bm = sBal[wv + k][2];
            if (bm) v[3] = -128 + 64 * k + 63 - __builtin_clzll(bm);
        }
        sv.t0[c] = v[0]; sv.p0[c] = v[1]; sv.mlo[c] = v[2]; sv.mhi[c] = v[3];
        sv.n_sigma[c] = sNs[lc];
        sv.den[c] = den;
        w.maxYc[c] = mx;
    }
    // ReLU(y) floored by 2^t_c, t_c = max(0, r_c - 1) with r_c the Q_A shift
    // this channel's own maximum would give: below 2^k_A in magnitude for the
    // occupied codes (clamped elsewhere, where the output pass never looks)
    const int tc = ystg_shift(mx, cf.k_A);
    int64_t z;
    if (wide) {
        const i128 zw = tc ? (Yw >> tc) : Yw;
        z = zw > 32767 ? 32767 : (zw < -32767 ? -32767 : (int64_t)zw);
    } else {
        z = Yr >> tc;
        z = z > 32767 ? 32767 : (z < -32767 ? -32767 : z);
    }
    if (own) sv.ystg[idx] = (int16_t)z;
}

// Output pass.  Every block first takes Q_A's shift r from the channels'
// maxima (block (0, 0) writes the output exponent and the saved header), then
//   * writes its share of the saved A codes, exactly from the xhat codes (the
//     table the inference path applies, every code included);
//   * builds its channels' gather table from the staged values:
//     code = ((z >> (r - 1 - t_c)) + 1) >> 1, the half-up rounding of
//     ReLU(y) by 2^r (half-up rounding of floor(v / 2^t) by 2^(r - t) equals
//     that of v for t < r), two codes per packed 16-bit operation.
// The loads of the maxima, the staged table, the share of xhat codes and the
// first row tile all go out together, so the prologue costs one round trip
// (131072 x 256 codes: 15.8 -> 14.0 us, 4.8 TB/s; 1024 x 16: 6.5 -> 4.5 us).
// U rows per lane and tile: 4, or 1 where four would leave most CUs idle.
template <int CPL, int G, int U>
FStat make_fapply(int64_t M, int64_t C)
{
    FStat f = make_fstat<CPL, G>(M, C);
    f.ntiles = (int32_t)ceil_div64(M, (int64_t)U * kNT / G);
    int64_t gx = kMaxBlocks / f.nsl;
    if (gx > f.ntiles) gx = f.ntiles;
    f.gx = (int32_t)(gx < 1 ? 1 : gx);
    return f;
}

template <int CPL, int G, int U>
__global__ __launch_bounds__(1024) void k_bnf_apply(const int8_t* __restrict__ x, int8_t* __restrict__ y,
                                                   FStat st, Saved sv, FwdWs w, BnCfg cf, const int32_t* x_exp,
                                                   const int8_t* gamma_q, const int8_t* beta_q, int32_t* y_exp)
{
    constexpr int CS = CPL * G, RPI = kNT / G, TV = (CS * 32 + kNT - 1) / kNT;
    __shared__ __attribute__((aligned(16))) int8_t lut[CS * kRowB];
    __shared__ uint64_t rmax[kWaves];
    const int t = threadIdx.x, g = t % G, rsub = t / G;
    const int c0 = blockIdx.y * CS + g * CPL, cb = blockIdx.y * CS;
    const int64_t last = st.M - 1;
    const int8_t* xb = x + (c0 < st.C ? c0 : 0);
    Vec<CPL> cur[U], nxt[U];
    auto load = [&](int tile, Vec<CPL>* v) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t r = (int64_t)tile * (U * RPI) + u * RPI + rsub;
            v[u] = vload<CPL>(xb + (r < last ? r : last) * st.C);
        }
    };
    uint64_t M = w.maxYc[t < st.C ? t : 0];
    const int32_t s_in = *x_exp;
    const int b = *w.b_glob;
    int4 zq[TV];
    uint64_t my[TV];
#pragma unroll
    for (int k = 0; k < TV; k++) {
        const int v = t + k * kNT, row = v >> 5;
        const int c = row < CS && cb + row < st.C ? cb + row : cb;
        zq[k] = *(const int4*)(sv.ystg + (int64_t)c * 256 + (v & 31) * 8);
        my[k] = w.maxYc[c];
    }
    // share of the saved A codes, four codes of one channel per step
    const int64_t nall = (int64_t)st.C * 64, nb = (int64_t)gridDim.x * gridDim.y;
    const int64_t per = (nall + nb - 1) / nb;
    const int64_t i0 = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * per;
    const int64_t i1 = i0 + per < nall ? i0 + per : nall;
    int64_t ia = i0 + t;
    const int64_t il = ia < i1 ? ia : 0;
    short4v xq = *(const short4v*)(sv.xcode + il * 4);
    int gq = gamma_q[il >> 6], bq = beta_q[il >> 6];
    int tile = blockIdx.x;
    if (tile < st.ntiles) load(tile, cur);
    for (int k = t + kNT; k < st.C; k += kNT) M = w.maxYc[k] > M ? w.maxYc[k] : M;
    M = wave_max_u64(M);
    if ((t & 63) == 0) rmax[t >> 6] = M;
    __syncthreads();
    M = rmax[0];
#pragma unroll
    for (int k = 1; k < kWaves; k++) M = rmax[k] > M ? rmax[k] : M;
    const int r = M ? bitlen_u64(M) - (cf.k_A - 1) : 0;
    const bool ok = sx_ok(s_in);
    const int32_t s_x = ok ? s_in : -14;          // outputs unspecified; keeps the shifts defined
    const FwdExps e = fwd_exps(s_x, b, cf);
    if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0 && ok) {
        *y_exp = e.e_y + r;
        sv.hdr[0] = b;
        sv.hdr[1] = e.e_y;
        sv.hdr[2] = e.e_y + r;
        sv.hdr[3] = s_x;
    }
    const short lim = (short)((1 << (cf.k_A - 1)) - 1);
    const short up = (short)(r < 0 ? -r : 0);
#pragma unroll
    for (int k = 0; k < TV; k++) {
        const int v = t + k * kNT, row = v >> 5, col = (v & 31) * 8;
        if (row >= CS) break;
        const int tc = ystg_shift(my[k], cf.k_A);
        const int qw[4] = {zq[k].x, zq[k].y, zq[k].z, zq[k].w};
        uint32_t ow[2] = {0, 0};
        const short sh = (short)(r > 0 ? min(max(r - 1 - tc, 0), 15) : 0);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            short2v zv = __builtin_bit_cast(short2v, qw[h]);
            if (r > 0) zv = ((zv >> sh) + (short)1) >> (short)1;
            else zv = zv << up;
            zv = zv > lim ? lim : zv;
            zv = zv < (short)-lim ? (short)-lim : zv;
            const uint32_t bb = ((uint32_t)(uint16_t)zv.x & 0xffu) | (((uint32_t)(uint16_t)zv.y & 0xffu) << 8);
            ow[h >> 1] |= bb << (16 * (h & 1));
        }
        *(uint32_t*)(lut + row * kRowB + col) = ok ? ow[0] : 0u;
        *(uint32_t*)(lut + row * kRowB + col + 4) = ok ? ow[1] : 0u;
    }
    if (ok) {
        const int gx = e.e_g + e.e_xh - e.e_y, gb = e.e_b - e.e_y;
        const bool wide = gx > 38 || gb > 48;      // uniform over the grid
        for (; ia < i1; ia += kNT) {
            if (ia != i0 + t) {
                xq = *(const short4v*)(sv.xcode + ia * 4);
                gq = gamma_q[ia >> 6];
                bq = beta_q[ia >> 6];
            }
            uint32_t o = 0;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                int64_t Yv = wide ? (int64_t)fwd_y((i128)xq[k], gq, bq, e)
                                  : (int64_t)(gq * xq[k]) * ((int64_t)1 << gx) + (int64_t)bq * ((int64_t)1 << gb);
                if (cf.relu && Yv < 0) Yv = 0;
                o |= (uint32_t)(uint8_t)sq_code(Yv, r, cf.k_A) << (8 * k);
            }
            *(uint32_t*)(sv.acode + ia * 4) = o;
        }
    }
    __syncthreads();
    const int8_t* l = lut + g * CPL * kRowB + 128;
    while (tile < st.ntiles) {
        const int tn = tile + st.gx;
        if (tn < st.ntiles) load(tn, nxt);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t rr = (int64_t)tile * (U * RPI) + u * RPI + rsub;
            Vec<CPL> o;
#pragma unroll
            for (int j = 0; j < CPL / 4; j++) {
                uint32_t ow = 0;
#pragma unroll
                for (int i = 0; i < 4; i++)
                    ow |= (uint32_t)(uint8_t)l[(j * 4 + i) * kRowB + sbyte(cur[u].w[j], i)] << (8 * i);
                o.w[j] = ow;
            }
            if (rr <= last && c0 < st.C) vstore<CPL>(y + rr * st.C + c0, o);
        }
#pragma unroll
        for (int u = 0; u < U; u++) cur[u] = nxt[u];
        tile = tn;
    }
}

// ---------------------------------------------------------------------------
// backward workspace
// ---------------------------------------------------------------------------
struct BwdWs {
    uint32_t* ctr;                   // arrival counters
    int32_t* smax;                   // [slices] bound on E1's exponent over each slice's channels
    int32_t* smaxF;                  // [slices] max |gamma delta| over each slice's channels (rounding E2)
    int32_t *p_sd, *p_z, *p_mmA, *p_mmB;   // [gx][C] partials (per-class extremes packed as bytes)
    long long *p_sdn, *p_sf, *p_sfn; // [gx][C]
    long long *sd, *sdn, *sf, *sfn;  // [C] reduced
    int32_t *Z, *mm;                 // [C], [C][6]
    int8_t* lut;                     // [C][3][256] dx codes (rounding E2)
    int32_t* cbnd;                   // [C] each channel's bound on E1's exponent (exact E2)
    int16_t* lutq;                   // [C][3][256] dx values at the channel's own bound (exact E2)
};

size_t bwd_ws_bytes(const Stream& st)
{
    size_t pc = (size_t)st.gx * st.C, C = (size_t)st.C;
    return ctr_bytes(st.C) + 2 * align256(C) + 4 * align256(pc * 4) + 3 * align256(pc * 8) +
           4 * align256(C * 8) + align256(C * 4) + align256(C * 24) + align256(C * 768) + align256(C * 4) +
           align256(C * 768 * 2);
}

BwdWs bwd_ws_map(void* base, const Stream& st)
{
    char* p = (char*)base;
    size_t pc = (size_t)st.gx * st.C, C = (size_t)st.C;
    BwdWs w;
    w.ctr = (uint32_t*)p; p += ctr_bytes(st.C);
    w.smax = (int32_t*)p; p += align256(C);          // slices <= C / 4
    w.smaxF = (int32_t*)p; p += align256(C);
    w.p_sd = (int32_t*)p; p += align256(pc * 4);
    w.p_z = (int32_t*)p; p += align256(pc * 4);
    w.p_mmA = (int32_t*)p; p += align256(pc * 4);
    w.p_mmB = (int32_t*)p; p += align256(pc * 4);
    w.p_sdn = (long long*)p; p += align256(pc * 8);
    w.p_sf = (long long*)p; p += align256(pc * 8);
    w.p_sfn = (long long*)p; p += align256(pc * 8);
    w.sd = (long long*)p; p += align256(C * 8);
    w.sdn = (long long*)p; p += align256(C * 8);
    w.sf = (long long*)p; p += align256(C * 8);
    w.sfn = (long long*)p; p += align256(C * 8);
    w.Z = (int32_t*)p; p += align256(C * 4);
    w.mm = (int32_t*)p; p += align256(C * 24);
    w.lut = (int8_t*)p; p += align256(C * 768);
    w.cbnd = (int32_t*)p; p += align256(C * 4);
    w.lutq = (int16_t*)p;
    return w;
}

// sgn class (sgn + 1) and ReLU mask of an input code from the thresholds
struct Thr {
    int t0, p0, mlo, mhi;
};

__device__ __forceinline__ int thr_cls(const Thr& t, int q) { return 1 + (q >= t.p0) - (q < t.t0); }
__device__ __forceinline__ bool thr_mask(const Thr& t, int q) { return q >= t.mlo && q <= t.mhi; }

// Copy the channel slice's per-(channel, code) entries (saved by the forward)
// into LDS rows of kRowW dwords, all loads of a thread issued before the first
// store.  The ReLU bit becomes a mask byte in bits 0..7 (0xff passes delta).
// With `lut_off` the upper half is replaced by the offset of the entry's
// sgn-class row in the slice's dx-code tables (three rows of kRowB bytes per
// channel, +128 for the signed delta).
constexpr int kTabV = 64 * 256 / 4 / kNT;    // 16-byte pieces per thread (CS <= 64)
__device__ __forceinline__ void load_bwd_tab(uint32_t* tab, const uint32_t* src, int CS, int relu,
                                             bool lut_off)
{
    const int nv = CS * 64;
    uint4 v[kTabV];
#pragma unroll
    for (int k = 0; k < kTabV; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < nv) v[k] = ((const uint4*)src)[i];
    }
#pragma unroll
    for (int k = 0; k < kTabV; k++) {
        const int i = threadIdx.x + k * kNT;
        if (i < nv) {
            uint32_t e[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint32_t m = (!relu || (e[j] & 1)) ? 0xffu : 0u;
                if (lut_off) {
                    const int cl = (4 * i + j) >> 8;
                    const int sg = ((int)(e[j] << 22)) >> 30;
                    e[j] = ((uint32_t)((cl * 3 + sg + 1) * kRowB + 128) << 16) | m;
                } else {
                    e[j] = (e[j] & 0xffffff00u) | m;
                }
            }
            uint32_t* d = tab + (i >> 6) * kRowW + (i & 63) * 4;
            d[0] = e[0]; d[1] = e[1]; d[2] = e[2]; d[3] = e[3];
        }
    }
}

// Per-class extremes of the masked delta travel between blocks as bytes:
// low ends as lo + 128 (255 for an empty class), high ends as hi + 128 (0 for
// an empty class), so a byte-wise min / max merges them and an empty class
// still reads lo > hi.  A = (lo, hi) of classes -1 and 0, B = (lo, hi) of +1.
__device__ __forceinline__ uint32_t pk_lo(int v) { return v > 127 ? 255u : (uint32_t)(v + 128); }
__device__ __forceinline__ uint32_t pk_hi(int v) { return v < -128 ? 0u : (uint32_t)(v + 128); }
__device__ __forceinline__ void mm_pack(const int* mm, uint32_t& A, uint32_t& B)
{
    A = pk_lo(mm[0]) | pk_hi(mm[1]) << 8 | pk_lo(mm[2]) << 16 | pk_hi(mm[3]) << 24;
    B = pk_lo(mm[4]) | pk_hi(mm[5]) << 8;
}
__device__ __forceinline__ void mm_merge(uint32_t A, uint32_t B, int* lo3, int* hi3)
{
    lo3[0] = min(lo3[0], (int)(A & 0xff)); hi3[0] = max(hi3[0], (int)((A >> 8) & 0xff));
    lo3[1] = min(lo3[1], (int)((A >> 16) & 0xff)); hi3[1] = max(hi3[1], (int)(A >> 24));
    lo3[2] = min(lo3[2], (int)(B & 0xff)); hi3[2] = max(hi3[2], (int)((B >> 8) & 0xff));
}

// Pass 1: sum delta, sum delta*xhat, sum sgn and the per-sgn-class extremes of
// the masked delta d.  The extremes come from four keys per element, d +- 1024 s
// and d +- 1024 |s| (s = sgn in {-1, 0, 1}, |d| <= 128): the minimum of d + 1024 s
// lies in class -1 whenever that class is present, its maximum in class +1, and
// likewise for the others, so six min/max updates replace per-class selects.
constexpr int kKey = 1024;
constexpr int kKeyInit = 4 * kKey;
struct BnbOut {
    const int32_t* dy_exp;
    const int8_t* gamma_q;
    int64_t *dgamma, *dbeta;
    int32_t *dgamma_exp, *dbeta_exp, *dx_exp, *dev_status;
};

__device__ __forceinline__ void bnb_round_tail1(uint32_t* lds, const Stream& st, const BwdWs& w, const Saved& sv,
                                                const BnCfg& cf, const BnbOut& o);

// Block totals per channel.  When the G lanes of a row (G = CS / 4) are a
// power of two, the lanes of a wave that hold the same channels are folded
// with shuffles and the 16 wave totals of each channel are staged in LDS
// (the caller's table space, no longer read) and summed by one thread per
// channel: LDS atomics from every wave onto the same channel slots serialize
// and cost several microseconds per block.  Other widths use LDS atomics.

template <int TAIL>                      // 1: exact E2, 2: rounding E2
__global__ __launch_bounds__(1024) void k_bnb_stats(const int8_t* __restrict__ dy,
                                                   const int8_t* __restrict__ x, Stream st, BwdWs w,
                                                   Saved sv, BnCfg cf, BnbOut out)
{
    const int relu = cf.relu;
    __shared__ __attribute__((aligned(16))) uint32_t tab[64 * kRowW];
    __shared__ unsigned long long sSdn[64];
    __shared__ int32_t sSd[64], sZ[64], sMM[64 * 6];
    const int64_t cbase = (int64_t)blockIdx.y * st.CS;
    const bool fold = (st.G & (st.G - 1)) == 0 && st.G <= 64;
    load_bwd_tab(tab, sv.btab + cbase * 256, st.CS, relu, false);
    if (!fold && (int)threadIdx.x < st.CS) {
        sSdn[threadIdx.x] = 0; sSd[threadIdx.x] = 0; sZ[threadIdx.x] = 0;
        for (int k = 0; k < 3; k++) { sMM[threadIdx.x * 6 + 2 * k] = 1000; sMM[threadIdx.x * 6 + 2 * k + 1] = -1000; }
    }
    __syncthreads();
    int g, rsub;
    const bool active = stream_lane(st, g, rsub);
    int32_t sd[4] = {0, 0, 0, 0}, z[4] = {0, 0, 0, 0};
    int64_t sdn[4] = {0, 0, 0, 0};
    // key extremes: min(d + 1024 s), max(d + 1024 s), min(d - 1024 s), max(d - 1024 s),
    // min(d + 1024 |s|), max(d - 1024 |s|)
    int32_t kmn0[4], kmx0[4], kmn1[4], kmx1[4], kmn2[4], kmx3[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        kmn0[i] = kmn1[i] = kmn2[i] = kKeyInit;
        kmx0[i] = kmx1[i] = kmx3[i] = -kKeyInit;
    }
    if (active) {
        const int c0 = (int)cbase + g * 4;
        const uint32_t* tb = tab + g * 4 * kRowW;
        const int64_t step = (int64_t)gridDim.x * st.rpi;
        auto elem = [&](uint32_t wx, uint32_t wd, int32_t* sdn32) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t e = tb[i * kRowW + ((wx >> (8 * i)) & 0xff)];
                const int dm = sbyte(wd, i) & (int)(int8_t)(e & 0xff);
                const int sg = ((int)(e << 22)) >> 30;            // bits 8..9, signed
                const int ab = (int)((e >> 10) & 1);
                sd[i] += dm;
                sdn32[i] += dm * ((int)e >> 16);
                z[i] += sg;
                const int k0 = dm + sg * kKey, k1 = dm - sg * kKey;
                const int k2 = dm + ab * kKey, k3 = dm - ab * kKey;
                kmn0[i] = min(kmn0[i], k0); kmx0[i] = max(kmx0[i], k0);
                kmn1[i] = min(kmn1[i], k1); kmx1[i] = max(kmx1[i], k1);
                kmn2[i] = min(kmn2[i], k2); kmx3[i] = max(kmx3[i], k3);
            }
        };
        // full groups of U rows (all in range), next group's loads issued
        // before this group's arithmetic; then the remaining rows one by one
        constexpr int U = 4;
        int64_t r = (int64_t)blockIdx.x * st.rpi + rsub;
        const int64_t full_end = st.M - (U - 1) * step;
        uint32_t vx[U], vd[U], nx[U], nd[U];
        auto load = [&](int64_t r0, uint32_t* ax, uint32_t* ad) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                ax[u] = *(const uint32_t*)(x + (r0 + u * step) * st.C + c0);
                ad[u] = *(const uint32_t*)(dy + (r0 + u * step) * st.C + c0);
            }
        };
        if (r < full_end) load(r, vx, vd);
        while (r < full_end) {
            const int64_t rn = r + U * step;
            if (rn < full_end) load(rn, nx, nd);
            int32_t sdn32[4] = {0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < U; u++) elem(vx[u], vd[u], sdn32);
#pragma unroll
            for (int i = 0; i < 4; i++) sdn[i] += sdn32[i];
#pragma unroll
            for (int u = 0; u < U; u++) { vx[u] = nx[u]; vd[u] = nd[u]; }
            r = rn;
        }
        for (; r < st.M; r += step) {
            int32_t sdn32[4] = {0, 0, 0, 0};
            elem(*(const uint32_t*)(x + r * st.C + c0), *(const uint32_t*)(dy + r * st.C + c0), sdn32);
#pragma unroll
            for (int i = 0; i < 4; i++) sdn[i] += sdn32[i];
        }
    }
    // decode the keys into (min, max) per class; an empty class gives (1000, -1000)
    int32_t mm[4][6];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        mm[i][0] = kmn0[i] <= -kKey + 128 ? kmn0[i] + kKey : 1000;     // class -1
        mm[i][1] = kmx1[i] >= kKey - 128 ? kmx1[i] - kKey : -1000;
        mm[i][2] = kmn2[i] <= 128 ? kmn2[i] : 1000;                     // class 0
        mm[i][3] = kmx3[i] >= -128 ? kmx3[i] : -1000;
        mm[i][4] = kmn1[i] <= -kKey + 128 ? kmn1[i] + kKey : 1000;     // class +1
        mm[i][5] = kmx0[i] >= kKey - 128 ? kmx0[i] - kKey : -1000;
    }
    with_g(st.G, [&](auto gc) {
        constexpr int GG = decltype(gc)::value;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            sd[i] = fold_g<GG>(sd[i], OpAdd());
            sdn[i] = fold_g<GG>(sdn[i], OpAdd());
            z[i] = fold_g<GG>(z[i], OpAdd());
#pragma unroll
            for (int k = 0; k < 3; k++) {
                mm[i][2 * k] = fold_g<GG>(mm[i][2 * k], OpMin());
                mm[i][2 * k + 1] = fold_g<GG>(mm[i][2 * k + 1], OpMax());
            }
        }
    });
    const int t = threadIdx.x;
    int32_t bsd = 0, bz = 0;
    long long bsdn = 0;
    int bmm[6] = {1000, -1000, 1000, -1000, 1000, -1000};
    if (fold) {
        __syncthreads();                                  // every wave is done with the table
        int32_t* wsd = (int32_t*)tab;                     // [kWaves][64] each
        int32_t* wz = wsd + kWaves * 64;
        int32_t* wmm = wz + kWaves * 64;                  // [6][kWaves][64]
        long long* wsdn = (long long*)(wmm + 6 * kWaves * 64);
        const int wv = t >> 6;
        if ((t & 63) < st.G) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int s = wv * 64 + g * 4 + i;
                wsd[s] = sd[i]; wz[s] = z[i]; wsdn[s] = sdn[i];
#pragma unroll
                for (int k = 0; k < 6; k++) wmm[k * kWaves * 64 + s] = mm[i][k];
            }
        }
        __syncthreads();
        if (t < st.CS) {
#pragma unroll 4
            for (int v = 0; v < kWaves; v++) {
                const int s = v * 64 + t;
                bsd += wsd[s]; bz += wz[s]; bsdn += wsdn[s];
#pragma unroll
                for (int k = 0; k < 6; k++) {
                    const int m = wmm[k * kWaves * 64 + s];
                    bmm[k] = (k & 1) ? max(bmm[k], m) : min(bmm[k], m);
                }
            }
        }
    } else {
        if (active && group_leader(st.G)) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                int cl = g * 4 + i;
                atomicAdd(&sSd[cl], sd[i]);
                atomicAdd(&sSdn[cl], (unsigned long long)sdn[i]);
                atomicAdd(&sZ[cl], z[i]);
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    atomicMin(&sMM[cl * 6 + 2 * k], mm[i][2 * k]);
                    atomicMax(&sMM[cl * 6 + 2 * k + 1], mm[i][2 * k + 1]);
                }
            }
        }
        __syncthreads();
        if (t < st.CS) {
            bsd = sSd[t]; bz = sZ[t]; bsdn = (long long)sSdn[t];
            for (int k = 0; k < 6; k++) bmm[k] = sMM[t * 6 + k];
        }
    }
    if (t < st.CS) {
        uint32_t A, B;
        mm_pack(bmm, A, B);
        if constexpr (TAIL == 1) {
            // [slice][block][channel of the slice]: one contiguous row per block
            const int64_t o = ((int64_t)blockIdx.y * st.gx + blockIdx.x) * st.CS + t;
            w.p_sd[o] = bsd;
            w.p_sdn[o] = bsdn;
            w.p_z[o] = bz;
            w.p_mmA[o] = (int32_t)A;
            w.p_mmB[o] = (int32_t)B;
        } else {
            const int64_t o = (int64_t)blockIdx.x * st.C + cbase + t;
            st_x(&w.p_sd[o], bsd);
            st_x(&w.p_sdn[o], bsdn);
            st_x(&w.p_z[o], bz);
            st_x(&w.p_mmA[o], (int32_t)A);
            st_x(&w.p_mmB[o], (int32_t)B);
        }
    }
    if constexpr (TAIL == 2) {
        if (arrive_last(w.ctr + 1 + blockIdx.y, gridDim.x)) {
            __syncthreads();                              // the staging above may still be read
            bnb_round_tail1(tab, st, w, sv, cf, out);
        }
    }
}


// E2's requant shift from max |gamma delta| (the slices' maxima)
__device__ __forceinline__ int bnb_r2_of(int32_t maxF, const BnCfg& cf)
{
    return maxF > 0 ? bitlen_u64((uint64_t)maxF) - (cf.k_E2 - 1) : 0;
}

__device__ __forceinline__ void bnb_round_tail2(uint32_t* lds, const Stream& st, const BwdWs& w,
                                                const Saved& sv, const BnCfg& cf, const BnbOut& o, int r2);

// pass 2 (only when E2's quantizer rounds): sum f and f*n_xhat; the tails
// reduce them and give each slice's bound on E1's exponent
__global__ __launch_bounds__(1024) void k_bnb_stats2(const int8_t* __restrict__ dy,
                                                    const int8_t* __restrict__ x, Stream st, BwdWs w,
                                                    Saved sv, BnCfg cf, BnbOut out)
{
    const int8_t* gamma_q = out.gamma_q;
    __shared__ __attribute__((aligned(16))) int16_t xc[64 * 256];
    __shared__ int16_t ft[64 * 256];                  // f = SQ(gamma_q d, k_E2) per (channel, d)
    __shared__ Thr thr[64];
    __shared__ unsigned long long sF[64], sFn[64];
    __shared__ int32_t rsh[kNT / 64];
    const int64_t cbase = (int64_t)blockIdx.y * st.CS;
    {
        copy_to_lds<64 * 512 / 16 / kNT>((uint4*)xc, (const uint4*)(sv.xcode + cbase * 256), st.CS * 32);
    }
    if ((int)threadIdx.x < st.CS) {
        int c = (int)cbase + threadIdx.x;
        thr[threadIdx.x] = Thr{sv.t0[c], sv.p0[c], cf.relu ? sv.mlo[c] : -1000, cf.relu ? sv.mhi[c] : 1000};
        sF[threadIdx.x] = 0; sFn[threadIdx.x] = 0;
    }
    // |f| < 2^(k_E2-1) <= 2^13 on this path
    const int r2 = bnb_r2_of(slices_max(w.smaxF, (int)gridDim.y, rsh), cf);
    for (int e = threadIdx.x; e < st.CS * 256; e += blockDim.x)
        ft[e] = (int16_t)sq_code((int64_t)gamma_q[cbase + (e >> 8)] * ((e & 255) - 128), r2, cf.k_E2);
    __syncthreads();
    int g, rsub;
    const bool active = stream_lane(st, g, rsub);
    int64_t sf[4] = {0, 0, 0, 0}, sfn[4] = {0, 0, 0, 0};
    if (active) {
        const int c0 = (int)cbase + g * 4;
        Thr t[4];
#pragma unroll
        for (int i = 0; i < 4; i++) t[i] = thr[g * 4 + i];
        stream_rows2<4, 8>(st, x, dy, c0, rsub, [&](int64_t, const Vec<4>& vxx, const Vec<4>& vdd) {
            const uint32_t vx = vxx.w[0], vd = vdd.w[0];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                int q = sbyte(vx, i);
                int d = thr_mask(t[i], q) ? sbyte(vd, i) : 0;
                const int f = ft[(g * 4 + i) * 256 + d + 128];
                sf[i] += f;
                sfn[i] += f * (int)xc[(g * 4 + i) * 256 + q + 128];     // |f x| < 2^28
            }
        });
    }
    with_g(st.G, [&](auto gc) {
        constexpr int GG = decltype(gc)::value;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            sf[i] = fold_g<GG>(sf[i], OpAdd());
            sfn[i] = fold_g<GG>(sfn[i], OpAdd());
        }
    });
    if (active && group_leader(st.G)) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            atomicAdd(&sF[g * 4 + i], (unsigned long long)sf[i]);
            atomicAdd(&sFn[g * 4 + i], (unsigned long long)sfn[i]);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < st.CS) {
        int64_t o = (int64_t)blockIdx.x * st.C + cbase + threadIdx.x;
        st_x(&w.p_sf[o], (long long)sF[threadIdx.x]);
        st_x(&w.p_sfn[o], (long long)sFn[threadIdx.x]);
    }
    if (arrive_last(w.ctr + 1 + blockIdx.y, gridDim.x)) {
        __syncthreads();
        bnb_round_tail2((uint32_t*)xc, st, w, sv, cf, out, r2);
    }
}

// bracket of the exact dx (times den M^2 / 2^Ebase) for a (f, sgn) pair
__device__ __forceinline__ i128 bnb_bracket(int64_t f, int s, i128 M, i128 Sf, i128 T, i128 Z, int e_xh)
{
    i128 a = M * M * (i128)f - M * Sf;
    i128 t = T * (M * (i128)s - Z);
    return e_xh >= 0 ? a - (t << e_xh) : (a << -e_xh) - t;
}

struct BnbChan {
    i128 Sf, T, Z;
    int e_xh, Ebase, r2;
};

// exponents of a channel's bracket for E2's shift r2
__device__ __forceinline__ BnbChan bnb_chan_exps(int r2, int32_t dy_exp, const Saved& sv, const BnCfg& cf)
{
    BnbChan ch;
    ch.r2 = r2;
    ch.e_xh = sv.hdr[0] - (cf.k_xhat - 1);
    const int e_sig = 2 - cf.k_sigma, e_g = 2 - cf.k_gamma;
    const int s2 = dy_exp + e_g + r2;
    ch.Ebase = s2 - e_sig + (ch.e_xh < 0 ? ch.e_xh : 0);
    return ch;
}

__device__ __forceinline__ void bnb_exps_out(const Saved& sv, const BnCfg& cf, const BnbOut& o)
{
    const int32_t s_d = *o.dy_exp;
    if (s_d < -60 || s_d > 16) set_status(o.dev_status, ISEG_DEV_RANGE);
    *o.dbeta_exp = s_d;
    *o.dgamma_exp = s_d + sv.hdr[0] - (cf.k_xhat - 1);
}

// dx code table for every (sgn class, masked error code) of a channel
// (rounding E2): E1's exponent and E2's shift from the slices' maxima
__global__ __launch_bounds__(256) void k_bnb_lut(int64_t Mrows, int nslices, BwdWs w, Saved sv, BnCfg cf,
                                                 BnbOut o)
{
    __shared__ int32_t rsh[4];
    const int c = blockIdx.x;
    const int d = (int)threadIdx.x - 128;
    const int gq = o.gamma_q[c];
    const int r2 = bnb_r2_of(slices_max(w.smaxF, nslices, rsh), cf);
    int bdx = slices_max(w.smax, nslices, rsh);
    if (bdx == kSentinelLo) bdx = 0;
    if (c == 0 && threadIdx.x == 0) {
        *o.dx_exp = bdx - (cf.k_E1 - 1);
        bnb_exps_out(sv, cf, o);
    }
    BnbChan ch = bnb_chan_exps(r2, *o.dy_exp, sv, cf);
    ch.Sf = (i128)w.sf[c];
    ch.T = (i128)w.sfn[c];
    ch.Z = (i128)w.Z[c];
    const i128 M = Mrows;
    const i128 Dd = (i128)sv.den[c] * M * M;
    const int64_t f = d < -127 ? 0 : sq_code((int64_t)gq * d, ch.r2, cf.k_E2);
    for (int k = 0; k < 3; k++) {
        int8_t code = 0;
        if (d >= -127) {
            i128 B = bnb_bracket(f, k - 1, M, ch.Sf, ch.T, ch.Z, ch.e_xh);
            code = (int8_t)clamp_k128(rhu128(B, ch.Ebase + (cf.k_E1 - 1) - bdx, Dd), cf.k_E1);
        }
        w.lut[((int64_t)c * 3 + k) * 256 + threadIdx.x] = code;
    }
}

// ---------------------------------------------------------------------------
// Exact E2 (k_E2 >= 15, |gamma delta| <= 127^2 < 2^(k_E2-1)): E2's requant
// shift r2 is <= 0 and scales every term of the bracket and the exponent base
// by inverse powers of two, so dx, its exponent bound and its codes are those
// of r2 = 0, with f = gamma_q delta; the stats kernel's tails replace a
// separate per-channel pass.
// ---------------------------------------------------------------------------
// stats tail (exact E2).  Slice: the pass-1 sums, dgamma and dbeta of its
// channels and each channel's bound on max|dx| (|dx| is extreme at a class's
// extreme deltas: six candidates per channel, one thread each); the largest
// bound of the slice goes to smax for the table kernel, which takes E1's
// exponent as the largest over the slices.  `lds` is the stats table, no
// longer read once the block has arrived.
struct Tail1Lds {
    int32_t *sd, *z, *mm, *cand;        // [kNT], [kNT], [6][kNT], [6 * CS]
    long long* sdn;                     // [kNT]
    __device__ explicit Tail1Lds(uint32_t* lds)
    {
        sd = (int32_t*)lds; z = sd + kNT; mm = z + kNT;
        sdn = (long long*)(mm + 6 * kNT); cand = (int32_t*)(sdn + kNT);
    }
};

// the slice's pass-1 sums from all blocks' partials: w.sd / sdn / Z / mm,
// dgamma, dbeta, and the channel totals in the group-0 slots of the LDS table
__device__ __forceinline__ void bnb_tail_reduce1(uint32_t* lds, const Stream& st, const BwdWs& w,
                                                 const BnbOut& o)
{
    const int CS = st.CS, ng = kNT / CS, t = threadIdx.x, ch = t % CS, grp = t / CS;
    const Tail1Lds L(lds);
    int32_t* tSd = L.sd;
    int32_t* tZ = L.z;
    int32_t* tMM = L.mm;
    long long* tSdn = L.sdn;
    const int64_t cb = (int64_t)blockIdx.y * CS;
    int sd = 0, z = 0;
    long long sdn = 0;
    int lo3[3] = {255, 255, 255}, hi3[3] = {0, 0, 0};   // byte-coded extremes
    constexpr int U = 8;                    // partial rows whose loads are in flight together
    if (grp < ng)
        for (int b0 = grp; b0 < st.gx; b0 += U * ng) {
            int32_t vsd[U], vz[U], vA[U], vB[U];
            long long vsdn[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int b = b0 + u * ng;
                const int64_t q = (int64_t)(b < st.gx ? b : b0) * st.C + cb + ch;
                vsd[u] = ld_x(&w.p_sd[q]);
                vsdn[u] = ld_x(&w.p_sdn[q]);
                vz[u] = ld_x(&w.p_z[q]);
                vA[u] = ld_x(&w.p_mmA[q]);
                vB[u] = ld_x(&w.p_mmB[q]);
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                mm_merge((uint32_t)vA[u], (uint32_t)vB[u], lo3, hi3);   // a repeated row changes nothing
                if (b0 + u * ng >= st.gx) continue;
                sd += vsd[u]; sdn += vsdn[u]; z += vz[u];
            }
        }
    tSd[t] = sd; tZ[t] = z; tSdn[t] = sdn;
#pragma unroll
    for (int k = 0; k < 3; k++) { tMM[2 * k * kNT + t] = lo3[k]; tMM[(2 * k + 1) * kNT + t] = hi3[k]; }
    __syncthreads();
    if (t < CS) {
        for (int g2 = 1; g2 < ng; g2++) {
            const int i = g2 * CS + t;
            sd += tSd[i]; z += tZ[i]; sdn += tSdn[i];
#pragma unroll
            for (int k = 0; k < 3; k++) {
                lo3[k] = min(lo3[k], tMM[2 * k * kNT + i]);
                hi3[k] = max(hi3[k], tMM[(2 * k + 1) * kNT + i]);
            }
        }
        int mm[6];
#pragma unroll
        for (int k = 0; k < 3; k++) { mm[2 * k] = lo3[k] - 128; mm[2 * k + 1] = hi3[k] - 128; }   // empty: lo > hi
        const int64_t c = cb + t;
        w.sd[c] = sd; w.sdn[c] = sdn; w.Z[c] = z;
#pragma unroll
        for (int k = 0; k < 6; k++) w.mm[c * 6 + k] = mm[k];
        o.dbeta[c] = sd;
        o.dgamma[c] = sdn;
        // the channel totals, in the slots of group 0, for the candidate threads
        tSd[t] = sd; tZ[t] = z; tSdn[t] = sdn;
#pragma unroll
        for (int k = 0; k < 6; k++) tMM[k * kNT + t] = mm[k];
    }
    __syncthreads();
}

// largest of the slice's per-channel values in tCand (6 per channel) into
// *dst (kSentinelLo when none)
__device__ __forceinline__ void slice_cand_max(const int32_t* tCand, int n, int32_t* dst, int32_t* sh)
{
    int32_t m = kSentinelLo;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = max(m, tCand[i]);
    m = block_max_nt(m, sh);
    if (threadIdx.x == 0) *dst = m;
}

// stats tail (rounding E2).  Slice: the pass-1 sums, dgamma, dbeta and the
// largest |gamma_q delta| over its channels' sgn classes, into smaxF; the
// second pass takes E2's Scale from the largest over the slices.
__device__ __forceinline__ void bnb_round_tail1(uint32_t* lds, const Stream& st, const BwdWs& w, const Saved& sv,
                                                const BnCfg& cf, const BnbOut& o)
{
    bnb_tail_reduce1(lds, st, w, o);
    const int CS = st.CS, t = threadIdx.x;
    const Tail1Lds L(lds);
    __shared__ int32_t rb[kNT / 64];
    const int64_t cb = (int64_t)blockIdx.y * CS;
    int F = 0;
    if (t < CS) {
        int amax = 0;
        for (int k = 0; k < 3; k++) {
            const int lo = L.mm[2 * k * kNT + t], hi = L.mm[(2 * k + 1) * kNT + t];
            if (lo > hi) continue;                     // empty class
            amax = max(amax, max(lo < 0 ? -lo : lo, hi < 0 ? -hi : hi));
        }
        const int gq = o.gamma_q[cb + t];
        F = (gq < 0 ? -gq : gq) * amax;                // <= 128 * 128
    }
    F = block_max_nt(F, rb);
    if (t == 0) w.smaxF[blockIdx.y] = F;
}

// stats2 tail.  Slice: the pass-2 sums (sum f, sum f n_xhat) and each
// channel's bound on max|dx| (six candidates, as the exact tail); the largest
// goes to smax.  `lds` is stats2's x-hat table, no longer read.
__device__ __forceinline__ void bnb_round_tail2(uint32_t* lds, const Stream& st, const BwdWs& w,
                                                const Saved& sv, const BnCfg& cf, const BnbOut& o, int r2)
{
    const int CS = st.CS, ng = kNT / CS, t = threadIdx.x, ch = t % CS, grp = t / CS;
    long long* tSf = (long long*)lds;                   // [kNT]
    long long* tSfn = tSf + kNT;                        // [kNT]
    int32_t* tCand = (int32_t*)(tSfn + kNT);            // [6 * CS]
    __shared__ int32_t rb[kNT / 64];
    const int64_t cb = (int64_t)blockIdx.y * CS;
    long long sf = 0, sfn = 0;
    constexpr int U = 8;                    // partial rows whose loads are in flight together
    if (grp < ng)
        for (int b0 = grp; b0 < st.gx; b0 += U * ng) {
            long long vf[U], vn[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int b = b0 + u * ng;
                const int64_t q = (int64_t)(b < st.gx ? b : b0) * st.C + cb + ch;
                vf[u] = ld_x(&w.p_sf[q]);
                vn[u] = ld_x(&w.p_sfn[q]);
            }
#pragma unroll
            for (int u = 0; u < U; u++)
                if (b0 + u * ng < st.gx) { sf += vf[u]; sfn += vn[u]; }
        }
    tSf[t] = sf; tSfn[t] = sfn;
    __syncthreads();
    if (t < CS) {
        for (int g2 = 1; g2 < ng; g2++) { sf += tSf[g2 * CS + t]; sfn += tSfn[g2 * CS + t]; }
        w.sf[cb + t] = sf; w.sfn[cb + t] = sfn;
        tSf[t] = sf; tSfn[t] = sfn;                     // only thread t reads slot t above
    }
    __syncthreads();
    if (t < 6 * CS) {
        const int cl = t / 6, k = t % 6;                // channel of the slice; class k / 2, low / high
        const int64_t c = cb + cl;
        const int lo = w.mm[c * 6 + (k & ~1)], hi = w.mm[c * 6 + (k | 1)];
        int best = kSentinelLo;
        if (lo <= hi) {
            const int gq = o.gamma_q[c];
            const BnbChan e = bnb_chan_exps(r2, *o.dy_exp, sv, cf);
            const i128 M = st.M;
            const int64_t f = sq_code((int64_t)gq * ((k & 1) ? hi : lo), e.r2, cf.k_E2);
            const i128 B = bnb_bracket(f, (k >> 1) - 1, M, (i128)tSf[cl], (i128)tSfn[cl], (i128)w.Z[c], e.e_xh);
            if (B != 0) best = ceil_pow2_exp128(abs128(B), (i128)sv.den[c] * M * M) + e.Ebase;
        }
        tCand[t] = best;
    }
    __syncthreads();
    slice_cand_max(tCand, 6 * CS, w.smax + blockIdx.y, rb);
}

// Exact E2 (k_E2 >= 15), one block per channel and one thread per masked
// error code: the channel's totals from the streaming blocks' partials
// (dbeta, dgamma), its bound on E1's exponent (the largest over its six
// per-class extremes; xhat and the bracket are linear in the code, so the
// extremes bound every code the channel's data holds), and its dx values at
// that bound: Q = floor(B 2^S / D) with S one more than the shift of the
// channel's own bound, for the (class, code) pairs inside the channel's
// per-class ranges (zero elsewhere: the output pass never looks them up).
// |Q| <= 2^k_E1 + 1 there, so int16 holds it; the output pass rounds Q by
// the gap between the largest bound and the channel's into the final code
// (half-up rounding of floor(x) by 2^g + 1 equals that of x).
__global__ __launch_bounds__(256) void k_bnb_chan_exact(int64_t Mrows, int gx, int CS, BwdWs w, Saved sv,
                                                        BnCfg cf, BnbOut o)
{
    __shared__ int32_t r_sd[4], r_z[4], r_lo[4][3], r_hi[4][3], r_cand;
    __shared__ long long r_sdn[4];
    const int c = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int sd = 0, z = 0;
    long long sdn = 0;
    int lo3[3] = {255, 255, 255}, hi3[3] = {0, 0, 0};       // byte-coded extremes (empty: lo > hi)
    const int sy = c / CS, sc = c - sy * CS;                  // slice, channel within it
    for (int b = t; b < gx; b += blockDim.x) {
        const int64_t q = ((int64_t)sy * gx + b) * CS + sc;
        sd += w.p_sd[q];
        sdn += w.p_sdn[q];
        z += w.p_z[q];
        mm_merge((uint32_t)w.p_mmA[q], (uint32_t)w.p_mmB[q], lo3, hi3);
    }
    for (int off = 32; off > 0; off >>= 1) {
        sd += __shfl_xor(sd, off, 64);
        z += __shfl_xor(z, off, 64);
        sdn += __shfl_xor(sdn, off, 64);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            lo3[k] = min(lo3[k], __shfl_xor(lo3[k], off, 64));
            hi3[k] = max(hi3[k], __shfl_xor(hi3[k], off, 64));
        }
    }
    if (lane == 0) {
        r_sd[wv] = sd; r_z[wv] = z; r_sdn[wv] = sdn;
#pragma unroll
        for (int k = 0; k < 3; k++) { r_lo[wv][k] = lo3[k]; r_hi[wv][k] = hi3[k]; }
    }
    __syncthreads();
    sd = (r_sd[0] + r_sd[1]) + (r_sd[2] + r_sd[3]);
    z = (r_z[0] + r_z[1]) + (r_z[2] + r_z[3]);
    sdn = (r_sdn[0] + r_sdn[1]) + (r_sdn[2] + r_sdn[3]);
    int mm[6];
#pragma unroll
    for (int k = 0; k < 3; k++) {
        mm[2 * k] = min(min(r_lo[0][k], r_lo[1][k]), min(r_lo[2][k], r_lo[3][k])) - 128;
        mm[2 * k + 1] = max(max(r_hi[0][k], r_hi[1][k]), max(r_hi[2][k], r_hi[3][k])) - 128;
    }
    if (t == 0) {
        o.dbeta[c] = sd;
        o.dgamma[c] = sdn;
    }
    const int gq = o.gamma_q[c];
    const int e_xh = sv.hdr[0] - (cf.k_xhat - 1);
    const int e_sig = 2 - cf.k_sigma, e_g = 2 - cf.k_gamma;
    const int Ebase = *o.dy_exp + e_g - e_sig + (e_xh < 0 ? e_xh : 0);
    const i128 M = Mrows;
    const i128 Dd = (i128)sv.den[c] * M * M;
    const i128 Sf = (i128)gq * sd, T = (i128)gq * sdn, Z = z;
    // the six per-class candidates (threads 0..5 of wave 0), their max
    if (wv == 0) {
        int cand = kSentinelLo;
        if (t < 6) {
            const int lo = mm[t & ~1], hi = mm[t | 1];
            if (lo <= hi) {
                const int64_t f = clamp_k((int64_t)gq * ((t & 1) ? hi : lo), cf.k_E2);
                const i128 B = bnb_bracket(f, (t >> 1) - 1, M, Sf, T, Z, e_xh);
                if (B != 0) cand = ceil_pow2_exp128(abs128(B), Dd) + Ebase;
            }
        }
        for (int off = 4; off > 0; off >>= 1) cand = max(cand, __shfl_xor(cand, off, 64));
        if (t == 0) {
            r_cand = cand;
            w.cbnd[c] = cand;
        }
    }
    __syncthreads();
    const int bc = r_cand;
    const int d = t - 128;
    const int S = Ebase + (cf.k_E1 - 1) - bc + 1;
    for (int k = 0; k < 3; k++) {
        int16_t q = 0;
        if (bc != kSentinelLo && d >= mm[2 * k] && d <= mm[2 * k + 1] && d >= -127) {
            const int64_t f = clamp_k((int64_t)gq * d, cf.k_E2);
            const i128 B = bnb_bracket(f, k - 1, M, Sf, T, Z, e_xh);
            i128 Q = S >= 0 ? floordiv128(B << S, Dd) : floordiv128(B, Dd << -S);
            Q = Q > 32767 ? 32767 : (Q < -32767 ? -32767 : Q);
            q = (int16_t)Q;
        }
        w.lutq[((int64_t)c * 3 + k) * 256 + t] = q;
    }
}

// Output pass: dx code = lut[c][sgn class][masked delta].  A per-(channel,
// code) entry gives the offset of the channel's class row in the block's LDS
// copy of the tables (bits 16..31) and the ReLU mask byte (bits 0..7), so each
// element costs two LDS reads and a handful of ALU operations.
// Exact E2: every block first takes E1's exponent from the channels' bounds
// (block (0, 0) writes it and the parameter-gradient exponents) and rounds
// its channels' staged values into the codes.
__global__ __launch_bounds__(1024) void k_bnb_apply(const int8_t* __restrict__ dy,
                                                   const int8_t* __restrict__ x,
                                                   int8_t* __restrict__ dx, Stream st, BwdWs w,
                                                   Saved sv, BnCfg cf, BnbOut o, int32_t exact)
{
    __shared__ __attribute__((aligned(16))) int8_t lut[64 * 3 * kRowB];
    __shared__ __attribute__((aligned(16))) uint32_t tab[64 * kRowW];
    __shared__ int32_t rb[kNT / 64];
    const int relu = cf.relu;
    const int64_t cbase = (int64_t)blockIdx.y * st.CS;
    if (exact) {
        int bdx = kSentinelLo;
        for (int i = threadIdx.x; i < st.C; i += kNT) bdx = max(bdx, w.cbnd[i]);
        bdx = block_max_nt(bdx, rb);
        if (bdx == kSentinelLo) bdx = 0;
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
            *o.dx_exp = bdx - (cf.k_E1 - 1);
            bnb_exps_out(sv, cf, o);
        }
        const short lim = (short)((1 << (cf.k_E1 - 1)) - 1);
        const int16_t* src = w.lutq + cbase * 768;
        for (int v = threadIdx.x; v < st.CS * 96; v += kNT) {      // eight values per step, two per op
            const int i0 = v * 8, row = i0 >> 8, col = i0 & 255;
            const int bc = w.cbnd[cbase + row / 3];
            const short sh = (short)(bc == kSentinelLo ? 15 : min(bdx - bc, 15));
            const int4 q = *(const int4*)(src + i0);
            const int qw[4] = {q.x, q.y, q.z, q.w};
            uint32_t ow[2] = {0, 0};
#pragma unroll
            for (int h = 0; h < 4; h++) {
                short2v qv = __builtin_bit_cast(short2v, qw[h]);
                qv = ((qv >> sh) + (short)1) >> (short)1;
                qv = qv > lim ? lim : qv;
                qv = qv < (short)-lim ? (short)-lim : qv;
                const uint32_t b = (uint32_t)(uint16_t)qv.x & 0xffu | ((uint32_t)(uint16_t)qv.y & 0xffu) << 8;
                ow[h >> 1] |= b << (16 * (h & 1));
            }
            *(uint32_t*)(lut + row * kRowB + col) = ow[0];
            *(uint32_t*)(lut + row * kRowB + col + 4) = ow[1];
        }
    } else {
        copy_rows_to_lds<64 * 3 * 16 / kNT>(lut, w.lut + cbase * 768, st.CS * 3);
    }
    load_bwd_tab(tab, sv.btab + cbase * 256, st.CS, relu, true);
    __syncthreads();
    int g, rsub;
    if (!stream_lane(st, g, rsub)) return;
    const int c0 = (int)cbase + g * 4;
    const uint32_t* tb = tab + g * 4 * kRowW;
    const int64_t step = (int64_t)gridDim.x * st.rpi;
    auto elem = [&](uint32_t wx, uint32_t wd) {
        uint32_t ow = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t e = tb[i * kRowW + ((wx >> (8 * i)) & 0xff)];
            const int idx = (int)(e >> 16) + (sbyte(wd, i) & (int)(int8_t)(e & 0xff));
            ow |= (uint32_t)(uint8_t)lut[idx] << (8 * i);
        }
        return ow;
    };
    // full groups of U rows with the next group's loads in flight, then the rest
    constexpr int U = 4;
    int64_t r = (int64_t)blockIdx.x * st.rpi + rsub;
    const int64_t full_end = st.M - (U - 1) * step;
    uint32_t vx[U], vd[U], nx[U], nd[U];
    auto load = [&](int64_t r0, uint32_t* ax, uint32_t* ad) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            ax[u] = *(const uint32_t*)(x + (r0 + u * step) * st.C + c0);
            ad[u] = *(const uint32_t*)(dy + (r0 + u * step) * st.C + c0);
        }
    };
    if (r < full_end) load(r, vx, vd);
    while (r < full_end) {
        const int64_t rn = r + U * step;
        if (rn < full_end) load(rn, nx, nd);
#pragma unroll
        for (int u = 0; u < U; u++) *(uint32_t*)(dx + (r + u * step) * st.C + c0) = elem(vx[u], vd[u]);
#pragma unroll
        for (int u = 0; u < U; u++) { vx[u] = nx[u]; vd[u] = nd[u]; }
        r = rn;
    }
    for (; r < st.M; r += step)
        *(uint32_t*)(dx + r * st.C + c0) =
            elem(*(const uint32_t*)(x + r * st.C + c0), *(const uint32_t*)(dy + r * st.C + c0));
}

bool cfg_ok(const iseg_bn_cfg* c)
{
    if (!c) return false;
    auto in = [](int v, int lo, int hi) { return v >= lo && v <= hi; };
    return in(c->k_mu, 2, 16) && in(c->k_sigma, 2, 16) && in(c->k_xhat, 2, 16) &&
           in(c->k_gamma, 2, 8) && in(c->k_beta, 2, 8) && in(c->k_A, 2, 8) && in(c->k_E1, 2, 8) &&
           in(c->k_E2, 2, 16) && in(c->eps_code, 0, 1 << 15) && (c->relu == 0 || c->relu == 1);
}

bool shape_ok(int64_t M, int64_t C) { return M >= 1 && C >= 4 && M <= ((int64_t)1 << 22) && C <= (1 << 16); }

}  // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" size_t iseg_bn_saved_bytes(int64_t C) { return C > 0 ? saved_bytes(C) : 0; }

extern "C" size_t iseg_bn_fwd_ws(int64_t M, int64_t C)
{
    if (!shape_ok(M, C) || C % 4) return 0;
    return fwd_ws_bytes(C);
}

extern "C" size_t iseg_bn_bwd_ws(int64_t M, int64_t C)
{
    int cs = pick_cs(C, 64);
    if (!shape_ok(M, C) || !cs) return 0;
    return bwd_ws_bytes(make_stream(M, C, cs, 4, ISEG_BNB_ROWS, kMaxBlocks));
}

static int bn_fwd_impl(const int8_t* x, const int32_t* x_exp, int64_t M, int64_t C,
                       const int8_t* gamma_q, const int8_t* beta_q, const iseg_bn_cfg* cfg,
                       int8_t* y_out, int32_t* y_exp, void* saved,
                       void* ws, size_t ws_bytes, int32_t* dev_status, hipStream_t stream)
{
    if (M < 1 || C < 4) return ISEG_ERR_SHAPE;
    if (!shape_ok(M, C)) return ISEG_ERR_UNSUPPORTED;
    if (!x || !x_exp || !gamma_q || !beta_q || !y_out || !y_exp || !saved || !cfg_ok(cfg))
        return ISEG_ERR_ARG;
    if (C % 4 || (((uintptr_t)x | (uintptr_t)y_out) & 3)) return ISEG_ERR_UNSUPPORTED;
    const bool v16 = C % 16 == 0 && (((uintptr_t)x | (uintptr_t)y_out) & 15) == 0;
    if (!ws || ws_bytes < fwd_ws_bytes(C)) return ISEG_ERR_WORKSPACE;
    BnCfg cf = to_cfg(cfg);
    Saved sv = saved_map(saved, C);
    FwdWs w = fwd_ws_map(ws, C);
    // 16 channels per lane wherever the rows allow 16-byte loads
    auto stats = [&](auto cpl, auto gl) {
        constexpr int CPL = decltype(cpl)::value, G = decltype(gl)::value;
        const FStat st = make_fstat<CPL, G>(M, C);
        const dim3 sg((unsigned)st.gx, (unsigned)st.nsl);
        ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_STATS1, stream, (k_bnf_stats1<CPL, G>), sg, dim3(kNT), 0, stream, x, st, w);
        ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_STATS2, stream, (k_bnf_stats2<CPL, G>), sg, dim3(kNT), 0, stream, x, x_exp,
                          st, w, sv, cf, dev_status);
        hipLaunchKernelGGL(k_bnf_fin2, dim3((unsigned)ceil_div64(C, kFinCh)), dim3(kNT), 0, stream, x_exp, st, w, sv,
                           cf, gamma_q, beta_q);
    };
    const std::integral_constant<int, 16> v16c;
    if (C % 16 == 0 && ((uintptr_t)x & 15) == 0) {
        switch (fstat_g16(C)) {
        case 1: stats(v16c, std::integral_constant<int, 1>()); break;
        case 2: stats(v16c, std::integral_constant<int, 2>()); break;
        default: stats(v16c, std::integral_constant<int, 4>()); break;
        }
    } else {
        stats(std::integral_constant<int, 4>(), std::integral_constant<int, 16>());
    }
    auto apply = [&](auto cpl, auto gl) {
        constexpr int CPL = decltype(cpl)::value, G = decltype(gl)::value;
        // four rows per lane keep the most loads in flight; one where that
        // would use less than half the CUs
        const FStat s4 = make_fapply<CPL, G, 4>(M, C), s1 = make_fapply<CPL, G, 1>(M, C);
        if (s4.gx * s4.nsl > kMaxBlocks / 2)
            ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_APPLY, stream, (k_bnf_apply<CPL, G, 4>),
                              dim3((unsigned)s4.gx, (unsigned)s4.nsl), dim3(kNT), 0, stream, x, y_out, s4, sv, w, cf,
                              x_exp, gamma_q, beta_q, y_exp);
        else
            ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_APPLY, stream, (k_bnf_apply<CPL, G, 1>),
                              dim3((unsigned)s1.gx, (unsigned)s1.nsl), dim3(kNT), 0, stream, x, y_out, s1, sv, w, cf,
                              x_exp, gamma_q, beta_q, y_exp);
    };
    if (v16) {
        switch (fstat_g16(C)) {
        case 1: apply(v16c, std::integral_constant<int, 1>()); break;
        case 2: apply(v16c, std::integral_constant<int, 2>()); break;
        default: apply(v16c, std::integral_constant<int, 4>()); break;
        }
    } else {
        apply(std::integral_constant<int, 4>(), std::integral_constant<int, 16>());
    }
    return launch_ok();
}

extern "C" int iseg_bn_fwd(const int8_t* x, const int32_t* x_exp, int64_t M, int64_t C,
                           const int8_t* gamma_q, const int8_t* beta_q, const iseg_bn_cfg* cfg,
                           int8_t* y_out, int32_t* y_exp, void* saved,
                           void* ws, size_t ws_bytes, int32_t* dev_status, hipStream_t stream)
{
    return bn_fwd_impl(x, x_exp, M, C, gamma_q, beta_q, cfg, y_out, y_exp, saved, ws, ws_bytes, dev_status,
                       stream);
}

// ---------------------------------------------------------------------------
// iseg_bn_fwd_noalloc: the same forward with its workspace in a static device
// array (one copy per GPU, held until the process ends) instead of a caller
// buffer.  In host code `scratch` names a host-side stand-in, not device
// memory: its device address is looked up once per device with
// hipGetSymbolAddress (with that device current) and only that address is
// passed to the kernels.  The array starts at zero and every call leaves
// the forward's arrival counters at zero; the rest of the workspace is
// written before it is read within a call, so nothing needs clearing between
// calls.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t kBnScratchBytes = (size_t)1 << 20;
constexpr int kScratchDevices = 64;
__device__ __align__(256) unsigned char scratch[kBnScratchBytes];
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

static void* bn_scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

extern "C" size_t iseg_bn_fwd_noalloc_max_bytes(void) { return kBnScratchBytes; }

extern "C" int iseg_bn_fwd_noalloc(const int8_t* x, const int32_t* x_exp, int64_t M, int64_t C,
                                   const int8_t* gamma_q, const int8_t* beta_q, const iseg_bn_cfg* cfg,
                                   int8_t* y_out, int32_t* y_exp, void* saved, int32_t* dev_status,
                                   hipStream_t stream)
{
    const size_t need = iseg_bn_fwd_ws(M, C);
    if (need == 0) return M < 1 || C < 4 ? ISEG_ERR_SHAPE : ISEG_ERR_UNSUPPORTED;
    if (need > kBnScratchBytes) return ISEG_ERR_WORKSPACE;
    void* ws = bn_scratch_ptr();
    if (!ws) return ISEG_ERR_DEVICE;
    return bn_fwd_impl(x, x_exp, M, C, gamma_q, beta_q, cfg, y_out, y_exp, saved, ws, kBnScratchBytes,
                       dev_status, stream);
}

extern "C" int iseg_bn_bwd(const int8_t* dy, const int32_t* dy_exp, const int8_t* x,
                           int64_t M, int64_t C, const int8_t* gamma_q, const iseg_bn_cfg* cfg,
                           const void* saved, int8_t* dx_out, int32_t* dx_exp,
                           int64_t* dgamma, int64_t* dbeta, int32_t* dgamma_exp, int32_t* dbeta_exp,
                           void* ws, size_t ws_bytes, int32_t* dev_status, hipStream_t stream)
{
    if (M < 1 || C < 4) return ISEG_ERR_SHAPE;
    if (!shape_ok(M, C)) return ISEG_ERR_UNSUPPORTED;
    if (!dy || !dy_exp || !x || !gamma_q || !saved || !dx_out || !dx_exp || !dgamma || !dbeta ||
        !dgamma_exp || !dbeta_exp || !cfg_ok(cfg))
        return ISEG_ERR_ARG;
    int cs = pick_cs(C, 64);
    if (!cs || (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx_out) & 3)) return ISEG_ERR_UNSUPPORTED;
    Stream st = make_stream(M, C, cs, 4, ISEG_BNB_ROWS, kMaxBlocks);
    if (!ws || ws_bytes < bwd_ws_bytes(st)) return ISEG_ERR_WORKSPACE;
    BnCfg cf = to_cfg(cfg);
    Saved sv = saved_map((void*)saved, C);
    BwdWs w = bwd_ws_map(ws, st);
    dim3 sg = stream_grid(st);
    dim3 cb((unsigned)C);
    // E2 = SQ(gamma delta, k_E2) is exact when |gamma delta| <= 127^2 < 2^(k_E2-1)
    const int exact_e2 = cf.k_E2 >= 15;
    const BnbOut out{dy_exp, gamma_q, dgamma, dbeta, dgamma_exp, dbeta_exp, dx_exp, dev_status};
    if (exact_e2) {
        ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_STATS, stream, k_bnb_stats<1>, sg, dim3(kNT), 0, stream, dy, x, st, w,
                          sv, cf, out);
        hipLaunchKernelGGL(k_bnb_chan_exact, cb, dim3(256), 0, stream, M, (int)st.gx, (int)st.CS, w, sv, cf, out);
    } else {
        ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_STATS, stream, k_bnb_stats<2>, sg, dim3(kNT), 0, stream, dy, x, st,
                          w, sv, cf, out);
        hipLaunchKernelGGL(k_bnb_stats2, sg, dim3(kNT), 0, stream, dy, x, st, w, sv, cf, out);
        hipLaunchKernelGGL(k_bnb_lut, cb, dim3(256), 0, stream, M, (int)sg.y, w, sv, cf, out);
    }
    // the output pass needs no partials: its grid holds more rows per lane
    const Stream sa = make_stream(M, C, cs, 4, 8, kMaxBlocks);
    ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_APPLY, stream, k_bnb_apply, stream_grid(sa), dim3(kNT), 0, stream, dy, x,
                      dx_out, sa, w, sv, cf, out, exact_e2);
    return launch_ok();
}

// ---------------------------------------------------------------------------
// Inference with the frozen state of a calibration forward (the state that
// iseg_bn_fwd saved): the per-(channel, code) A table, built from that pass's
// n_mu, denominator and the fixed steps of Q_xhat and Q_A, is applied to new
// inputs.  A wide input (the raw int32 sums of a conv) first goes to the
// calibration's Z grid with a fixed-step quantizer (half-up, clipped to 8
// bits): the requant, L1BN, ReLU and Q_A of a layer in one pass.
// ---------------------------------------------------------------------------
namespace {
template <bool WIDE>
__global__ __launch_bounds__(256) void k_bn_infer(const void* __restrict__ in, const int32_t* in_exp,
                                                  const int32_t* w_exp, int64_t n4, int32_t C, Saved sv,
                                                  int8_t* __restrict__ out, int32_t* out_exp,
                                                  int32_t* dev_status)
{
    const int32_t ez = sv.hdr[3];
    const int32_t es = *in_exp + (WIDE ? *w_exp : 0);
    const int r = ez - es;                 // Z = sums 2^-r on the calibration's grid
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *out_exp = sv.hdr[2];
        if (!WIDE && r != 0) set_status(dev_status, ISEG_DEV_RANGE);   // codes on another grid
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const int c0 = (int)((i * 4) % C);
        int z[4];
        if (WIDE) {
            const int4 v = ((const int4*)in)[i];
            const int s[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                int64_t q;
                if (r > 0) q = ((int64_t)s[j] + ((int64_t)1 << (r - 1))) >> r;
                else if (r >= -32) q = (int64_t)s[j] * ((int64_t)1 << -r);
                else q = s[j] > 0 ? 128 : (s[j] < 0 ? -128 : 0);
                z[j] = (int)clamp_k(q, 8);
            }
        } else {
            const uint32_t v = ((const uint32_t*)in)[i];
#pragma unroll
            for (int j = 0; j < 4; j++) z[j] = (int)(int8_t)(v >> (8 * j));
        }
        uint32_t o = 0;
#pragma unroll
        for (int j = 0; j < 4; j++)
            o |= (uint32_t)(uint8_t)sv.acode[(int64_t)(c0 + j) * 256 + z[j] + 128] << (8 * j);
        ((uint32_t*)out)[i] = o;
    }
}
}  // namespace

extern "C" int iseg_bn_infer(const int8_t* z, const int32_t* z_exp, int64_t M, int64_t C, const void* saved,
                             int8_t* a_out, int32_t* a_exp, int32_t* dev_status, hipStream_t stream)
{
    if (M < 1 || C < 4) return ISEG_ERR_SHAPE;
    if (!shape_ok(M, C) || C % 4) return ISEG_ERR_UNSUPPORTED;
    if (!z || !z_exp || !saved || !a_out || !a_exp) return ISEG_ERR_ARG;
    if (((uintptr_t)z | (uintptr_t)a_out) & 3) return ISEG_ERR_UNSUPPORTED;
    const Saved sv = saved_map((void*)saved, C);
    const int64_t n4 = M * C / 4;
    hipLaunchKernelGGL(k_bn_infer<false>, dim3(grid_for(n4, 256 * 4, 4096)), dim3(256), 0, stream, z, z_exp,
                       z_exp, n4, (int32_t)C, sv, a_out, a_exp, dev_status);
    return launch_ok();
}

extern "C" size_t iseg_conv_bn_infer_ws(const iseg_conv_geom* g)
{
    const size_t cw = iseg_conv_fwd_ws(g, ISEG_OUT_RAW);
    if (!cw || !g) return 0;
    const int64_t P = (g->H + 2 * g->pad_h - g->dil_h * (g->R - 1) - 1) / g->stride_h + 1;
    const int64_t Q = (g->W + 2 * g->pad_w - g->dil_w * (g->S - 1) - 1) / g->stride_w + 1;
    return align256((size_t)(g->N * P * Q * g->K) * 4) + cw;
}

extern "C" int iseg_conv_bn_infer(const int8_t* x, const int32_t* x_exp, const int8_t* w, const int32_t* w_exp,
                                  const iseg_conv_geom* g, const void* saved, int8_t* a_out, int32_t* a_exp,
                                  void* ws, size_t ws_bytes, int32_t* dev_status, hipStream_t stream)
{
    if (!g || !saved || !a_out || !a_exp || !x_exp || !w_exp) return ISEG_ERR_ARG;
    const size_t need = iseg_conv_bn_infer_ws(g);
    if (!need) return ISEG_ERR_SHAPE;
    if (!ws || ws_bytes < need) return ISEG_ERR_WORKSPACE;
    const int64_t P = (g->H + 2 * g->pad_h - g->dil_h * (g->R - 1) - 1) / g->stride_h + 1;
    const int64_t Q = (g->W + 2 * g->pad_w - g->dil_w * (g->S - 1) - 1) / g->stride_w + 1;
    const int64_t M = g->N * P * Q, C = g->K;
    if (M < 1 || C < 4) return ISEG_ERR_SHAPE;
    if (!shape_ok(M, C) || C % 4 || ((uintptr_t)a_out & 3)) return ISEG_ERR_UNSUPPORTED;
    int32_t* sums = (int32_t*)ws;
    char* cws = (char*)ws + align256((size_t)(M * C) * 4);
    // the sums' own exponent slot: the conv writes x_exp + w_exp there; the pass reads both inputs' exponents
    int32_t* sexp = (int32_t*)a_exp;
    int rc = iseg_conv_fwd(x, x_exp, w, w_exp, g, ISEG_OUT_RAW, sums, sexp, cws, ws_bytes - (cws - (char*)ws),
                           dev_status, stream);
    if (rc) return rc;
    const Saved sv = saved_map((void*)saved, C);
    const int64_t n4 = M * C / 4;
    hipLaunchKernelGGL(k_bn_infer<true>, dim3(grid_for(n4, 256 * 4, 4096)), dim3(256), 0, stream, sums, x_exp,
                       w_exp, n4, (int32_t)C, sv, a_out, a_exp, dev_status);
    return launch_ok();
}
