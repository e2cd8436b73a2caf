// bn.hip -- L1 batch normalization (Eq. 12-15) and its backward on gfx950.
//
// Because the input of BN is an int8 code tensor, every per-element quantity
// of the forward (xhat_q, y, the ReLU mask, sgn(x - mu_q), the output code A)
// is a function of (channel, input code) only, and the backward's dx code is
// a function of (channel, sgn class, masked error code).  The work therefore
// splits into
//   * streaming passes over [M, C]: 16 channels per lane in the forward where the
//     rows allow 16-byte loads, else four, four rows in flight per lane,
//     per-channel sums reduced in LDS and written as one partial per block and
//     channel (stats2 instead adds its two sums to the channel's word by one
//     64-bit atomic per block: whole numbers, so in any order the same);
//   * finalize steps that reduce the partials and do the exact rational
//     arithmetic once per channel or per table entry, in kernels of their own.
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
// Backward: stats (block partials of sum delta, sum delta*xhat, sum sgn and the
//           per-class extremes of delta) -> per-channel kernel (dgamma, dbeta,
//           the channel's bound on E1's exponent, its dx values staged at that
//           bound) -> apply (E1's exponent from the channels' bounds; staged
//           values rounded into the gather table).  Rounding E2 (k_E2 < 15) adds
//           a second streaming pass before the per-channel kernel, with E2's
//           scale from the first pass's block maxima of |gamma delta|.
#include <algorithm>
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

constexpr int kNT = ISEG_BN_NT;
constexpr int kWaves = kNT / 64;       // waves per streaming block

// the CPL channels of a lane's row (4: one dword, 16: one 16-byte vector)
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

struct OpAdd { template <typename T> __device__ T operator()(T a, T b) const { return a + b; } };
struct OpMin { template <typename T> __device__ T operator()(T a, T b) const { return a < b ? a : b; } };
struct OpMax { template <typename T> __device__ T operator()(T a, T b) const { return a > b ? a : b; } };

// LDS tables are kept one dword longer per row than in global memory: a
// table row is 256 entries (a multiple of the bank count), so without the skew
// every channel's entry for the same input code would sit in the same bank,
// and real activations concentrate on a few codes.
constexpr int kRowB = 256 + 4;      // bytes per row of a byte table in LDS
constexpr int kRowW = 256 + 1;      // dwords per row of a dword table in LDS

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
    int32_t paired;                  // slice_grid's order of the blocks
};

// Blocks of a slice: one per tile, or an equal share of kMaxBlocks in a multiple
// of the eight XCDs.  Consecutive blocks go to the XCDs in turn, so the blocks that
// read the same rows of different slices then share an L2; rows whose length is
// no multiple of 128 bytes have most of their lines in two slices, which every
// XCD otherwise fetches for itself (131072 rows, forward / backward, 85 blocks
// against 80 at 176 channels: 51.7 / 65.8 -> 36.4 / 51.6 us, 51 against 48 at 272:
// 73.0 / 95.4 -> 45.1 / 70.3, 21 against 16 at 720, 32768 rows: 52.1 / 71.4 -> 36.0 / 59.5).
int32_t slice_blocks(int64_t nsl, int64_t ntiles)
{
    int64_t n = kMaxBlocks / nsl;
    if (ntiles <= n) return (int32_t)ntiles;
    if (nsl > 1 && n >= 8) n &= ~(int64_t)7;
    return (int32_t)(n < 1 ? 1 : n);
}

// The grid of a streaming pass.  Past 2048 channels a slice has fewer blocks than
// there are XCDs; the two slices of each 128-byte line then take every second
// eight of one row of blocks, which puts the blocks of the same rows on one XCD
// again (8192 x 4096 codes: the first and the output pass of the forward 12.8 ->
// 9.7 and 21.4 -> 18.2 us, those of the backward 33.3 -> 26.2 and 38.3 -> 28.4).
dim3 slice_grid(const FStat& f)
{
    if (!f.paired) return dim3((unsigned)f.gx, (unsigned)f.nsl);
    return dim3((unsigned)(ceil_div64(ceil_div64(f.nsl, 2) * f.gx, 8) * 16));
}

// block bx of slice by; false: none (a block past the last slice)
template <bool PAIRED>
__device__ __forceinline__ bool slice_of(const FStat& st, int& bx, int& by)
{
    bx = blockIdx.x;
    by = blockIdx.y;
    if constexpr (!PAIRED) return true;
    const int q = blockIdx.x, v = (q >> 4) * 8 + (q & 7), pair = v / st.gx;
    bx = v - pair * st.gx;
    by = 2 * pair + ((q >> 3) & 1);
    return by < st.nsl;
}

// f(PAIRED), for the geometries wide enough to have it
template <int CS, typename F>
void with_paired(const FStat& st, F f)
{
    if constexpr (CS == 64) {
        if (st.paired) return f(std::true_type());
    }
    f(std::false_type());
}

template <int CPL, int G>
FStat make_fstat(int64_t M, int64_t C)
{
    constexpr int CS = CPL * G, TR = 4 * kNT / G;
    FStat f;
    f.M = M; f.C = (int32_t)C;
    f.nsl = (int32_t)ceil_div64(C, CS);
    f.ntiles = (int32_t)ceil_div64(M, TR);
    f.pad = (int32_t)((int64_t)f.ntiles * TR - M);
    f.gx = slice_blocks(f.nsl, f.ntiles);
    f.paired = kMaxBlocks / f.nsl < 8;
    return f;
}

// lanes per row of the 16-channel-lane variant
int fstat_g16(int64_t C) { return C <= 16 ? 1 : (C <= 32 ? 2 : 4); }

// ---------------------------------------------------------------------------
// forward workspace
// ---------------------------------------------------------------------------
struct FwdWs {
    int32_t* b_glob;                 // exponent of Q_xhat's scale (fin2, block 0)
    int32_t* bnd;                    // [block] largest bound on it (k_bnf_den; at most 64 blocks)
    int2* part;                      // [slice][gx][CS] sum q; (min q + 128) | (max q + 128) << 16
    unsigned long long* acc;         // [C] sum |q - T| (low half) and sum |q - T - 1| (high half)
    int32_t* sumq;                   // [C] sum q
    unsigned long long* maxYc;       // [C] max |ReLU(y)| of channel c over its occupied codes (fin2);
                                     // in the space of `part`, which no kernel from fin2 on reads
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
    return 512 + align256(fwd_part_entries(C) * 8) + align256(c * 8) + align256(c * 4);
}

FwdWs fwd_ws_map(void* base, int64_t C)
{
    char* p = (char*)base;
    const size_t c = (size_t)C;
    FwdWs w;
    w.b_glob = (int32_t*)p; p += 256;
    w.bnd = (int32_t*)p; p += 256;
    w.part = (int2*)p;
    w.maxYc = (unsigned long long*)p; p += align256(fwd_part_entries(C) * 8);
    w.acc = (unsigned long long*)p; p += align256(c * 8);
    w.sumq = (int32_t*)p;
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
    if constexpr (sizeof(T) == 8) {
        const uint64_t x = (uint64_t)a, y = (uint64_t)b;
        uint32_t al, ah, bl, bh;
        if constexpr (O == 32) {
            const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
            al = l[0]; bl = l[1]; ah = h[0]; bh = h[1];
        } else {
            const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
            al = l[0]; bl = l[1]; ah = h[0]; bh = h[1];
        }
        return op((T)((uint64_t)al | ((uint64_t)ah << 32)), (T)((uint64_t)bl | ((uint64_t)bh << 32)));
    } else if constexpr (O == 32) {
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
        if constexpr (sizeof(T) == 8) {
            const int l = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(uint64_t)v, 0x120 + N, 0xf, 0xf, false);
            const int h = __builtin_amdgcn_update_dpp(0, (int)((uint64_t)v >> 32), 0x120 + N, 0xf, 0xf, false);
            v = op(v, (T)((uint64_t)(uint32_t)l | ((uint64_t)(uint32_t)h << 32)));
        } else {
            const int u = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, false);
            v = op(v, __builtin_bit_cast(T, u));
        }
    };
    if constexpr (G <= 8) ror(std::integral_constant<int, 8>());
    if constexpr (G <= 4) ror(std::integral_constant<int, 4>());
    if constexpr (G <= 2) ror(std::integral_constant<int, 2>());
    if constexpr (G <= 1) ror(std::integral_constant<int, 1>());
    return v;
}

// Fold N = CPL values (channel i of the lane) over the wave's rows: the lane
// ends with channels fold_ch(l) + 0 .. CPL / 4 - 1 in v[0 ..].  Two reduce-scatter steps halve
// the channels a lane holds, so 16 channels cost 12 swaps instead of 32.
template <int CPL, int G, typename T, typename Op>
__device__ __forceinline__ void wave_fold(T (&v)[CPL], Op op)
{
#pragma unroll
    for (int i = 0; i < CPL / 2; i++) v[i] = swap_fold<32>(v[i], v[i + CPL / 2], op);
#pragma unroll
    for (int i = 0; i < CPL / 4; i++) v[i] = swap_fold<16>(v[i], v[i + CPL / 4], op);
#pragma unroll
    for (int i = 0; i < CPL / 4; i++) v[i] = row_fold<G>(v[i], op);
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
__device__ __forceinline__ void fstat_rows(const FStat& st, int bx, const int8_t* __restrict__ x, int c0, F f)
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
    int tile = bx;
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
// 8.5 us; on 8192 x 256 the 64-channel slices cost this pass 4.7 -> 5.5 us and
// save the next one, which reads their partials, 13.2 -> 5.4).  Sums by v_dot4 against a
// selector byte, minima and maxima as packed 16-bit operations on the bytes in
// the high halves (the low byte below them cannot change which high byte wins).
template <int CPL, int G, bool PAIRED>
__global__ __launch_bounds__(1024) void k_bnf_stats1(const int8_t* __restrict__ x, FStat st, FwdWs w)
{
    int bx, by;
    if (!slice_of<PAIRED>(st, bx, by)) return;
    constexpr int CS = CPL * G, DW = CPL / 4;
    __shared__ int32_t sS[kWaves * CS];
    __shared__ int32_t sMm[kWaves * CS];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = t % G;
    const int c0 = by * CS + g * CPL;
    int s[CPL];
    short2v mnh[DW], mnl[DW], mxh[DW], mxl[DW];
#pragma unroll
    for (int i = 0; i < CPL; i++) s[i] = 0;
#pragma unroll
    for (int j = 0; j < DW; j++) { mnh[j] = mnl[j] = (short)0x7fff; mxh[j] = mxl[j] = (short)-0x8000; }
    fstat_rows<CPL, G>(st, bx, x, c0 < st.C ? c0 : 0, [&](const Vec<CPL>* v, const bool* ok) {
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
    const int c = by * CS + t;
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
        w.part[((int64_t)by * st.gx + bx) * CS + t] = make_int2(bs, lo | (hi << 16));
        if (bx == 0 && c < st.C) w.acc[c] = 0;
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
template <int CPL, int G, bool PAIRED>
__global__ __launch_bounds__(1024) void k_bnf_stats2(const int8_t* __restrict__ x, const int32_t* x_exp,
                                                    FStat st, FwdWs w, Saved sv, BnCfg cf, int32_t* dev_status)
{
    int bx, by;
    if (!slice_of<PAIRED>(st, bx, by)) return;
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
        const int2* ps = w.part + (int64_t)by * st.gx * CS;
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
            const int c = by * CS + t;
            if (bx == 0 && c < st.C) {
                sv.n_mu[c] = nm;
                sv.qmin[c] = lo - 128;
                sv.qmax[c] = hi - 128;
                w.sumq[c] = sum;
            }
        }
        __syncthreads();
    }
    const int c0 = by * CS + g * CPL;
    uint32_t a0[CPL], a1[CPL], r0[CPL];
#pragma unroll
    for (int i = 0; i < CPL; i++) {
        a0[i] = a1[i] = 0;
        r0[i] = (uint32_t)sRef[g * CPL + i] * 0x01010101u;
    }
    fstat_rows<CPL, G>(st, bx, x, c0 < st.C ? c0 : 0, [&](const Vec<CPL>* v, const bool* ok) {
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
    const int c = by * CS + t;
    if (!sx_ok(s_in) && bx == 0 && by == 0 && t == 0) set_status(dev_status, ISEG_DEV_RANGE);
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
// codes (y is monotone in q, so over qmin and qmax).  Up to kDenWide channels
// every block forms all channels' denominators and bounds on b itself (at most
// two per thread): the arrival, reload and arithmetic of a tail in
// the statistics pass took longer.  Bound by latency: the loads, two exact
// divisions and three barriers.  PRE: k_bnf_den has formed them (forward of 64 x
// 4096 codes: 39.0 -> 37.1 us, 64 x 65536: 572 -> 256; 64 x 2048: 29.5 against 30.3).
constexpr int kFinCh = kNT / 256;              // channels at a time
constexpr int kFinGrp = 16;                    // at most so many groups of them per block
constexpr int64_t kDenWide = 2048;

// a channel's denominator, and its bound on b (its largest |x-hat|: at qmin or
// qmax, x-hat is linear in q)
__device__ __forceinline__ int bnf_bound(int32_t lo, int32_t hi, int32_t nm, int32_t den, int32_t s_x, int e_mu,
                                         int e_sig)
{
    const int64_t D0 = bn_D(lo, s_x, nm, e_mu), D1 = bn_D(hi, s_x, nm, e_mu);
    const uint64_t m0 = (uint64_t)(D0 < 0 ? -D0 : D0), m1 = (uint64_t)(D1 < 0 ? -D1 : D1);
    const uint64_t m = m0 > m1 ? m0 : m1;
    return m ? ceil_pow2_exp64(m, (uint64_t)den) + min(s_x, e_mu) - e_sig : kSentinelLo;
}

// wide layers: the denominators, and the largest bound of each block's kNT channels
__global__ __launch_bounds__(1024) void k_bnf_den(const int32_t* x_exp, FStat st, FwdWs w, Saved sv, BnCfg cf)
{
    __shared__ int32_t rsh[kWaves];
    const int c = blockIdx.x * kNT + threadIdx.x;
    const int e_mu = 2 - cf.k_mu, e_sig = 2 - cf.k_sigma;
    const int32_t s_in = *x_exp, s_x = sx_ok(s_in) ? s_in : -14;
    int best = kSentinelLo;
    if (c < st.C) {
        const int32_t nm = sv.n_mu[c], ns = bnf_sigma(w.acc[c], w.sumq[c], st, s_x, nm, e_mu, cf);
        const int32_t den = max(ns + cf.eps_code, 1);
        sv.n_sigma[c] = ns;
        sv.den[c] = den;
        best = bnf_bound(sv.qmin[c], sv.qmax[c], nm, den, s_x, e_mu, e_sig);
    }
    best = block_max_nt(best, rsh);
    if (threadIdx.x == 0) w.bnd[blockIdx.x] = best;
}

template <bool PRE>
__global__ __launch_bounds__(1024) void k_bnf_fin2(const int32_t* x_exp, FStat st, int grp, FwdWs w, Saved sv,
                                                  BnCfg cf, const int8_t* gamma_q, const int8_t* beta_q)
{
    __shared__ int32_t rsh[kWaves], sNs[kFinGrp * kFinCh], sDen[kFinGrp * kFinCh];
    __shared__ uint64_t sBal[2][kWaves][3], sAy[2][kFinCh][2];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, lc = t >> 8;
    const int cfirst = blockIdx.x * grp * kFinCh;          // the block's channels: grp groups of kFinCh
    const int q = (t & 255) - 128;
    // every load of the first round goes out before the first wait (no branch on
    // a loaded value in between)
    const int32_t s_in = *x_exp;
    const int cs0 = cfirst + lc < st.C ? cfirst + lc : 0;
    int32_t nmu = sv.n_mu[cs0], qlo = sv.qmin[cs0], qhi = sv.qmax[cs0];
    int gq = gamma_q[cs0], bq = beta_q[cs0];
    const int e_mu = 2 - cf.k_mu, e_sig = 2 - cf.k_sigma;
    const int32_t s_x = sx_ok(s_in) ? s_in : -14;     // outputs unspecified, shifts defined
    int best = kSentinelLo;
    if constexpr (PRE) {
        const int nb = (st.C + kNT - 1) / kNT;        // at most 64
        best = w.bnd[lane < nb ? lane : 0];
        if (t < grp * kFinCh) sDen[t] = sv.den[cfirst + t < st.C ? cfirst + t : 0];
    } else {
        const int k0 = t < st.C ? t : 0;
        int32_t nm = sv.n_mu[k0], lo = sv.qmin[k0], hi = sv.qmax[k0], sumq = w.sumq[k0];
        unsigned long long acc = w.acc[k0];
        for (int k = t; k < st.C; k += kNT) {
            if (k != t) { nm = sv.n_mu[k]; lo = sv.qmin[k]; hi = sv.qmax[k]; sumq = w.sumq[k]; acc = w.acc[k]; }
            const int32_t ns = bnf_sigma(acc, sumq, st, s_x, nm, e_mu, cf);
            const int32_t den = max(ns + cf.eps_code, 1);
            if (k >= cfirst && k < cfirst + grp * kFinCh) { sNs[k - cfirst] = ns; sDen[k - cfirst] = den; }
            best = max(best, bnf_bound(lo, hi, nm, den, s_x, e_mu, e_sig));
        }
    }
    for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
    if (lane == 0) rsh[wv] = best;
    __syncthreads();
    int b = rsh[0];
#pragma unroll
    for (int k = 1; k < kWaves; k++) b = max(b, rsh[k]);
    if (b == kSentinelLo) b = 0;
    if (blockIdx.x == 0 && t == 0) *w.b_glob = b;
    const FwdExps e = fwd_exps(s_x, b, cf);
    for (int g = 0; g < grp; g++) {
        const int c = cfirst + g * kFinCh + lc;
        const bool own = c < st.C;
        if (g) {
            const int cs = own ? c : 0;
            nmu = sv.n_mu[cs]; qlo = sv.qmin[cs]; qhi = sv.qmax[cs];
            gq = gamma_q[cs]; bq = beta_q[cs];
        }
        const int32_t den = own ? sDen[g * kFinCh + lc] : 1;
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
        if (lane == 0) { sBal[g & 1][wv][0] = m0; sBal[g & 1][wv][1] = m1; sBal[g & 1][wv][2] = m2; }
        const uint64_t ay = wide ? (uint64_t)abs128(Yw) : (uint64_t)(Yr < 0 ? -Yr : Yr);
        if (q == qlo) sAy[g & 1][lc][0] = ay;
        if (q == qhi) sAy[g & 1][lc][1] = ay;
        __syncthreads();
        const uint64_t mx = sAy[g & 1][lc][0] > sAy[g & 1][lc][1] ? sAy[g & 1][lc][0] : sAy[g & 1][lc][1];
        if (own && (t & 255) == 0) {
            int v[4] = {128, 128, 128, -129};
#pragma unroll
            for (int k = 3; k >= 0; k--)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    const uint64_t bm = sBal[g & 1][wv + k][j];
                    if (bm) v[j] = -128 + 64 * k + __builtin_ctzll(bm);
                }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint64_t bm = sBal[g & 1][wv + k][2];
                if (bm) v[3] = -128 + 64 * k + 63 - __builtin_clzll(bm);
            }
            sv.t0[c] = v[0]; sv.p0[c] = v[1]; sv.mlo[c] = v[2]; sv.mhi[c] = v[3];
            if constexpr (!PRE) {
                sv.n_sigma[c] = sNs[g * kFinCh + lc];
                sv.den[c] = den;
            }
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
    f.gx = slice_blocks(f.nsl, f.ntiles);
    f.paired = kMaxBlocks / f.nsl < 8;
    return f;
}

template <int CPL, int G, int U, bool PAIRED>
__global__ __launch_bounds__(1024) void k_bnf_apply(const int8_t* __restrict__ x, int8_t* __restrict__ y,
                                                   FStat st, Saved sv, FwdWs w, BnCfg cf, const int32_t* x_exp,
                                                   const int8_t* gamma_q, const int8_t* beta_q, int32_t* y_exp)
{
    int bx, by;
    if (!slice_of<PAIRED>(st, bx, by)) return;
    constexpr int CS = CPL * G, RPI = kNT / G, TV = (CS * 32 + kNT - 1) / kNT;
    __shared__ __attribute__((aligned(16))) int8_t lut[CS * kRowB];
    __shared__ uint64_t rmax[kWaves];
    const int t = threadIdx.x, g = t % G, rsub = t / G;
    const int c0 = by * CS + g * CPL, cb = by * CS;
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
    const int64_t nall = (int64_t)st.C * 64, nb = (int64_t)st.gx * st.nsl;
    const int64_t per = (nall + nb - 1) / nb;
    const int64_t i0 = ((int64_t)by * st.gx + bx) * per;
    const int64_t i1 = i0 + per < nall ? i0 + per : nall;
    int64_t ia = i0 + t;
    const int64_t il = ia < i1 ? ia : 0;
    short4v xq = *(const short4v*)(sv.xcode + il * 4);
    int gq = gamma_q[il >> 6], bq = beta_q[il >> 6];
    int tile = bx;
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
    if (bx == 0 && by == 0 && t == 0 && ok) {
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
    int32_t* pF;                     // [streaming block] largest |gamma delta| of the block (rounding E2)
    int32_t *p_sd, *p_z, *p_mmA, *p_mmB;   // [slice][gx][CS] partials (per-class extremes packed as bytes)
    long long *p_sdn, *p_sf, *p_sfn;       // [slice][gx][CS]
    int32_t* cbnd;                   // [C] each channel's bound on E1's exponent
    int16_t* lutq;                   // [C][3][256] dx values at the channel's own bound
};

// streaming blocks of either pass: at most max(kMaxBlocks, slices), CS <= 64
size_t bwd_blocks(int64_t C)
{
    const int64_t n64 = ceil_div64(C, 64);
    return (size_t)(n64 > kMaxBlocks ? n64 : kMaxBlocks);
}

size_t bwd_ws_bytes(int64_t C)
{
    const size_t nb = bwd_blocks(C), pc = nb * 64, c = (size_t)C;
    return align256(nb * 4) + 4 * align256(pc * 4) + 3 * align256(pc * 8) + align256(c * 4) +
           align256(c * 768 * 2);
}

BwdWs bwd_ws_map(void* base, int64_t C)
{
    char* p = (char*)base;
    const size_t nb = bwd_blocks(C), pc = nb * 64, c = (size_t)C;
    BwdWs w;
    w.pF = (int32_t*)p; p += align256(nb * 4);
    w.p_sd = (int32_t*)p; p += align256(pc * 4);
    w.p_z = (int32_t*)p; p += align256(pc * 4);
    w.p_mmA = (int32_t*)p; p += align256(pc * 4);
    w.p_mmB = (int32_t*)p; p += align256(pc * 4);
    w.p_sdn = (long long*)p; p += align256(pc * 8);
    w.p_sf = (long long*)p; p += align256(pc * 8);
    w.p_sfn = (long long*)p; p += align256(pc * 8);
    w.cbnd = (int32_t*)p; p += align256(c * 4);
    w.lutq = (int16_t*)p;
    return w;
}

// streaming geometry of the backward: slices of 4 G channels (four per lane),
// tiles of U kNT / G rows
template <int G, int U>
FStat make_bstat(int64_t M, int64_t C)
{
    constexpr int CS = 4 * G, TR = U * kNT / G;
    FStat f;
    f.M = M; f.C = (int32_t)C;
    f.nsl = (int32_t)ceil_div64(C, CS);
    f.ntiles = (int32_t)ceil_div64(M, TR);
    f.pad = (int32_t)((int64_t)f.ntiles * TR - M);
    f.gx = slice_blocks(f.nsl, f.ntiles);
    f.paired = kMaxBlocks / f.nsl < 8;
    return f;
}

// Per-class extremes of the masked delta travel between kernels as bytes:
// low ends as lo + 128 (255 for an empty class), high ends as hi + 128 (0 for
// an empty class), so a byte-wise min / max merges them and an empty class
// still reads lo > hi.  A = (lo, hi) of classes -1 and 0, B = (lo, hi) of +1.
__device__ __forceinline__ void mm_merge(uint32_t A, uint32_t B, int* lo3, int* hi3)
{
    lo3[0] = min(lo3[0], (int)(A & 0xff)); hi3[0] = max(hi3[0], (int)((A >> 8) & 0xff));
    lo3[1] = min(lo3[1], (int)((A >> 16) & 0xff)); hi3[1] = max(hi3[1], (int)(A >> 24));
    lo3[2] = min(lo3[2], (int)(B & 0xff)); hi3[2] = max(hi3[2], (int)((B >> 8) & 0xff));
}

struct BnbOut {
    const int32_t* dy_exp;
    const int8_t* gamma_q;
    int64_t *dgamma, *dbeta;
    int32_t *dgamma_exp, *dbeta_exp, *dx_exp, *dev_status;
};

// E2's requant shift from max |gamma delta|
__device__ __forceinline__ int bnb_r2_of(int32_t maxF, const BnCfg& cf)
{
    return maxF > 0 ? bitlen_u64((uint64_t)maxF) - (cf.k_E2 - 1) : 0;
}

// the largest |gamma delta| from the streaming blocks' partials (every thread
// of the block gets it; sh holds one value per wave)
__device__ __forceinline__ int32_t bnb_max_F(const int32_t* pF, int n, int32_t* sh)
{
    int32_t m = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = max(m, pF[i]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    m = sh[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); k++) m = max(m, sh[k]);
    return m;
}

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

struct OpPkMax {
    __device__ uint32_t operator()(uint32_t a, uint32_t b) const
    {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2v, a),
                                                                      __builtin_bit_cast(ushort2v, b)));
    }
};
struct OpPkMin {
    __device__ uint32_t operator()(uint32_t a, uint32_t b) const
    {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(ushort2v, a),
                                                                      __builtin_bit_cast(ushort2v, b)));
    }
};

// Streaming pass of the backward.  MODE 0 / 1 (exact / rounding E2, first
// pass): sum delta, sum delta xhat, sum sgn and the extremes of the masked
// delta d per sgn class.  MODE 2 (rounding E2, second pass): sum f and sum f
// xhat, f = SQ(gamma d, k_E2).
//
// A per-(channel, code) entry in LDS holds xhat (bits 16-31, zero where the
// ReLU masks), the class byte (bits 8-15: 0x00 for sgn -1, 0x80 for 0, 0xff for
// +1) and the mask byte.  Two rows of one channel make one packed step: with
// d' = d + 128 (128 where masked), the key (class << 8) | d' has the extremes of
// class +1 at its maximum and of class -1 at its minimum, the key with the
// class byte inverted the other two; sums come from v_dot4 / v_dot2 on the
// same packed values.  11.5 VALU operations per element instead of 20; a wave's
// VALU operation of this mix takes 4.4 clocks, so they and the 2 bytes per
// element cost about the same (131072 x 256 codes: 28.2 -> 22.5 us, 3.0 TB/s,
// 3 us of it the 64 KB table; 1024 x 16: 10.2 -> 5.4; rounding E2, both passes at
// 12255 x 144: 36 -> 16.5 with the arrivals and tails gone).  Class 0 holds at
// most one code of a channel, and only where mu_q is a code: channels of a
// wave that have one (in their occupied range) take six more operations.
constexpr int kBndU = 4;                 // rows per lane and tile

template <int G, int MODE, bool PAIRED>
__global__ __launch_bounds__(1024) void k_bnb_stats(const int8_t* __restrict__ dy, const int8_t* __restrict__ x,
                                                   FStat st, BwdWs w, Saved sv, BnCfg cf, BnbOut out)
{
    int bx, by;
    if (!slice_of<PAIRED>(st, bx, by)) return;
    constexpr int CS = 4 * G, RPI = kNT / G, U = kBndU, TR = U * RPI, TV = CS * 64 / kNT;
    __shared__ __attribute__((aligned(16))) uint32_t tab[CS * kRowW];
    __shared__ int32_t rsh[kWaves], sZf[CS];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = t % G, rsub = t / G;
    const int cb = by * CS, c0 = cb + g * 4;
    const int64_t last = st.M - 1;
    const int8_t* xb = x + (c0 < st.C ? c0 : 0);
    const int8_t* db = dy + (c0 < st.C ? c0 : 0);
    // table pieces, class-0 flags and the first tile all load together
    uint4 tv[TV];
#pragma unroll
    for (int k = 0; k < TV; k++) {
        const int i = t + k * kNT, row = i >> 6;
        const int c = cb + row < st.C ? cb + row : cb;
        tv[k] = ((const uint4*)(sv.btab + (int64_t)c * 256))[i & 63];
    }
    int zero_cls = 0;
    if (MODE != 2 && t < CS) {
        const int c = cb + t < st.C ? cb + t : cb;
        const int t0 = sv.t0[c], p0 = sv.p0[c], lo = sv.qmin[c], hi = sv.qmax[c];
        zero_cls = t0 < p0 && t0 >= lo && t0 <= hi;
    }
    uint32_t vx[U], vd[U], nx[U], nd[U];
    auto load = [&](int tile, uint32_t* ax, uint32_t* ad) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t r = (int64_t)tile * TR + u * RPI + rsub, rr = (r < last ? r : last) * st.C;
            ax[u] = *(const uint32_t*)(xb + rr);
            ad[u] = *(const uint32_t*)(db + rr);
        }
    };
    int tile = bx;
    if (tile < st.ntiles) load(tile, vx, vd);
    int gam[4] = {0, 0, 0, 0};
    int r2 = 0;
    if constexpr (MODE == 2) {
#pragma unroll
        for (int i = 0; i < 4; i++) gam[i] = out.gamma_q[(c0 < st.C ? c0 : 0) + i];
        r2 = bnb_r2_of(bnb_max_F(w.pF, st.gx * st.nsl, rsh), cf);
    }
    if (t < CS) sZf[t] = zero_cls;
#pragma unroll
    for (int k = 0; k < TV; k++) {
        const int i = t + k * kNT;
        const uint32_t e4[4] = {tv[k].x, tv[k].y, tv[k].z, tv[k].w};
        uint32_t* d = tab + (i >> 6) * kRowW + (i & 63) * 4;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint32_t e = e4[j];
            const int sg = ((int)(e << 22)) >> 30;
            const uint32_t cls = sg < 0 ? 0u : (sg > 0 ? 0xff00u : 0x8000u);
            d[j] = (!cf.relu || (e & 1) ? (e & 0xffff0000u) | 0xffu : 0u) | cls;
        }
    }
    __syncthreads();
    // zf[i]: some lane's i-th channel has a code in class 0 (wave-uniform, and
    // the same in every wave)
    bool zf[4], zflag = false;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        zf[i] = MODE != 2 && __ballot(sZf[g * 4 + i] != 0) != 0;
        zflag |= zf[i];
    }
    const uint32_t* tb = tab + g * 4 * kRowW;
    uint32_t sd[4] = {0, 0, 0, 0}, z[4] = {0, 0, 0, 0};
    int32_t sn[4] = {0, 0, 0, 0}, sf[4] = {0, 0, 0, 0};
    int64_t sdn[4] = {0, 0, 0, 0}, sff[4] = {0, 0, 0, 0};
    uint32_t mx1[4] = {0, 0, 0, 0}, mx2[4] = {0, 0, 0, 0}, mn1[4] = {~0u, ~0u, ~0u, ~0u}, mn2[4] = {~0u, ~0u, ~0u, ~0u};
    uint32_t mx0[4] = {0, 0, 0, 0}, mn0[4] = {~0u, ~0u, ~0u, ~0u}, np[4] = {0, 0, 0, 0};
    // one row pair; v0, v1: whether the rows count (a repeated row only repeats keys)
    auto pair = [&](uint32_t x0, uint32_t x1, uint32_t d0, uint32_t d1, auto all, bool v0, bool v1) {
        d0 ^= kSign4; d1 ^= kSign4;
        const uint32_t vsel = decltype(all)::value ? 0x00010001u : (v0 ? 1u : 0u) | (v1 ? 0x10000u : 0u);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t e0 = tb[i * kRowW + ((x0 >> (8 * i)) & 0xff)];
            const uint32_t e1 = tb[i * kRowW + ((x1 >> (8 * i)) & 0xff)];
            uint32_t xp = __builtin_amdgcn_perm(e1, e0, 0x07060302u);
            const uint32_t cp = __builtin_amdgcn_perm(e1, e0, 0x05040100u);
            const uint32_t dp = __builtin_amdgcn_perm(d1, d0, 0x0d000d00u | (uint32_t)(4 + i) << 16 | (uint32_t)i);
            const uint32_t k1 = (cp & dp) | (~cp & 0x00800080u);
            if constexpr (!decltype(all)::value) xp &= vsel * 0xffffu;
            short2v dm = __builtin_bit_cast(short2v, k1 & 0x00ff00ffu) - (short)128;
            const short2v xs = __builtin_bit_cast(short2v, xp);
            if constexpr (MODE == 2) {
                short2v f = dm * (short)gam[i];
                if (r2 > 0) f = (f + (short)(1 << (r2 - 1))) >> (short)r2;
                else f = f << (short)-r2;
                const short lim = (short)((1 << (cf.k_E2 - 1)) - 1);
                f = __builtin_elementwise_min(f, (short2v)lim);
                f = __builtin_elementwise_max(f, (short2v)(short)-lim);
                sf[i] = __builtin_amdgcn_sdot2(f, __builtin_bit_cast(short2v, vsel), sf[i], false);
                sn[i] = __builtin_amdgcn_sdot2(f, xs, sn[i], false);
            } else {
                const uint32_t k2 = k1 ^ 0xff00ff00u;
                mx1[i] = OpPkMax()(mx1[i], k1);
                mn1[i] = OpPkMin()(mn1[i], k1);
                mx2[i] = OpPkMax()(mx2[i], k2);
                mn2[i] = OpPkMin()(mn2[i], k2);
                sd[i] = __builtin_amdgcn_udot4(k1, vsel, sd[i], false);
                z[i] = __builtin_amdgcn_udot4(k1, vsel << 8, z[i], false);
                sn[i] = __builtin_amdgcn_sdot2(dm, xs, sn[i], false);
                if (zf[i]) {                 // class 0 to the top / to the bottom; rows of class +1
                    mx0[i] = OpPkMax()(mx0[i], k1 ^ 0x7f007f00u);
                    mn0[i] = OpPkMin()(mn0[i], k1 ^ 0x80008000u);
                    np[i] = __builtin_amdgcn_udot4(k1 & 0x01000100u, vsel << 8, np[i], false);
                }
            }
        }
    };
    int64_t nrows = 0;                       // rows the block has counted
    int flush = 0;
    while (tile < st.ntiles) {
        const int tn = tile + st.gx;
        if (tn < st.ntiles) load(tn, nx, nd);
        const int64_t r0 = (int64_t)tile * TR;
        if (r0 + TR <= st.M) {
#pragma unroll
            for (int u = 0; u < U; u += 2) pair(vx[u], vx[u + 1], vd[u], vd[u + 1], std::true_type(), true, true);
            nrows += TR;
        } else {
#pragma unroll
            for (int u = 0; u < U; u += 2)
                pair(vx[u], vx[u + 1], vd[u], vd[u + 1], std::false_type(), r0 + u * RPI + rsub <= last,
                     r0 + (u + 1) * RPI + rsub <= last);
            nrows += st.M - r0;
        }
        // |a pair's products| <= 2^23 (MODE 2: |f| <= 2^13, 2^29): far from 2^31 at
        // every flush
        if (MODE == 2 || ++flush == 32) {
            flush = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) { sdn[i] += sn[i]; sff[i] += sf[i]; sn[i] = sf[i] = 0; }
        }
#pragma unroll
        for (int u = 0; u < U; u++) { vx[u] = nx[u]; vd[u] = nd[u]; }
        tile = tn;
    }
#pragma unroll
    for (int i = 0; i < 4; i++) { sdn[i] += sn[i]; sff[i] += sf[i]; }
    // the halves hold the even and the odd rows: fold them, then the two maxima
    // (minima) of a channel share a register
    uint32_t kmx[4], kmn[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        kmx[i] = max(mx1[i] & 0xffff, mx1[i] >> 16) | max(mx2[i] & 0xffff, mx2[i] >> 16) << 16;
        kmn[i] = min(mn1[i] & 0xffff, mn1[i] >> 16) | min(mn2[i] & 0xffff, mn2[i] >> 16) << 16;
        mx0[i] = max(mx0[i] & 0xffff, mx0[i] >> 16);
        mn0[i] = min(mn0[i] & 0xffff, mn0[i] >> 16);
    }
    wave_fold<4, G>(sdn, OpAdd());
    if constexpr (MODE == 2) {
        wave_fold<4, G>(sff, OpAdd());
    } else {
        wave_fold<4, G>(sd, OpAdd());
        wave_fold<4, G>(z, OpAdd());
        wave_fold<4, G>(kmx, OpPkMax());
        wave_fold<4, G>(kmn, OpPkMin());
        if (zflag) {
            wave_fold<4, G>(mx0, OpPkMax());
            wave_fold<4, G>(mn0, OpPkMin());
            wave_fold<4, G>(np, OpAdd());
        }
    }
    // the wave totals of each channel, staged in the table's space
    __syncthreads();
    long long* wsn = (long long*)tab;                  // [kWaves][CS]
    uint32_t* wsd = (uint32_t*)(wsn + kWaves * CS);    // [4][kWaves][CS], with class 0 [7]
    long long* wsf = wsn + kWaves * CS;                // MODE 2: [kWaves][CS]
    if ((lane & 15) < G) {
        const int o = wv * CS + g * 4 + fold_ch<4>(lane);
        wsn[o] = sdn[0];
        if constexpr (MODE == 2) {
            wsf[o] = sff[0];
        } else {
            wsd[o] = sd[0];
            wsd[kWaves * CS + o] = z[0];
            wsd[2 * kWaves * CS + o] = kmx[0];
            wsd[3 * kWaves * CS + o] = kmn[0];
            if (zflag) {
                wsd[4 * kWaves * CS + o] = mx0[0];
                wsd[5 * kWaves * CS + o] = mn0[0];
                wsd[6 * kWaves * CS + o] = np[0];
            }
        }
    }
    __syncthreads();
    int F = 0;
    if (t < CS) {
        // [slice][block][channel of the slice]: one contiguous row per block
        const int64_t o = ((int64_t)by * st.gx + bx) * CS + t;
        long long bn = 0, bf = 0;
        int32_t bs = 0;
        uint32_t bz = 0, bx = 0, bm = ~0u, x0 = 0, m0 = 0xffff, bnp = 0;
#pragma unroll 4
        for (int v = 0; v < kWaves; v++) {
            bn += wsn[v * CS + t];
            if constexpr (MODE == 2) {
                bf += wsf[v * CS + t];
            } else {
                bs += (int32_t)wsd[v * CS + t];
                bz += wsd[(kWaves + v) * CS + t];
                bx = OpPkMax()(bx, wsd[(2 * kWaves + v) * CS + t]);
                bm = OpPkMin()(bm, wsd[(3 * kWaves + v) * CS + t]);
                if (zflag) {
                    x0 = max(x0, wsd[(4 * kWaves + v) * CS + t]);
                    m0 = min(m0, wsd[(5 * kWaves + v) * CS + t]);
                    bnp += wsd[(6 * kWaves + v) * CS + t];
                }
            }
        }
        if constexpr (MODE == 2) {
            w.p_sf[o] = bf;
            w.p_sfn[o] = bn;
        } else {
            // sum sgn = N(+1) - N(-1) from sum class = 255 N(+1) + 128 N(0)
            // (no class 0 unless the channel was flagged)
            const int n0 = sZf[t] ? (int)((bz - 255u * bnp) / 128u) : 0;
            const int np = sZf[t] ? (int)bnp : (int)(bz / 255u);
            w.p_sd[o] = bs - (int32_t)(128 * nrows);
            w.p_sdn[o] = bn;
            w.p_z[o] = 2 * np + n0 - (int32_t)nrows;
            // class -1: minimum of the key, maximum of the inverted one; class +1 the others
            const uint32_t x1 = bx & 0xffff, x2 = bx >> 16, m1 = bm & 0xffff, m2 = bm >> 16;
            const int lo0 = (m1 >> 8) == 0 ? (int)m1 : 255, hi0 = (x2 >> 8) == 0xff ? (int)(x2 & 0xff) : 0;
            const int lo2 = (m2 >> 8) == 0 ? (int)m2 : 255, hi2 = (x1 >> 8) == 0xff ? (int)(x1 & 0xff) : 0;
            const int lo1 = sZf[t] && (m0 >> 8) == 0 ? (int)m0 : 255, hi1 = sZf[t] && (x0 >> 8) == 0xff ? (int)(x0 & 0xff) : 0;
            w.p_mmA[o] = lo0 | hi0 << 8 | lo1 << 16 | hi1 << 24;
            w.p_mmB[o] = lo2 | hi2 << 8;
            if (MODE == 1 && cb + t < st.C) {
                // largest |gamma d|: |d| is largest at a class extreme
                const int lo = min(min(lo0, lo1), lo2) - 128, hi = max(max(hi0, hi1), hi2) - 128;
                const int gq = out.gamma_q[cb + t];
                F = (gq < 0 ? -gq : gq) * max(lo < 0 ? -lo : lo, hi < 0 ? -hi : hi);
            }
        }
    }
    if constexpr (MODE == 1) {
        F = block_max_nt(F, rsh);
        if (t == 0) w.pF[by * st.gx + bx] = F;
    }
}

// bracket of the exact dx (times den M^2 / 2^Ebase) for a (f, sgn) pair
__device__ __forceinline__ i128 bnb_bracket(int64_t f, int s, i128 M, i128 Sf, i128 T, i128 Z, int e_xh)
{
    i128 a = M * M * (i128)f - M * Sf;
    i128 t = T * (M * (i128)s - Z);
    return e_xh >= 0 ? a - (t << e_xh) : (a << -e_xh) - t;
}

__device__ __forceinline__ void bnb_exps_out(const Saved& sv, const BnCfg& cf, const BnbOut& o)
{
    const int32_t s_d = *o.dy_exp;
    if (s_d < -60 || s_d > 16) set_status(o.dev_status, ISEG_DEV_RANGE);
    *o.dbeta_exp = s_d;
    *o.dgamma_exp = s_d + sv.hdr[0] - (cf.k_xhat - 1);
}

// One block per channel, one thread per masked error code and one or three of
// the sgn classes: the channel's totals from the streaming blocks' partials (dbeta, dgamma), its
// bound on E1's exponent (the largest over its six per-class extremes; E2 is
// monotone and the bracket linear in the code, so the extremes bound every
// code the channel's data holds), and its dx values at that bound: Q =
// floor(B 2^S / D) with S one more than the shift of the channel's own bound,
// for the (class, code) pairs inside the channel's per-class ranges (zero
// elsewhere: the output pass never looks them up).  |Q| <= 2^k_E1 + 1 there, so
// int16 holds it; the output pass rounds Q by the gap between the largest
// bound and the channel's into the final code (half-up rounding of floor(x)
// by 2^g + 1 equals that of x).  Exact E2 (k_E2 >= 15, |gamma delta| <= 127^2 <
// 2^(k_E2-1)): E2's shift r2 is <= 0 and scales every term of the bracket and
// the exponent base by inverse powers of two, so dx is that of r2 = 0 with f =
// gamma_q delta.  Up to kChanWide channels every block is resident and latency
// bounds it: a thread per class (768) saves two of three 128-bit divisions in a
// row (backward of 1024 x 256: 20.9 -> 20.5 us).  Past that the blocks queue, and
// four waves that hold all classes repeat the totals and the bound for a third
// of the threads: 64 x 1024 26.2 -> 22.6 us, 64 x 2048 35.7 -> 27.9, 64 x 16384 162 -> 86
// (even at 512).
constexpr int64_t kChanWide = 512;
template <bool ROUND, int NT>
__global__ __launch_bounds__(NT) void k_bnb_chan(FStat st, int CS, BwdWs w, Saved sv, BnCfg cf, BnbOut o)
{
    constexpr int NW = NT / 64;
    __shared__ int32_t r_sd[NW], r_z[NW], r_lo[NW][3], r_hi[NW][3], r_cand, rsh[NW];
    __shared__ long long r_sdn[NW], r_sf[NW], r_sfn[NW];
    const int c = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6, gx = st.gx;
    const int gq = o.gamma_q[c], den = sv.den[c], hdr0 = sv.hdr[0], dye = *o.dy_exp;
    int sd = 0, z = 0;
    long long sdn = 0, sf = 0, sfn = 0;
    int lo3[3] = {255, 255, 255}, hi3[3] = {0, 0, 0};       // byte-coded extremes (empty: lo > hi)
    const int sy = c / CS, sc = c - sy * CS;                // slice, channel within it
    const int nw = min(NW, (gx + 63) >> 6);                 // waves that hold partials
    if (wv < nw) {
        for (int b = t; b < gx; b += NT) {
            const int64_t q = ((int64_t)sy * gx + b) * CS + sc;
            sd += w.p_sd[q];
            sdn += w.p_sdn[q];
            z += w.p_z[q];
            if constexpr (ROUND) { sf += w.p_sf[q]; sfn += w.p_sfn[q]; }
            mm_merge((uint32_t)w.p_mmA[q], (uint32_t)w.p_mmB[q], lo3, hi3);
        }
        for (int off = 32; off > 0; off >>= 1) {
            sd += __shfl_xor(sd, off, 64);
            z += __shfl_xor(z, off, 64);
            sdn += __shfl_xor(sdn, off, 64);
            if constexpr (ROUND) { sf += __shfl_xor(sf, off, 64); sfn += __shfl_xor(sfn, off, 64); }
#pragma unroll
            for (int k = 0; k < 3; k++) {
                lo3[k] = min(lo3[k], __shfl_xor(lo3[k], off, 64));
                hi3[k] = max(hi3[k], __shfl_xor(hi3[k], off, 64));
            }
        }
        if (lane == 0) {
            r_sd[wv] = sd; r_z[wv] = z; r_sdn[wv] = sdn; r_sf[wv] = sf; r_sfn[wv] = sfn;
#pragma unroll
            for (int k = 0; k < 3; k++) { r_lo[wv][k] = lo3[k]; r_hi[wv][k] = hi3[k]; }
        }
    }
    int r2 = 0;
    if constexpr (ROUND) r2 = bnb_r2_of(bnb_max_F(w.pF, gx * st.nsl, rsh), cf);
    __syncthreads();
    sd = r_sd[0]; z = r_z[0]; sdn = r_sdn[0]; sf = r_sf[0]; sfn = r_sfn[0];
    int mm[6];
#pragma unroll
    for (int k = 0; k < 3; k++) { lo3[k] = r_lo[0][k]; hi3[k] = r_hi[0][k]; }
    for (int v = 1; v < nw; v++) {
        sd += r_sd[v]; z += r_z[v]; sdn += r_sdn[v]; sf += r_sf[v]; sfn += r_sfn[v];
#pragma unroll
        for (int k = 0; k < 3; k++) { lo3[k] = min(lo3[k], r_lo[v][k]); hi3[k] = max(hi3[k], r_hi[v][k]); }
    }
#pragma unroll
    for (int k = 0; k < 3; k++) { mm[2 * k] = lo3[k] - 128; mm[2 * k + 1] = hi3[k] - 128; }
    if (t == 0) {
        o.dbeta[c] = sd;
        o.dgamma[c] = sdn;
    }
    const int e_xh = hdr0 - (cf.k_xhat - 1);
    const int e_sig = 2 - cf.k_sigma, e_g = 2 - cf.k_gamma;
    const int Ebase = dye + e_g + r2 - e_sig + (e_xh < 0 ? e_xh : 0);
    const i128 M = st.M;
    const i128 Dd = (i128)den * M * M;
    const i128 Sf = ROUND ? (i128)sf : (i128)gq * sd, T = ROUND ? (i128)sfn : (i128)gq * sdn, Z = z;
    auto f_of = [&](int d) {
        return ROUND ? sq_code((int64_t)gq * d, r2, cf.k_E2) : clamp_k((int64_t)gq * d, cf.k_E2);
    };
    // the six per-class candidates (threads 0..5 of wave 0), their max
    if (wv == 0) {
        int cand = kSentinelLo;
        if (t < 6) {
            const int cls = t >> 1;
            const int lo = cls == 0 ? mm[0] : (cls == 1 ? mm[2] : mm[4]);
            const int hi = cls == 0 ? mm[1] : (cls == 1 ? mm[3] : mm[5]);
            if (lo <= hi) {
                const i128 B = bnb_bracket(f_of((t & 1) ? hi : lo), cls - 1, M, Sf, T, Z, e_xh);
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
    int k = t >> 8;
    const int d = (t & 255) - 128;
    do {
        const int lo = k == 0 ? mm[0] : (k == 1 ? mm[2] : mm[4]), hi = k == 0 ? mm[1] : (k == 1 ? mm[3] : mm[5]);
        const int S = Ebase + (cf.k_E1 - 1) - bc + 1;
        int16_t q = 0;
        if (bc != kSentinelLo && d >= lo && d <= hi && d >= -127) {
            const i128 B = bnb_bracket(f_of(d), k - 1, M, Sf, T, Z, e_xh);
            i128 Q = S >= 0 ? floordiv128(B << S, Dd) : floordiv128(B, Dd << -S);
            Q = Q > 32767 ? 32767 : (Q < -32767 ? -32767 : Q);
            q = (int16_t)Q;
        }
        w.lutq[(int64_t)c * 768 + k * 256 + (t & 255)] = q;
        k += NT / 256;
    } while (NT < 768 && k < 3);
}

// Output pass: dx code = lut[c][sgn class][masked delta].  Every block first
// takes E1's exponent from the channels' bounds (block (0, 0) writes it and the
// parameter-gradient exponents) and rounds its channels' staged values into
// the byte table.  The class and the ReLU mask come from the channel's
// thresholds in packed 16-bit arithmetic, two channels per operation: sgn =
// clamp(2 q - t0 - p0 + 1, -1, 1) (t0 <= p0 <= t0 + 1 bound class 0), and the
// codes with y > 0 are those with ms q + mt >= 0.  One LDS gather per element,
// 50 KB of tables per block instead of two and 115 KB.  Bound by memory on the
// large tensors (131072 x 256 codes: 24.0 -> 23.1 us; its row loop runs at 6.1
// TB/s after 4 us of prologue), by the prologue on the small ones.
template <int G, bool PAIRED>
__global__ __launch_bounds__(1024) void k_bnb_apply(const int8_t* __restrict__ dy, const int8_t* __restrict__ x,
                                                   int8_t* __restrict__ dx, FStat st, BwdWs w, Saved sv,
                                                   BnCfg cf, BnbOut o)
{
    int bx, by;
    if (!slice_of<PAIRED>(st, bx, by)) return;
    constexpr int CS = 4 * G, RPI = kNT / G, U = kBndU, TR = U * RPI;
    constexpr int NV = (CS * 96 + kNT - 1) / kNT;
    __shared__ __attribute__((aligned(16))) int8_t lut[CS * 3 * kRowB];
    __shared__ int32_t rb[kWaves];
    const int t = threadIdx.x, g = t % G, rsub = t / G;
    const int cb = by * CS, c0 = cb + g * 4;
    const int cl = c0 < st.C ? c0 : 0;
    const int64_t last = st.M - 1;
    // staged values, bounds, thresholds and the first tile all load together
    int4 zq[NV];
    int bc[NV];
#pragma unroll
    for (int k = 0; k < NV; k++) {
        const int v = t + k * kNT, row = v / 96;
        const int c = row < CS && cb + row < st.C ? cb + row : cb;
        zq[k] = *(const int4*)(w.lutq + (int64_t)c * 768 + (v - row * 96) * 8);
        bc[k] = w.cbnd[c];
    }
    int t0[4], p0[4], mlo[4], mhi[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        t0[i] = sv.t0[cl + i]; p0[i] = sv.p0[cl + i];
        mlo[i] = sv.mlo[cl + i]; mhi[i] = sv.mhi[cl + i];
    }
    uint32_t vx[U], vd[U], nx[U], nd[U];
    auto load = [&](int tile, uint32_t* ax, uint32_t* ad) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t r = (int64_t)tile * TR + u * RPI + rsub, rr = (r < last ? r : last) * st.C + cl;
            ax[u] = *(const uint32_t*)(x + rr);
            ad[u] = *(const uint32_t*)(dy + rr);
        }
    };
    int tile = bx;
    if (tile < st.ntiles) load(tile, vx, vd);
    int bdx = kSentinelLo;
    for (int i = t; i < st.C; i += kNT) bdx = max(bdx, w.cbnd[i]);
    bdx = block_max_nt(bdx, rb);
    if (bdx == kSentinelLo) bdx = 0;
    if (bx == 0 && by == 0 && t == 0) {
        *o.dx_exp = bdx - (cf.k_E1 - 1);
        bnb_exps_out(sv, cf, o);
    }
    const short lim = (short)((1 << (cf.k_E1 - 1)) - 1);
#pragma unroll
    for (int k = 0; k < NV; k++) {                // eight values per step, two per op
        const int v = t + k * kNT, row = v >> 5, col = (v & 31) * 8;
        if (row >= CS * 3) break;
        const short sh = (short)(bc[k] == kSentinelLo ? 15 : min(bdx - bc[k], 15));
        const int qw[4] = {zq[k].x, zq[k].y, zq[k].z, zq[k].w};
        uint32_t ow[2] = {0, 0};
#pragma unroll
        for (int h = 0; h < 4; h++) {
            short2v qv = __builtin_bit_cast(short2v, qw[h]);
            qv = ((qv >> sh) + (short)1) >> (short)1;
            qv = qv > lim ? lim : qv;
            qv = qv < (short)-lim ? (short)-lim : qv;
            const uint32_t b = ((uint32_t)(uint16_t)qv.x & 0xffu) | ((uint32_t)(uint16_t)qv.y & 0xffu) << 8;
            ow[h >> 1] |= b << (16 * (h & 1));
        }
        *(uint32_t*)(lut + row * kRowB + col) = ow[0];
        *(uint32_t*)(lut + row * kRowB + col + 4) = ow[1];
    }
    // thresholds as 16-bit pairs: channels 0, 2 and channels 1, 3
    short2v tc[2], ms[2], mt[2];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        // codes with y > 0: [mlo, mhi], a prefix or a suffix of the code range,
        // everything (without ReLU too) or nothing
        const bool all = !cf.relu || (mlo[i] == -128 && mhi[i] == 127), none = mlo[i] > mhi[i];
        const int m = all || none ? 0 : (mhi[i] == 127 ? 1 : -1);
        const int a = all ? 0 : (none ? -1 : (m > 0 ? -mlo[i] : mhi[i]));
        const short vt = (short)(1 - t0[i] - p0[i]), vm = (short)m, va = (short)a;
        if (i & 2) { tc[i & 1].y = vt; ms[i & 1].y = vm; mt[i & 1].y = va; }
        else { tc[i & 1].x = vt; ms[i & 1].x = vm; mt[i & 1].x = va; }
    }
    const short base = (short)(g * 4 * 3 * kRowB + kRowB + 128);    // class 0, d = 0 of the lane's first channel
    __syncthreads();
    auto elem = [&](uint32_t wx, uint32_t wd) {
        const short2v q2[2] = {__builtin_bit_cast(short2v, wx << 8) >> (short)8, __builtin_bit_cast(short2v, wx) >> (short)8};
        const short2v d2[2] = {__builtin_bit_cast(short2v, wd << 8) >> (short)8, __builtin_bit_cast(short2v, wd) >> (short)8};
        uint32_t ix[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            short2v s = q2[h] * (short)2 + tc[h];
            s = __builtin_elementwise_max(s, (short2v)(short)-1);
            s = __builtin_elementwise_min(s, (short2v)(short)1);
            const uint32_t neg = __builtin_bit_cast(uint32_t, (short2v)((q2[h] * ms[h] + mt[h]) >> (short)15));
            const short2v dm = __builtin_bit_cast(short2v, __builtin_bit_cast(uint32_t, d2[h]) & ~neg);
            ix[h] = __builtin_bit_cast(uint32_t, (short2v)(s * (short)kRowB + (short2v)(dm + base)));
        }
        const uint32_t b0 = (uint8_t)lut[ix[0] & 0xffff], b1 = (uint8_t)lut[(ix[1] & 0xffff) + 3 * kRowB];
        const uint32_t b2 = (uint8_t)lut[(ix[0] >> 16) + 6 * kRowB], b3 = (uint8_t)lut[(ix[1] >> 16) + 9 * kRowB];
        return (b0 | b1 << 8) | (b2 | b3 << 8) << 16;
    };
    while (tile < st.ntiles) {
        const int tn = tile + st.gx;
        if (tn < st.ntiles) load(tn, nx, nd);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t r = (int64_t)tile * TR + u * RPI + rsub;
            const uint32_t v = elem(vx[u], vd[u]);
            if (r <= last && c0 < st.C) *(uint32_t*)(dx + r * st.C + c0) = v;
        }
#pragma unroll
        for (int u = 0; u < U; u++) { vx[u] = nx[u]; vd[u] = nd[u]; }
        tile = tn;
    }
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
    if (!shape_ok(M, C) || C % 4) return 0;
    return bwd_ws_bytes(C);
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
        const dim3 sg = slice_grid(st);
        with_paired<CPL * G>(st, [&](auto pc) {
            constexpr bool P = decltype(pc)::value;
            ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_STATS1, stream, (k_bnf_stats1<CPL, G, P>), sg, dim3(kNT), 0, stream, x,
                              st, w);
            ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_STATS2, stream, (k_bnf_stats2<CPL, G, P>), sg, dim3(kNT), 0, stream, x,
                              x_exp, st, w, sv, cf, dev_status);
        });
        // every block forms all C denominators, so past one block per CU a block
        // takes more channels (2048 channels: 14.2 us with 512 blocks, 7.2 with 256)
        const int grp = (int)std::min<int64_t>(kFinGrp, ceil_div64(C, 256 * kFinCh));
        const dim3 fg((unsigned)ceil_div64(C, grp * kFinCh));
        if (C <= kDenWide) {
            hipLaunchKernelGGL(k_bnf_fin2<false>, fg, dim3(kNT), 0, stream, x_exp, st, grp, w, sv, cf, gamma_q,
                               beta_q);
        } else {
            hipLaunchKernelGGL(k_bnf_den, dim3((unsigned)ceil_div64(C, kNT)), dim3(kNT), 0, stream, x_exp, st, w, sv,
                               cf);
            hipLaunchKernelGGL(k_bnf_fin2<true>, fg, dim3(kNT), 0, stream, x_exp, st, grp, w, sv, cf, gamma_q, beta_q);
        }
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
        with_paired<CPL * G>(s4, [&](auto pc) {
            constexpr bool P = decltype(pc)::value;
            if (s4.gx * s4.nsl > kMaxBlocks / 2)
                ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_APPLY, stream, (k_bnf_apply<CPL, G, 4, P>), slice_grid(s4),
                                  dim3(kNT), 0, stream, x, y_out, s4, sv, w, cf, x_exp, gamma_q, beta_q, y_exp);
            else
                ISEG_TIMED_LAUNCH(ISEG_KID_BN_FWD_APPLY, stream, (k_bnf_apply<CPL, G, 1, P>), slice_grid(s1),
                                  dim3(kNT), 0, stream, x, y_out, s1, sv, w, cf, x_exp, gamma_q, beta_q, y_exp);
        });
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
// passed to the kernels.  The workspace is written before it is read within
// a call, so nothing needs clearing between calls.
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
    if (C % 4 || (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx_out) & 3)) return ISEG_ERR_UNSUPPORTED;
    if (!ws || ws_bytes < bwd_ws_bytes(C)) return ISEG_ERR_WORKSPACE;
    BnCfg cf = to_cfg(cfg);
    Saved sv = saved_map((void*)saved, C);
    BwdWs w = bwd_ws_map(ws, C);
    // E2 = SQ(gamma delta, k_E2) is exact when |gamma delta| <= 127^2 < 2^(k_E2-1)
    const bool exact_e2 = cf.k_E2 >= 15;
    const BnbOut out{dy_exp, gamma_q, dgamma, dbeta, dgamma_exp, dbeta_exp, dx_exp, dev_status};
    auto chan = [&](auto rnd, const FStat& st, int cs) {
        constexpr bool R = decltype(rnd)::value;
        if (C <= kChanWide)
            hipLaunchKernelGGL((k_bnb_chan<R, 768>), dim3((unsigned)C), dim3(768), 0, stream, st, cs, w, sv, cf, out);
        else
            hipLaunchKernelGGL((k_bnb_chan<R, 256>), dim3((unsigned)C), dim3(256), 0, stream, st, cs, w, sv, cf, out);
    };
    auto run = [&](auto gl) {
        constexpr int G = decltype(gl)::value;
        const FStat st = make_bstat<G, kBndU>(M, C);
        const dim3 sg = slice_grid(st);
        with_paired<4 * G>(st, [&](auto pc) {
            constexpr bool P = decltype(pc)::value;
            if (exact_e2) {
                ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_STATS, stream, (k_bnb_stats<G, 0, P>), sg, dim3(kNT), 0, stream, dy,
                                  x, st, w, sv, cf, out);
                chan(std::false_type(), st, 4 * G);
            } else {
                ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_STATS, stream, (k_bnb_stats<G, 1, P>), sg, dim3(kNT), 0, stream, dy,
                                  x, st, w, sv, cf, out);
                hipLaunchKernelGGL((k_bnb_stats<G, 2, P>), sg, dim3(kNT), 0, stream, dy, x, st, w, sv, cf, out);
                chan(std::true_type(), st, 4 * G);
            }
            ISEG_TIMED_LAUNCH(ISEG_KID_BN_BWD_APPLY, stream, (k_bnb_apply<G, P>), sg, dim3(kNT), 0, stream, dy, x,
                              dx_out, st, w, sv, cf, out);
        });
    };
    if (C <= 16) run(std::integral_constant<int, 4>());
    else if (C <= 32) run(std::integral_constant<int, 8>());
    else run(std::integral_constant<int, 16>());
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
