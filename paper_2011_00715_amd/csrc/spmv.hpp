// CSR SpMV kernels for gfx950 (y = A x, the MatMult on AIJ of Sec. 4).
//
// Three families, chosen from row-length statistics at matrix creation:
//  * stream : a block owns a tile of R consecutive rows.  All 256 lanes read
//             the tile's column and value streams contiguously (non-temporal,
//             so x stays in cache), gather x, and stage the products in LDS;
//             then one lane per row sums its products in order.  Every lane is
//             busy during the loads even for 5..27-entry rows.
//  * vector : L lanes per row (L = 64 is one row per wavefront), lane-strided
//             FMA partial sums, butterfly shuffle reduction inside the group.
//  * merge  : merge-path over the sequence of (row ends + nonzeros), split into
//             equal tiles of 2048 items; each lane walks 8 items, a segmented
//             scan in LDS combines rows split across lanes, and a fix-up pass
//             adds rows split across tiles in tile order (no atomics, so the
//             result is reproducible bit for bit).
#pragma once

#include <type_traits>

#include "common.hpp"

namespace spk {

enum { kGateNone = 0, kGateInner64 = 1, kGateInner32 = 2, kGateResid = 3 };

// The state fields that decide whether a solver kernel runs.  Kernels load
// them together with their first operands (one memory round trip) and test
// them afterwards.
struct Gate {
    int32_t status, phase, mixed;
};

__device__ __forceinline__ Gate load_gate(const SysState *st)
{
    return Gate{st->status, st->phase, st->mixed};
}

// Whether a solver kernel launched inside a captured graph should run.
__device__ __forceinline__ bool gate_ok(const Gate &g, int mode)
{
    switch (mode) {
    case kGateNone: return true;
    case kGateInner64:
        return g.status == SPK_RUNNING && g.phase == kPhaseInner && g.mixed == 0;
    case kGateInner32:
        return g.status == SPK_RUNNING && g.phase == kPhaseInner && g.mixed == 1;
    case kGateResid:
        return g.status == SPK_RUNNING && g.mixed == 1 &&
               (g.phase == kPhaseResid || g.phase == kPhaseUpdate);
    }
    return false;
}

__device__ __forceinline__ bool gate_open(const SysState *st, int mode)
{
    return mode == kGateNone || gate_ok(load_gate(st), mode);
}

// sum over k = k0, k0 + L, ... below e of val[k] x[col[k]] in that order
// (FMA), four entries per round with their gathers issued together.
template <class V, int L>
__device__ __forceinline__ V strided_dot(int k0, int e, const int32_t *__restrict__ col,
                                         const V *__restrict__ val, const V *__restrict__ x)
{
    constexpr int U = 4;
    V s = V(0);
    for (int kb = k0; kb < e; kb += L * U) {
        int c[U];
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = kb + u * L < e ? kb + u * L : e - 1;
            c[u] = ld_stream(col + k);
            v[u] = ld_stream(val + k);
        }
        V xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (kb + u * L < e) s = fma(v[u], xv[u], s);
    }
    return s;
}

template <class V>
struct TileLds {
    static constexpr int kCap = kTileBytes / (int)sizeof(V);
    V prod[kCap];
    int32_t rp[kBlock + 1];
    V red[kBlock / kWave];
};

// One tile of rows [r0, r1) (r1 - r0 <= kBlock).  fn(row, value) is called
// once per row, by the lane that owns it.  Products are rounded to V and
// summed in V in column order.  Tiles with more than kCap nonzeros take the
// block-per-row path (block-wide FMA partials and a fixed-order block sum).
template <class V, class Fn>
__device__ __forceinline__ void stream_tile(int r0, int r1, const int32_t *__restrict__ rowptr,
                                            const int32_t *__restrict__ col,
                                            const V *__restrict__ val, const V *__restrict__ x,
                                            TileLds<V> &sm, Fn &&fn)
{
    const int nr = r1 - r0;
    for (int i = threadIdx.x; i <= nr; i += kBlock) sm.rp[i] = rowptr[r0 + i];
    __syncthreads();
    const int k0 = sm.rp[0];
    const int k1 = sm.rp[nr];
    if (k1 - k0 <= TileLds<V>::kCap) {
        constexpr int U = 4;
        for (int kb = k0 + (int)threadIdx.x; kb < k1; kb += kBlock * U) {
            int c[U];
            V v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb + u * kBlock;
                const int kc = k < k1 ? k : k1 - 1;
                c[u] = ld_stream(col + kc);
                v[u] = ld_stream(val + kc);
            }
            // all gathers before the first store: one latency per round
            V xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb + u * kBlock;
                if (k < k1) sm.prod[k - k0] = v[u] * xv[u];
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < nr) {
            const int a = sm.rp[threadIdx.x] - k0;
            const int e = sm.rp[threadIdx.x + 1] - k0;
            V s = V(0);
            for (int k = a; k < e; ++k) s += sm.prod[k];
            fn(r0 + (int)threadIdx.x, s);
        }
    } else {
        for (int i = 0; i < nr; ++i) {
            const int a = sm.rp[i];
            const int e = sm.rp[i + 1];
            const V s = block_sum(strided_dot<V, kBlock>(a + (int)threadIdx.x, e, col, val, x), sm.red);
            if (threadIdx.x == 0) fn(r0 + i, s);
            __syncthreads();
        }
    }
    __syncthreads();
}

// Standalone stream SpMV: grid = nblk logical blocks, each a contiguous chunk
// of tiles (XCD-aware).
template <class V>
__global__ __launch_bounds__(kBlock) void k_spmv_stream(int n, int R, int ntiles, int nblk,
                                                        const int32_t *__restrict__ rowptr,
                                                        const int32_t *__restrict__ col,
                                                        const V *__restrict__ val,
                                                        const V *__restrict__ x, V *__restrict__ y)
{
    __shared__ TileLds<V> sm;
    const int j = xcd_remap(blockIdx.x, nblk);
    int t0, t1;
    block_tiles(j, nblk, ntiles, t0, t1);
    for (int t = t0; t < t1; ++t) {
        const int r0 = t * R;
        const int r1 = min(r0 + R, n);
        stream_tile<V>(r0, r1, rowptr, col, val, x, sm, [&](int i, V s) { y[i] = s; });
    }
}

// Vector CSR: L lanes per row, rows of a block contiguous (XCD-aware chunks).
template <class V, int L>
__global__ __launch_bounds__(kBlock) void k_spmv_vector(int n, const int32_t *__restrict__ rowptr,
                                                        const int32_t *__restrict__ col,
                                                        const V *__restrict__ val,
                                                        const V *__restrict__ x, V *__restrict__ y,
                                                        const SysState *gate_st, int gate_mode)
{
    if (gate_st && !gate_open(gate_st, gate_mode)) return;
    const int nb = gridDim.x;
    const int j = xcd_remap(blockIdx.x, nb);
    constexpr int RPB = kBlock / L;  // rows per block pass
    const int64_t rows_per_blk = (((int64_t)n + nb - 1) / nb + RPB - 1) / RPB * RPB;
    const int rb = (int)min((int64_t)n, (int64_t)j * rows_per_blk);
    const int re = (int)min((int64_t)n, (int64_t)(j + 1) * rows_per_blk);
    const int lane = threadIdx.x % L;
    for (int row = rb + (int)threadIdx.x / L; row < re; row += RPB) {
        const int a = rowptr[row];
        const int e = rowptr[row + 1];
        V s = strided_dot<V, L>(a + lane, e, col, val, x);
#pragma unroll
        for (int off = L / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, L);
        if (lane == 0) y[row] = s;
    }
}

// ------------------------------------------------------------------ SELL-64
// Sliced ELLPACK with one slice of 64 consecutive rows per wavefront: lane l
// streams row (64 s + l) with coalesced loads and no LDS, no barrier and no
// cross-lane reduction.  Inside a slice of width w (its longest row) the
// entries are stored in pairs: entries 2p and 2p + 1 of lane l sit next to
// each other at element 128 p + 2 l, so one 8- or 16-byte load per lane
// fetches two entries (a wavefront load moves 512 B / 1 KB instead of
// 128 B / 512 B: fewer memory instructions per byte, 11 % faster on the
// 27-point 160^3 product), and the last entry of an odd width sits at
// 128 (w / 2) + l.  Columns are stored as offsets from the row (int16 when
// every |col - row| < 2^15, which holds for stencils), so an FP64 nonzero
// costs 10 bytes instead of CSR's 12 (FP32: 6 instead of 8); this is the
// index compression Challenge A7 points to.  Rows shorter than their slice
// are padded; padding is never multiplied (per-row length test).
//
// Shared offsets (stencil-like matrices): when the rows of every slice use
// between them at most 32 distinct column offsets, each slice stores its
// sorted offset list once (int32, one per position) and each row a 32-bit
// mask of the positions it occupies, the other positions holding zeros.
// An FP64 nonzero then costs 8 bytes plus 4 per row and 4 per slice
// position (FP32: 4), a row's entries still sit in column order and only
// masked positions are multiplied, so the sums are the same as with
// per-lane offsets.  Gathers of unmasked positions read a clamped valid
// element of x and are discarded.
//
// One value per offset (constant coefficients): where a stencil matrix has at
// most 27 distinct column offsets and every offset carries one and the same
// number in all rows that have it (Laplacians and other constant-coefficient
// stencils, and their Galerkin products), the layout is one list of offsets
// and numbers for the whole matrix and each row's mask over it.  A product
// then reads 4 bytes per row of matrix instead of 8 per entry, with the same
// operands in the same order and so the same bits.  A matrix that varies
// anywhere keeps a value per entry (stencil_slices below).
constexpr int kSell = 64;
constexpr int kSellSharedMax = 32;

// Element of entry k of lane `lane` in a slice of w entries per row,
// relative to the slice's first element.
__host__ __device__ __forceinline__ size_t sell_pos(int k, int w, int lane)
{
    return k < (w & ~1) ? (size_t)(k >> 1) * (2 * kSell) + 2 * lane + (k & 1)
                        : (size_t)(w >> 1) * (2 * kSell) + lane;
}

// Two-element vectors for the paired loads.
template <class T> struct Pair2;
template <> struct Pair2<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct Pair2<float> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct Pair2<int16_t> { typedef short type __attribute__((ext_vector_type(2))); };
template <> struct Pair2<int32_t> { typedef int type __attribute__((ext_vector_type(2))); };

struct SellView {
    const int32_t *ptr;    // element offset of each slice (nslices + 1)
    const void *col;       // int16 or int32 row-relative column offsets (per entry, or
                           // per slice position with shared offsets)
    const uint8_t *len;    // row lengths (rows of at most 255 entries), or null
    int plain;             // load policy of offsets and values, see kSellPlain64/32; kSellUniform
    const uint16_t *len16; // row lengths when some row has more than 255 entries
    const int32_t *perm;   // SELL-C-sigma: matrix row of each sorted position, or null
    const uint32_t *mask;  // shared offsets: per-row position masks (col then holds
                           // each slice's int32 offsets at element ptr[s] / 64), or null
};

// Load policy of the SELL entries.  A matrix whose stored entries fit well
// inside the 256 MB Infinity Cache is read with ordinary loads, so that it
// stays resident from one SpMV (or Krylov iteration) to the next; a larger
// one is streamed with nontemporal loads, which keep it from evicting the
// vectors that do fit.  One bit per value precision (FP64 / FP32 kernels).
constexpr int kSellPlain64 = 1, kSellPlain32 = 2;
// Third bit: one value per offset (col and val then hold the matrix's one
// list, its length in the bits from kSellWidthShift on, and ptr is null).
constexpr int kSellUniform = 4, kSellWidthShift = 8;
constexpr int kSellUniformMax = 27;  // offsets of such a list: one round of the widest walk built
// The kernels' offset type CI for it (beside int16_t and int32_t): a kernel of
// its own, because as a branch of the int32_t kernels its scalars cost those
// registers (27-point 160^3 solve 96.6 -> 100.0 ms).
struct Stencil {};

template <bool NT, class T>
__device__ __forceinline__ T sell_ld(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// What a row gathers: at(j) loads what the operand at column j is made of,
// sh(base, l) the same for column base + l with base wave-uniform, which costs
// no vector address arithmetic (scalar base, lane offset), and of(raw) forms
// the operand.  Loading and forming are apart so that a round's loads are all
// issued before the first is used: formed in the same breath, the compiler
// waited for each operand in turn (the fused kernel of the 7-point 128^3
// system 37.7 -> 29.1 us with the list in scalar
// registers).
template <class V>
struct GatherX {
    const V *__restrict__ x;
    using Raw = V;
    __device__ V at(int j) const { return x[j]; }
    __device__ V sh(int64_t base, unsigned l) const { return (x + base)[l]; }
    __device__ V of(V v) const { return v; }
};

// Row sum of lane `lane` of the slice starting at element b with slen
// entries per row; the row has rlen of them.  Entries in column order, FMA.
// UP pairs per round: the round's offset and value pairs are loaded
// together, then all 2 UP gathers of x are issued before the first FMA, so
// a round costs one memory latency.  Pairs past the slice width repeat its
// last pair and padding has offset 0, so every gather reads a valid element
// of x; only the row's own entries are multiplied.  UP is chosen per matrix
// from the widest slice (3 for a 7-point stencil: one round and the tail).
// gat gives the gathered operands: x[j] for a plain product; the fused PCG
// kernels form p = z + beta p there.
//
template <class V, class CI, int UP, bool NT, class G>
__device__ __forceinline__ V sell_row(const SellView &sv, const V *__restrict__ val, G &&gat,
                                      int32_t b, int slen, int rlen, int lane, int row)
{
    using CP = typename Pair2<CI>::type;
    using VP = typename Pair2<V>::type;
    const CP *__restrict__ cp = reinterpret_cast<const CP *>(reinterpret_cast<const CI *>(sv.col) + b) + lane;
    const VP *__restrict__ vp = reinterpret_cast<const VP *>(val + b) + lane;
    const int np = slen >> 1;
    // the odd last entry is loaded first and gathered with the first round,
    // so an odd width costs no extra memory round trip; it is added last
    const bool odd = slen & 1;
    CI ct = CI(0);
    using Raw = typename std::remove_reference_t<G>::Raw;
    V at = V(0);
    Raw xt{};
    if (odd) {
        const size_t t = (size_t)b + (size_t)np * (2 * kSell) + lane;
        ct = sell_ld<NT>(reinterpret_cast<const CI *>(sv.col) + t);
        at = sell_ld<NT>(val + t);
    }
    V acc = V(0);
    for (int p0 = 0; p0 < np; p0 += UP) {
        CP c[UP];
        VP a[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            const int p = p0 + u < np ? p0 + u : np - 1;
            c[u] = sell_ld<NT>(cp + (size_t)p * kSell);
            a[u] = sell_ld<NT>(vp + (size_t)p * kSell);
        }
        Raw xv[2 * UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            xv[2 * u] = gat.at(row + (int)c[u].x);
            xv[2 * u + 1] = gat.at(row + (int)c[u].y);
        }
        if (p0 == 0 && odd) xt = gat.at(row + (int)ct);
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            const int k = 2 * (p0 + u);
            if (p0 + u < np) {
                if (k < rlen) acc = fma(a[u].x, gat.of(xv[2 * u]), acc);
                if (k + 1 < rlen) acc = fma(a[u].y, gat.of(xv[2 * u + 1]), acc);
            }
        }
    }
    if (odd) {
        if (np == 0) xt = gat.at(row + (int)ct);
        if (slen - 1 < rlen) acc = fma(at, gat.of(xt), acc);
    }
    return acc;
}


// Slices s, s + stride, ... below ceil(n/64), one per wavefront at a time;
// fn(row, y, own) is called by the lane that owns row (< n), own being what
// pre(row) loaded of the row's own operands (which no other row's fn
// writes).  Callers pass
// s = 4 * (physical block) + wave and stride = 4 * (blocks), so the slices in
// flight at any moment are adjacent in memory (one DRAM stream front rather
// than one per block).  The first slice's header is loaded before go() is
// asked whether to run (go holds no barrier: waves may own different counts).
template <class V, class CI, int U, bool NT, class G, class Go, class Pre, class Fn>
__device__ __forceinline__ void sell_slices_run(int n, int s, int stride, const SellView &sv,
                                                const V *__restrict__ val, G &&gat, Go &&go, Pre &&pre, Fn &&fn)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int ns = (n + kSell - 1) / kSell;
    // position j = 64 s + lane of the layout holds matrix row perm[j]
    // (SELL-C-sigma) or row j; its length is in len or len16
    auto head = [&](int j, int &rlen, int &row) {
        rlen = j < n ? (sv.len16 ? (int)sv.len16[j] : (int)sv.len[j]) : 0;
        row = j < n && sv.perm ? sv.perm[j] : j;
    };
    int32_t b = 0, e = 0;
    int rlen = 0, row = 0;
    if (s < ns) {
        b = sv.ptr[s];
        e = sv.ptr[s + 1];
        head(s * kSell + lane, rlen, row);
    }
    if (!go()) return;
    while (s < ns) {
        const int slen = (e - b) / kSell;
        if (s * kSell + lane < n) {
            const V y = sell_row<V, CI, U, NT>(sv, val, gat, b, slen, rlen, lane, row);
            fn(row, y, pre(row));
        }
        s += stride;
        if (s >= ns) break;
        b = sv.ptr[s];
        e = sv.ptr[s + 1];
        head(s * kSell + lane, rlen, row);
    }
}

// Memory that no kernel writes while this one runs, for scalar loads.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_constant(const T *p)
{
    return (const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// The same walk for offsets shared per slice: list and slice pointers are read
// by scalar loads, a row's mask says which positions it uses, and inside the
// matrix a gather is a scalar base and the lane, with no vector arithmetic per
// entry (elsewhere its column is clamped into [0, n) for the positions that a
// row does not use).  The general walk read the list into vector registers, one
// more round trip before the gathers, and spent about eight vector instructions
// an entry on columns: wide product of the 27-point 160^3 system 189 -> 175 us
// (0.94 GB, all 27 entries of a row in flight; 183, 200, 190 us with 14, 18, 10
// of them, 239 with the registers held to four waves).
template <class V, int UP, bool NT, class G, class Go, class Pre, class Fn>
__device__ __forceinline__ void shared_slices(int n, int s0, int stride, const SellView &sv,
                                              const V *__restrict__ val, G &&gat, Go &&go, Pre &&pre, Fn &&fn)
{
    using VP = typename Pair2<V>::type;
    using Raw = typename std::remove_reference_t<G>::Raw;
    const unsigned lane = threadIdx.x & (kWave - 1);
    const int ns = (n + kSell - 1) / kSell;
    const auto *ptr = as_constant(sv.ptr);
    const auto *lists = as_constant(reinterpret_cast<const int32_t *>(sv.col));
    auto masks = [&](int t) -> uint32_t {
        const int j = t * kSell + (int)lane;
        return j < n ? sv.mask[j] : 0u;
    };
    int s = __builtin_amdgcn_readfirstlane(s0);
    int32_t b = 0, e = 0;
    uint32_t m = 0;
    if (s < ns) {
        b = ptr[s];
        e = ptr[s + 1];
        m = masks(s);
    }
    if (!go()) return;
    while (s < ns) {
        const int r0 = s * kSell, row = r0 + (int)lane;
        const int slen = (e - b) / kSell, np = slen >> 1;
        const bool odd = slen & 1;
        const auto *o = lists + b / kSell;
        const VP *__restrict__ vp = reinterpret_cast<const VP *>(val + b) + lane;
        auto gather = [&](int off) -> Raw { return gat.at(min(max(row + off, 0), n - 1)); };
        // the odd last entry is gathered with the first round and added last
        V at = V(0);
        Raw xt{};
        int ot = 0;
        if (odd) {
            ot = o[slen - 1];
            at = sell_ld<NT>(val + b + (size_t)np * (2 * kSell) + lane);
        }
        V acc = V(0);
        for (int p0 = 0; p0 < np; p0 += UP) {
            VP a[UP];
            int c[2 * UP];
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                const int p = min(p0 + u, np - 1);
                c[2 * u] = o[2 * p];
                c[2 * u + 1] = o[2 * p + 1];
                a[u] = sell_ld<NT>(vp + (size_t)p * kSell);
            }
            // the list ascends; asked of the round's own entries, so that they and
            // the values are on their way before the first is waited for
            const int last = p0 == 0 && odd ? ot : c[2 * UP - 1];
            const bool in = r0 + c[0] >= 0 && (int64_t)r0 + (kSell - 1) + last < n;
            Raw xv[2 * UP];
            if (in) {
#pragma unroll
                for (int u = 0; u < 2 * UP; ++u) xv[u] = gat.sh((int64_t)r0 + c[u], lane);
                if (p0 == 0 && odd) xt = gat.sh((int64_t)r0 + ot, lane);
            } else {
#pragma unroll
                for (int u = 0; u < 2 * UP; ++u) xv[u] = gather(c[u]);
                if (p0 == 0 && odd) xt = gather(ot);
            }
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                const int k = 2 * (p0 + u);
                if (p0 + u < np) {
                    if ((m >> k) & 1u) acc = fma(a[u].x, gat.of(xv[2 * u]), acc);
                    if ((m >> (k + 1)) & 1u) acc = fma(a[u].y, gat.of(xv[2 * u + 1]), acc);
                }
            }
        }
        if (odd) {
            if (np == 0) xt = gather(ot);
            if ((m >> (slen - 1)) & 1u) acc = fma(at, gat.of(xt), acc);
        }
        if (row < n) fn(row, acc, pre(row));
        s += stride;
        if (s >= ns) break;
        b = ptr[s];
        e = ptr[s + 1];
        m = masks(s);
    }
}

// The same walk for a matrix of one value per offset.  With 4 bytes of matrix
// per row the walk is bound by its instructions and its round trips, no
// longer by HBM: so a slice whose rows' offsets all stay inside [0, n), known
// from the list's ends alone, gathers at scalar bases without clamping (the
// lane is the only vector part of an address), all of a slice's gathers and
// its rows' own operands are issued together, and the next slice's masks
// before them.  Entries a row does not have are loaded (in the other slices
// at columns clamped into the matrix) and not multiplied.  The list is never
// empty.  7-point 128^3, against the walk of a value per entry: an FP64 PCG
// iteration 61 -> 46.5 us (F 43.4 -> 29.1), the FP32 one 40.2 -> 30.3, two
// smoothing steps 39.6 -> 20.0, the product 25.9 -> 15; with the wavefront sums
// of lane swaps and one D^-1 for the matrix 41 us (F 28.3), 27.5 and 13.4.
template <class V, int U, class G, class Go, class Pre, class Fn>
__device__ __forceinline__ void stencil_slices(int n, int s0, int stride, const SellView &sv,
                                               const V *__restrict__ val, G &&gat, Go &&go, Pre &&pre, Fn &&fn)
{
    constexpr int W = 2 * U + 1;  // at least the list's length
    const unsigned lane = threadIdx.x & (kWave - 1);
    const int ns = (n + kSell - 1) / kSell;
    const int w = sv.plain >> kSellWidthShift;
    // constant for the kernel's life: read by scalar loads
    const auto *ou = as_constant(reinterpret_cast<const int32_t *>(sv.col));
    const auto *uv = as_constant(val);
    const int64_t lo = ou[0], hi = ou[w - 1];
    // positions past the list repeat its last one; no mask has their bits.  A
    // short list stays in registers; a long one is read from the scalar cache
    // for each slice (kept across the loop it spills).
    constexpr bool kKeep = W <= 9;
    int ok[kKeep ? W : 1];
    V vk[kKeep ? W : 1];
    if constexpr (kKeep) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
            ok[k] = ou[min(k, w - 1)];
            vk[k] = uv[min(k, w - 1)];
        }
    }
    int s = __builtin_amdgcn_readfirstlane(s0);
    auto masks = [&](int t) -> uint32_t {
        const int j = t * kSell + (int)lane;
        return j < n ? sv.mask[j] : 0u;
    };
    uint32_t next = s < ns ? masks(s) : 0u;
    if (!go()) return;
    while (s < ns) {
        const int r0 = s * kSell, row = r0 + (int)lane;
        const uint32_t m = next;
        s += stride;
        if (s < ns) next = masks(s);
        const auto *o = ou;
        const auto *v = uv;
        if constexpr (!kKeep) asm volatile("" : "+s"(o), "+s"(v));
        auto off = [&](int k) -> int {
            if constexpr (kKeep) return ok[k];
            else return o[min(k, w - 1)];
        };
        auto value = [&](int k) -> V {
            if constexpr (kKeep) return vk[k];
            else return v[min(k, w - 1)];
        };
        // before the gathers, and without a branch, which would keep them waiting
        const auto own = pre(min(row, n - 1));
        typename std::remove_reference_t<G>::Raw xv[W];
        if (r0 + lo >= 0 && r0 + (kSell - 1) + hi < n) {
#pragma unroll
            for (int k = 0; k < W; ++k) xv[k] = gat.sh((int64_t)r0 + off(k), lane);
        } else {
#pragma unroll
            for (int k = 0; k < W; ++k) xv[k] = gat.at(min(max(row + off(k), 0), n - 1));
        }
        V acc = V(0);
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const V t = fma(value(k), gat.of(xv[k]), acc);
            acc = (m >> k) & 1u ? t : acc;
        }
        if (row < n) fn(row, acc, own);
    }
}

// The load policy is chosen here, around the whole slice loop, so that the
// two variants stay separate code (a branch inside the round lets the
// compiler merge the loads and drop the nontemporal hint).
template <class V, class CI, int U, class G, class Go, class Pre, class Fn>
__device__ __forceinline__ void sell_slices_g(int n, int s, int stride, const SellView &sv,
                                              const V *__restrict__ val, G &&gat, Go &&go, Pre &&pre, Fn &&fn)
{
    const bool plain = sv.plain & (sizeof(V) == 4 ? kSellPlain32 : kSellPlain64);
    if constexpr (std::is_same<CI, Stencil>::value) {
        stencil_slices<V, U>(n, s, stride, sv, val, gat, go, pre, fn);
    } else {
        if constexpr (std::is_same<CI, int32_t>::value) {
            if (sv.mask) {
                if (plain) shared_slices<V, U, false>(n, s, stride, sv, val, gat, go, pre, fn);
                else shared_slices<V, U, true>(n, s, stride, sv, val, gat, go, pre, fn);
                return;
            }
        }
        if (plain) sell_slices_run<V, CI, U, false>(n, s, stride, sv, val, gat, go, pre, fn);
        else sell_slices_run<V, CI, U, true>(n, s, stride, sv, val, gat, go, pre, fn);
    }
}

// The plain product: the gathered operand is x.
template <class V, class CI, int U, class Go, class Pre, class Fn>
__device__ __forceinline__ void sell_slices(int n, int s, int stride, const SellView &sv,
                                            const V *__restrict__ val, const V *__restrict__ x,
                                            Go &&go, Pre &&pre, Fn &&fn)
{
    sell_slices_g<V, CI, U>(n, s, stride, sv, val, GatherX<V>{x}, go, pre, fn);
}

// Own operands of rows whose epilogue needs none.
struct NoOwn {
    __device__ int operator()(int) const { return 0; }
};

// Standalone SELL SpMV; the grid has up to one wavefront per slice.
template <class V, class CI, int U>
__global__ __launch_bounds__(kBlock) void k_spmv_sell(int n, SellView sv, const V *__restrict__ val,
                                                      const V *__restrict__ x, V *__restrict__ y)
{
    sell_slices<V, CI, U>(n, blockIdx.x * (kBlock / kWave) + (int)threadIdx.x / kWave,
                          gridDim.x * (kBlock / kWave), sv, val, x, [] { return true; }, NoOwn{},
                          [&](int i, V s, int) { y[i] = s; });
}

// Calls f with a value of the kernels' offset type for a layout: cw bytes per
// offset, and its policy and layout bits.
template <class F>
inline void with_sell_ci(int cw, int plain, F &&f)
{
    if (plain & kSellUniform) f(Stencil{});
    else if (cw == 2) f(int16_t{});
    else f(int32_t{});
}

// Pairs per round UP the SELL kernels are built for, and the launch
// helper: calls f(std::integral_constant<int, UP>) for the handle's UP.
template <class F>
inline void with_sell_u(int u, F &&f)
{
    switch (u) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 13: f(std::integral_constant<int, 13>{}); break;
    default: f(std::integral_constant<int, 7>{}); break;
    }
}

// UP for a matrix whose widest slice has w entries per row: the fewest
// rounds, then the fewest repeated pairs, among the built values (2 below 3
// pairs).  One round beats register room: the 27-point rows (13 pairs) in
// one round of 13 (FP64 140 VGPRs, 3 wavefronts per SIMD) took the 160^3
// PCG product from 225.7 to 216.3 us against two rounds of 7 (95 VGPRs,
// 5 per SIMD); rounds of 5 and 4 (6 and 7 per SIMD) took 231.7 and 233.1.
inline int pick_sell_u(int w)
{
    const int np = w >> 1;
    if (np <= 2) return 2;
    constexpr int kBuilt[] = {3, 4, 5, 6, 7, 9, 13};
    int best = 13, rounds = 1 << 30, waste = 1 << 30;
    for (const int u : kBuilt) {
        const int r = (np + u - 1) / u, wst = r * u - np;
        if (r < rounds || (r == rounds && wst < waste)) { best = u; rounds = r; waste = wst; }
    }
    return best;
}

// Layout fill: one lane per layout position j writes the entries of its
// matrix row (perm[j], or j) and the slice padding; the row's length goes to
// slen (one byte) or, for rows longer than 255 entries, to slen16.
template <class CI>
__global__ void k_sell_fill(int n, const int32_t *__restrict__ rowptr,
                            const int32_t *__restrict__ col, const double *__restrict__ val,
                            const int32_t *__restrict__ sptr, const int32_t *__restrict__ perm,
                            CI *__restrict__ scol, double *__restrict__ sval, uint8_t *__restrict__ slen,
                            uint16_t *__restrict__ slen16)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int s = i / kSell, lane = i % kSell;
        const int r = perm ? perm[i] : i;
        const int b = sptr[s];
        const int len = (sptr[s + 1] - b) / kSell;
        const int a = rowptr[r], e = rowptr[r + 1];
        if (slen16) slen16[i] = (uint16_t)(e - a);
        else slen[i] = (uint8_t)(e - a);
        for (int j = 0; j < len; ++j) {
            const size_t d = (size_t)b + sell_pos(j, len, lane);
            const bool real = a + j < e;
            scol[d] = real ? (CI)(col[a + j] - r) : (CI)0;
            sval[d] = real ? val[a + j] : 0.0;
        }
    }
}

// ------------------------------------------------------------------ merge path
// Split point of diagonal d on the merge of row ends (rowptr[i+1]) with
// nonzero indices: (i, d - i) with i the number of completed rows.
static __global__ void k_merge_partition(int n, int nnz, const int32_t *__restrict__ rowptr, int ntiles, int per,
                                  int32_t *__restrict__ tile_row, int32_t *__restrict__ tile_k)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t > ntiles) return;
    const int64_t total = (int64_t)n + nnz;
    const int64_t d64 = min((int64_t)t * per, total);
    const int d = (int)d64;
    int lo = d > nnz ? d - nnz : 0;
    int hi = d < n ? d : n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (rowptr[mid + 1] <= d - mid - 1) lo = mid + 1; else hi = mid;
    }
    tile_row[t] = lo;
    tile_k[t] = d - lo;
}

template <class V>
struct MergeLds {
    V prod[kMergeItems];
    int32_t rend[kMergeItems + 1];
    V sv[2][kBlock];
    int32_t sk[kBlock];
};

// Merge-path tile t, computed by one block.  Rows that end inside the tile
// are written (complete rows directly, rows split across lanes after a
// segmented scan); the partial of the row still open at the tile end goes to
// carry_{row,val}.
template <class V>
__device__ __forceinline__ void merge_tile(int t, int n, const int32_t *__restrict__ rowptr,
                                           const int32_t *__restrict__ col, const V *__restrict__ val,
                                           const V *__restrict__ x, V *__restrict__ y,
                                           const int32_t *__restrict__ tile_row,
                                           const int32_t *__restrict__ tile_k, int32_t *__restrict__ carry_row,
                                           V *__restrict__ carry_val, MergeLds<V> &sm)
{
    const int i0 = tile_row[t], k0 = tile_k[t];
    const int i1 = tile_row[t + 1], k1 = tile_k[t + 1];
    const int nrows = i1 - i0;   // row ends inside the tile
    const int nk = k1 - k0;      // nonzeros inside the tile
    for (int r = threadIdx.x; r <= nrows; r += kBlock)
        sm.rend[r] = (i0 + r < n) ? rowptr[i0 + r + 1] - k0 : nk;
    {
        constexpr int U = 4;
        for (int kb = k0 + (int)threadIdx.x; kb < k1; kb += kBlock * U) {
            int c[U];
            V v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb + u * kBlock;
                const int kc = k < k1 ? k : k1 - 1;
                c[u] = ld_stream(col + kc);
                v[u] = ld_stream(val + kc);
            }
            V xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = kb + u * kBlock;
                if (k < k1) sm.prod[k - k0] = v[u] * xv[u];
            }
        }
    }
    __syncthreads();
    // this lane's start on the tile-local merge path
    const int total = nrows + nk;
    const int dd = min((int)threadIdx.x * kMergeIpt, total);
    int lo = dd > nk ? dd - nk : 0;
    int hi = dd < nrows ? dd : nrows;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sm.rend[mid] <= dd - mid - 1) lo = mid + 1; else hi = mid;
    }
    int r = lo;
    int kk = dd - lo;
    const int items = min(kMergeIpt, total - dd);
    V acc = V(0);
    V head = V(0);
    int head_row = -1;
    for (int it = 0; it < items; ++it) {
        if (kk < nk && kk < sm.rend[r]) {
            acc += sm.prod[kk];
            ++kk;
        } else {
            if (r >= nrows || i0 + r >= n) break;  // never taken on a consistent path
            if (head_row < 0) { head = acc; head_row = r; }
            else y[i0 + r] = acc;
            acc = V(0);
            ++r;
        }
    }
    // inclusive segmented scan of (carry row, carry value) over the lanes
    sm.sk[threadIdx.x] = r;
    sm.sv[0][threadIdx.x] = acc;
    __syncthreads();
    int cur = 0;
#pragma unroll
    for (int off = 1; off < kBlock; off <<= 1) {
        V v = sm.sv[cur][threadIdx.x];
        if ((int)threadIdx.x >= off && sm.sk[threadIdx.x - off] == r)
            v = sm.sv[cur][threadIdx.x - off] + v;
        sm.sv[cur ^ 1][threadIdx.x] = v;
        cur ^= 1;
        __syncthreads();
    }
    if (head_row >= 0) {
        const V cin = threadIdx.x > 0 ? sm.sv[cur][threadIdx.x - 1] : V(0);
        y[i0 + head_row] = cin + head;
    }
    if (threadIdx.x == kBlock - 1) {
        carry_row[t] = i0 + r;
        carry_val[t] = sm.sv[cur][threadIdx.x];
    }
}

// One merge-path tile per block.
template <class V>
__global__ __launch_bounds__(kBlock) void k_spmv_merge(int n, int nnz,
                                                       const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ col,
                                                       const V *__restrict__ val,
                                                       const V *__restrict__ x, V *__restrict__ y,
                                                       const int32_t *__restrict__ tile_row,
                                                       const int32_t *__restrict__ tile_k,
                                                       int32_t *__restrict__ carry_row,
                                                       V *__restrict__ carry_val,
                                                       const SysState *gate_st, int gate_mode)
{
    if (gate_st && !gate_open(gate_st, gate_mode)) return;
    (void)nnz;
    __shared__ MergeLds<V> sm;
    merge_tile<V>(blockIdx.x, n, rowptr, col, val, x, y, tile_row, tile_k, carry_row, carry_val, sm);
}

// Adds the carries of rows that span tiles, in tile order; one lane per chain.
template <class V>
__global__ void k_merge_fixup(int n, int ntiles, const int32_t *__restrict__ carry_row,
                              const V *__restrict__ carry_val, V *__restrict__ y,
                              const SysState *gate_st, int gate_mode)
{
    if (gate_st && !gate_open(gate_st, gate_mode)) return;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    const int c = carry_row[t];
    if (c >= n) return;
    if (t > 0 && carry_row[t - 1] == c) return;
    V s = carry_val[t];
    // the row goes on while the carries name it; loaded some at a time, since
    // one load a tile is a chain of round trips (merge-path product of 1 M rows
    // of 9 and one that is full: 197 -> 145 us).  Most rows do not: the next
    // tile's alone says so (7-point 61 x 47 x 53: 14.0 -> 13.5 us)
    constexpr int P = 8;
    bool on = t + 1 < ntiles && carry_row[t + 1] == c;
    for (int u0 = t + 1; on && u0 < ntiles; u0 += P) {
        int32_t r[P];
        V v[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            r[k] = carry_row[min(u0 + k, ntiles - 1)];
            v[k] = carry_val[min(u0 + k, ntiles - 1)];
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            on = on && u0 + k < ntiles && r[k] == c;
            if (on) s += v[k];
        }
    }
    y[c] += s;
}

}  // namespace spk
