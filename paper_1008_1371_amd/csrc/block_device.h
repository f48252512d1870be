// Device-side building blocks of the block-column path, shared by the
// per-launch kernels of single and grouped solves (block_kernels.hip) and the
// persistent batched kernel (batch_persist.hip): the MFMA wrappers, the Gram
// of one block pair, the two inner solves of one block pair and the update
// of its columns.  Each takes its block pair index and its LDS explicitly, so
// a caller can run any of them for any pair and share one LDS area between
// them.
#pragma once

#include "internal.h"

namespace hsvd {
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// 16x16x4 MFMA per storage type.  Operand A element (i, k) and operand B
// element (k, j) sit in lane i + 16k resp. j + 16k for both types; the
// accumulator layouts differ (checked on the device):
//   v_mfma_f64_16x16x4f64: register v of lane l holds D(l/16 + 4v, l%16)
//   v_mfma_f32_16x16x4f32: register v of lane l holds D(4(l/16) + v, l%16)
template <typename T>
struct MF;
template <>
struct MF<double> {
    typedef d4 acc;
    static __device__ __forceinline__ acc zero() { return d4{0.0, 0.0, 0.0, 0.0}; }
    static __device__ __forceinline__ acc mma(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};
template <>
struct MF<float> {
    typedef f4 acc;
    static __device__ __forceinline__ acc zero() { return f4{0.f, 0.f, 0.f, 0.f}; }
    static __device__ __forceinline__ acc mma(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

constexpr int kB = 32;        // block width b
constexpr int kB2 = 2 * kB;   // columns of a block pair
constexpr int kLd = kB2 + 1;  // LDS row stride (doubles)
constexpr int kMaxSplits = 32; // row splits of the Gram (the host keeps splits <= this)

// Points the argument block at problem blockIdx.z of a batched group; false
// when that problem has already converged.
template <typename T>
__device__ __forceinline__ bool bind_problem(BlockArgsT<T> &a)
{
    if (a.nprob <= 1 && !a.done) return true;
    const int z = blockIdx.z;
    if (a.done && a.done[z]) return false;
    const size_t mat = (size_t)a.ldg * a.r;
    const int pairs = a.nb / 2;
    a.G += z * mat;
    if (a.V) a.V += z * mat;
    a.rho += (size_t)z * a.r;
    a.partial += (size_t)z * pairs * a.splits * (kB2 * kB2);
    a.W += (size_t)z * pairs * (kB2 * kB2);
    a.active += (size_t)z * pairs;
    a.C += (size_t)z * pairs;
    a.nrot += (size_t)z * pairs;
    a.nskip += (size_t)z * pairs;
    a.nact += (size_t)z * pairs;
    a.ntc += (size_t)z * pairs;
    a.maxt += (size_t)z * pairs;
    a.ctl += z;
    if (a.pvec) a.p = a.pvec[z];
    if (a.tolvec) a.tol = a.tolvec[z];
    if (a.tthvec) a.tthresh = a.tthvec[z];
    return true;
}

template <typename T>
__device__ __forceinline__ int2 outer_pair(const BlockArgsT<T> &a, int k)
{
    if (a.ordering == HSVD_ORD_MODMOD) {
        const int4 s = a.S_in[k];
        return make_int2(s.z, s.w);
    }
    return roundrobin_pair(k, a.nb, a.step);
}

__device__ __forceinline__ int local_pos(int x, int I, int J)
{
    return x < kB ? I * kB + x : J * kB + (x - kB);
}


// ---------------------------------------------------------------------------
// Gram: partial[k][split] = G_P(rows of split)^T G_P(rows of split)
// ---------------------------------------------------------------------------
// The Gram matrix is symmetric: only the 10 upper-triangular 16 x 16 tiles
// (xt <= yt) of the 4 x 4 tiling are formed; readers take entry
// (min(x, y), max(x, y)).  An MFMA slice contracts 4 rows; operand A(i, k)
// sits in lane i + 16k, operand B(k, j) in lane j + 16k, so with lane
// (i, k) holding G(row_k, column 16t + i) the same register is the A operand
// of column tile t and the B operand of tile t, and a wave issues all 10
// products from its 4 tile registers.  The rows of a slice need not be
// consecutive: lane (i, k) loads 16 consecutive bytes of column 16t + i
// (V = 16 / sizeof(T) rows) at row offset V k, and element e of that load
// serves slice e.  One load per tile (FP32) or two (FP64, rows + 4V) make a
// chunk of 16 rows; lanes of one load instruction read 64 contiguous bytes
// per column.  No LDS staging: the loads are the MFMA operands.  Wave w
// takes every fourth chunk of the split; the four waves' tiles are summed in
// wave order at the end.
constexpr int kGramTiles = 10;
static __constant__ int kGramTX[kGramTiles] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};
static __constant__ int kGramTY[kGramTiles] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};

// The Gram of block pair k over the rows of `split`, by 256 threads (tid among
// them); red: kGramRed elements of LDS.  kGramBarriers workgroup barriers.
//
// The functions of this file that take a tid work with NT threads of a
// workgroup that may hold several such groups, each with a block pair of its
// own: every group passes the same barriers.
constexpr int kGramBarriers = 3;
constexpr int kGramRed = 3 * (kGramTiles / 2) * 256;
template <typename T>
__device__ __forceinline__ void gram_pair(const BlockArgsT<T> &a, int k, int split, T *red, int tid)
{
    constexpr int kV = 16 / (int)sizeof(T);  // rows per 16-byte load
    // loads per tile and chunk: FP32 one (16 rows), FP64 two (8 rows each)
    constexpr int NH = sizeof(T) == 4 ? 1 : 2;
    constexpr int kRC = 4 * NH * kV;  // rows per chunk
    typedef T vec __attribute__((ext_vector_type(kV)));
    constexpr int kHalf = kGramTiles / 2;
    const int2 IJ = outer_pair(a, k);
    const int lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int row_begin = split * a.rows_per_split;
    const int row_end = min(a.ldg, row_begin + a.rows_per_split);
    const int nchunk = (row_end - row_begin) / kRC;
    // byte offsets of this lane's first row in its 4 columns, 32-bit from the
    // uniform base (r, ldg <= 16448: below 2^32 bytes)
    const char *__restrict__ G = reinterpret_cast<const char *>(a.G);
    unsigned off[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
        off[t] = ((unsigned)a.rho[local_pos(16 * t + lr, IJ.x, IJ.y)] * (unsigned)a.ldg +
                  (unsigned)(row_begin + kV * lk)) * (unsigned)sizeof(T);
    typename MF<T>::acc acc[kGramTiles];
#pragma unroll
    for (int q = 0; q < kGramTiles; ++q) acc[q] = MF<T>::zero();
    // no prefetch: the registers go to occupancy instead (measured faster)
    for (int c = wave; c < nchunk; c += 4) {
        vec cur[4][NH];
        const unsigned rb = (unsigned)(c * kRC) * (unsigned)sizeof(T);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < NH; ++h)
                cur[t][h] = *reinterpret_cast<const vec *>(G + (off[t] + rb + (unsigned)(h * 4 * kV) * sizeof(T)));
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < kV; ++e) {
                const T x0 = cur[0][h][e], x1 = cur[1][h][e], x2 = cur[2][h][e], x3 = cur[3][h][e];
                acc[0] = MF<T>::mma(x0, x0, acc[0]);
                acc[1] = MF<T>::mma(x0, x1, acc[1]);
                acc[2] = MF<T>::mma(x0, x2, acc[2]);
                acc[3] = MF<T>::mma(x0, x3, acc[3]);
                acc[4] = MF<T>::mma(x1, x1, acc[4]);
                acc[5] = MF<T>::mma(x1, x2, acc[5]);
                acc[6] = MF<T>::mma(x1, x3, acc[6]);
                acc[7] = MF<T>::mma(x2, x2, acc[7]);
                acc[8] = MF<T>::mma(x2, x3, acc[8]);
                acc[9] = MF<T>::mma(x3, x3, acc[9]);
            }
    }
    // sum over the waves in wave order, five tiles at a time (waves 1..3
    // deposit, wave 0 adds and stores)
    T *out = a.partial + ((size_t)k * a.splits + split) * (kB2 * kB2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h) __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int j = 0; j < kHalf; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[((wave - 1) * kHalf + j) * 256 + v * 64 + lane] = acc[h * kHalf + j][v];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int j = 0; j < kHalf; ++j) {
                const int q = h * kHalf + j;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    T sum = acc[q][v];
#pragma unroll
                    for (int w = 0; w < 3; ++w) sum += red[(w * kHalf + j) * 256 + v * 64 + lane];
                    const int x = kGramTX[q] * 16 + MF<T>::row(lane, v);
                    const int y = kGramTY[q] * 16 + lr;
                    out[x * kB2 + y] = sum;
                }
            }
        }
    }
}

// A_P = sum of the partial Grams in split order, put(x, y, A_P(x, y)), by NT
// threads.  Only the 10 upper-triangular 16 x 16 tiles hold data: work item i
// sums the entries (x, y), (x, y + 1) of tile i / 128 of every split with
// vector loads.
template <typename T, int NT, typename Put>
__device__ __forceinline__ void stage_gram(const BlockArgsT<T> &a, int k, int tid, Put put)
{
    constexpr int kItems = kGramTiles * 128;
    typedef T v2 __attribute__((ext_vector_type(2)));
    constexpr int kChunk = 8;
#pragma unroll
    for (int q = 0; q < (kItems + NT - 1) / NT; ++q) {
        const int item = tid + NT * q;
        if (kItems % NT == 0 || item < kItems) {
            const int tile = item >> 7, x = kGramTX[tile] * 16 + ((item >> 3) & 15), y = kGramTY[tile] * 16 + (item & 7) * 2;
            const T *P = a.partial + (size_t)k * a.splits * (kB2 * kB2) + x * kB2 + y;
            double g0 = 0.0, g1 = 0.0;
            for (int base = 0; base < a.splits; base += kChunk) {
                v2 v[kChunk];
#pragma unroll
                for (int c = 0; c < kChunk; ++c)
                    v[c] = base + c < a.splits
                               ? *reinterpret_cast<const v2 *>(P + (size_t)(base + c) * (kB2 * kB2))
                               : v2{0, 0};
#pragma unroll
                for (int c = 0; c < kChunk; ++c)
                    if (base + c < a.splits) {
                        const bool first = base + c == 0;
                        g0 = first ? (double)v[c][0] : g0 + (double)v[c][0];
                        g1 = first ? (double)v[c][1] : g1 + (double)v[c][1];
                    }
            }
            put(x, y, g0);
            put(x, y + 1, g1);
        }
    }
}

// The sweep's counters of a slot, read ahead of an inner solve and written
// after it (one thread).
struct SweepSoFar {
    double maxt = 0.0;
    int C = 0;
    unsigned rot = 0, skip = 0, act = 0, tc = 0;
    template <typename T>
    __device__ __forceinline__ void read(const BlockArgsT<T> &a, int k)
    {
        maxt = a.maxt[k];
        C = a.C[k];
        rot = a.nrot[k];
        skip = a.nskip[k];
        act = a.nact[k];
        tc = a.ntc[k];
    }
    template <typename T>
    __device__ __forceinline__ void write(const BlockArgsT<T> &a, int k, int code, int rank, double mt, unsigned nrot,
                                          unsigned nskip, unsigned long long mask) const
    {
        if (rank) atomicOr(&a.ctl->rank, 1);
        a.maxt[k] = fmax(maxt, mt);
        a.C[k] = C | code;
        a.nrot[k] = rot + nrot;
        a.nskip[k] = skip + nskip;
        a.nact[k] = act + (nrot > 0 ? 1u : 0u);
        a.ntc[k] = tc + (unsigned)__popcll(mask);
        a.active[k] = mask;
    }
};

// Per-slot rotation of the cross kernel in the precision its blocks are held
// in: (t, c) with c negated for an applied trigonometric rotation, decoded to
// (t, |c|, h) with h = -t for such a rotation, h = t otherwise (bit
// operations: no compare or select).
template <typename C>
struct SlotRot;
template <>
struct SlotRot<float> {
    typedef float2 packed;
    static __device__ __forceinline__ float2 pack(double t, double c) { return make_float2((float)t, (float)c); }
    static __device__ __forceinline__ float with_sign(float t, float c)
    {
        return __uint_as_float(__float_as_uint(t) ^ (__float_as_uint(c) & 0x80000000u));
    }
};
template <>
struct SlotRot<double> {
    typedef double2 packed;
    static __device__ __forceinline__ double2 pack(double t, double c) { return make_double2(t, c); }
    static __device__ __forceinline__ double with_sign(double t, double c)
    {
        return __hiloint2double(__double2hiint(t) ^ (__double2hiint(c) & (int)0x80000000), __double2loint(t));
    }
};
template <typename C>
struct Rot3 {
    C x, y, z;  // t, |c|, h
};
template <typename C, typename P>
__device__ __forceinline__ Rot3<C> unpack_rot(P r)
{
    return Rot3<C>{r.x, fabs(r.y), SlotRot<C>::with_sign(r.x, r.y)};
}

// Lane moves of the cross solve, on 32-bit words without the LDS pipe.
// In 16-lane rows: lane i takes lane i + 1 mod 16.
__device__ __forceinline__ int row_next(int v) { return __builtin_amdgcn_update_dpp(v, v, 0x12F, 0xf, 0xf, false); }
__device__ __forceinline__ float row_next(float v) { return __int_as_float(row_next(__float_as_int(v))); }
__device__ __forceinline__ double row_next(double v)
{
    return __hiloint2double(row_next(__double2hiint(v)), row_next(__double2loint(v)));
}

// ---------------------------------------------------------------------------
// Inner solve of one block pair for the cross steps (every outer step but the
// first of a sweep), register-resident.
//
// Slot coordinates: at inner step u slot s pairs local column L_s = s with
// R_s(u) = b + ((s + u) mod b).  A_P in these coordinates is P(x, y) =
// A(L_x, L_y), M(x, y) = A(L_x, R_y), N(x, y) = A(R_x, R_y); P and N are
// symmetric, so the unordered slot pairs {lo <= hi} with P, M(lo, hi),
// M(hi, lo) and N hold all of it.  A step rotates such a 2 x 2 block by its
// columns (slot hi), then by its rows (slot lo).  Since R_s(u + 1) =
// R_{s+1}(u), moving to the next step maps
//   M(x, y) <- M(x, y + 1),   N(x, y) <- N(x + 1, y + 1),   P unchanged.
//
// The waves of the workgroup take different parts:
//  - wave 0, the pivot wave: the blocks {s, s} (rows 0, 1 of its lanes, even
//    and odd s) and {s, s + 1} (rows 2, 3).  They carry the pivots of the
//    next step: it evaluates the b rotations from its own registers and
//    leaves them in LDS.
//  - waves 1 and 2: the other blocks in 2 x 2 tiles of slots, one tile
//    {2 ti, 2 ti + 1} x {2 tj, 2 tj + 1} per lane, by tile diagonals dd =
//    tj - ti mod 16 = 1 .. 8, 16 lanes each.  Half of a tile's shift stays in
//    the lane, one entry comes from the next lane, and six entries from
//    the tiles {ti, tj + 1} and {ti + 1, tj} through LDS.
//  - W, the accumulated rotations: lane j of a 16-lane row holds the
//    columns of slots 2 j and 2 j + 1 for a few rows; its shift is one move
//    within the row, so it reads nothing but the rotations.  With NT >= 512
//    the last four waves hold W (4 rows a lane); with 256 threads waves 1
//    and 2 (4 rows a lane) and wave 3 (8 rows a lane).
// One barrier per inner step separates a step's rotations and the entries
// exchanged at the last one (both double-buffered) from their readers.  The
// step's time is the pivot wave's dependency chain (read, rotate, move, about
// 35 dependent FP64 operations of rotation_params_fast), with the other
// waves' work beside it.
//
// What bounds it: that chain, in single solves (one block pair per compute
// unit), and the FP64 issue rate in batches.  A layout with every block held
// twice (both triangles, 1024 lanes), every shift through LDS and the rotation
// chain behind range and skip branches took 34.8 us for an inner launch of a
// graded n = 1024 solve (16 block pairs, FP64, V half included), this one 24.8;
// 300 batched problems of order 8 to 256 in the persistent launch: 32.8 ms,
// now 27.3.
// ---------------------------------------------------------------------------
constexpr int kXRows = 9;                   // exchange rows: tile diagonals 1 .. 8, then the diagonal tiles
constexpr int kXPart = kXRows * 16;         // one exchanged entry of every tile
constexpr int kXGroup = 3 * kXPart;         // the three entries a tile hands to one neighbour
// one step: both neighbours' entries, M(s, s + 2) for the pivot wave, and words that only keep lanes without an entry
// to write from branching
constexpr int kXBuf = 2 * kXGroup + kB + 128 + 256;

template <typename T>
struct CrossLds {
    // A_P staging at the start, the exchange buffers in the loop
    double buf[kB2 * kLd];
    // per slot (t, c), c negated for an applied trigonometric rotation (whose
    // h is -t; otherwise h = t).  The blocks of A_P and W are held in the
    // storage precision T: FP32 in the FP32 sweeps, where the rotations are
    // still computed in FP64 from the FP32 pivots and applied in FP32 (W is
    // rounded to T on output in any case).
    typename SlotRot<T>::packed prm[2][kB];
};
static_assert(2 * kXBuf <= kB2 * kLd, "exchange buffers fit the staging area");

// The 2 x 2 block (x00 x01; x10 x11): columns by pa, then rows by pq.
template <typename T>
__device__ __forceinline__ void rotate_block(T &x00, T &x01, T &x10, T &x11, const Rot3<T> &pa, const Rot3<T> &pq)
{
    const T f00 = fma(pa.z, x01, x00) * pa.y, f01 = fma(pa.x, x00, x01) * pa.y;
    const T f10 = fma(pa.z, x11, x10) * pa.y, f11 = fma(pa.x, x10, x11) * pa.y;
    x00 = fma(pq.z, f10, f00) * pq.y;
    x10 = fma(pq.x, f00, f10) * pq.y;
    x01 = fma(pq.z, f11, f01) * pq.y;
    x11 = fma(pq.x, f01, f11) * pq.y;
}

// W of RG rows and the slots 2 j, 2 j + 1 of this lane (RG = 0: none).  Held
// in vector values: as arrays of a structure the compiler left some of them
// in scratch memory.
template <typename T, int RG>
struct WRows {
    typedef T vec __attribute__((ext_vector_type(RG)));
    vec l0, r0, l1, r1;
    __device__ __forceinline__ void init(int row, int j)
    {
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            l0[q] = row + q == 2 * j ? T(1) : T(0);
            l1[q] = row + q == 2 * j + 1 ? T(1) : T(0);
            r0[q] = row + q == kB + 2 * j ? T(1) : T(0);
            r1[q] = row + q == kB + 2 * j + 1 ? T(1) : T(0);
        }
    }
    static __device__ __forceinline__ vec rotated(T z, vec b, vec a, T c)
    {
        vec o;
#pragma unroll
        for (int q = 0; q < RG; ++q) o[q] = fma(z, b[q], a[q]) * c;
        return o;
    }
    __device__ __forceinline__ void step(const Rot3<T> &p0, const Rot3<T> &p1)
    {
        const vec a0 = rotated(p0.z, r0, l0, p0.y), b0 = rotated(p0.x, l0, r0, p0.y);
        const vec a1 = rotated(p1.z, r1, l1, p1.y), b1 = rotated(p1.x, l1, r1, p1.y);
        l0 = a0;
        l1 = a1;
        r0 = b1;
#pragma unroll
        for (int q = 0; q < RG; ++q) r1[q] = row_next(b0[q]);
    }
    __device__ __forceinline__ void store(T *__restrict__ Wg, int row, int j) const
    {
        typedef T v2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            *reinterpret_cast<v2 *>(Wg + (row + q) * kB2 + 2 * j) = v2{l0[q], l1[q]};
            *reinterpret_cast<v2 *>(Wg + (row + q) * kB2 + kB + 2 * j) = v2{r0[q], r1[q]};
        }
    }
};
template <typename T>
struct WRows<T, 0> {
    __device__ __forceinline__ void init(int, int) {}
    __device__ __forceinline__ void step(const Rot3<T> &, const Rot3<T> &) {}
    __device__ __forceinline__ void store(T *, int, int) const {}
};

// Exchange address of the unordered tile pair {x, y}: its entries for the
// neighbour on x's side (x is the tile whose slots the entries' R columns
// belong to).  Group 0 when x is the higher tile, 1 when the lower.
__device__ __forceinline__ int cross_source(int other, int x)
{
    if (other == x) return 8 * 16 + x;
    const int dist = (x - other) & 15;
    const int row = dist <= 8 ? dist : 16 - dist, i = dist <= 8 ? other : x;
    return (x > other ? 0 : kXGroup) + (row - 1) * 16 + i;
}

// Signs of the pairs of a block pair: all trigonometric, all hyperbolic, or
// both kinds (one of the blocks holds columns of both signs, or the pairs lie
// within blocks of different signs).
enum { kTrig = 0, kHyp = 1, kBothKinds = 2 };

// Skip test and rotation of one slot for the inner solves' rotation waves,
// evaluated side by side (independent dependency chains).  A lone wave issues
// one vector instruction in about six cycles whatever it depends on, so the
// step time of an inner solve is this instruction count: the signs of the
// pairs are settled outside the loop where they can be, and one integer
// compare covers the ranges of the short rotation form and of the squared skip
// test; the branch is taken only when an entry leaves them.
struct SlotRotator {
    double tol, tol2;
    unsigned range_lo, range_len;  // high words of the entries the short forms take
    __device__ __forceinline__ explicit SlotRotator(double tol_) : tol(tol_), tol2(tol_ * tol_)
    {
        // entries in [2^E, 2^480), E >= -480 and tol^2 2^(2E) >= 2^-999
        int E = -480;
        if (!(tol2 >= 0x1p-38)) E = max(E, tol2 >= 0x1p-1000 ? (-998 - ilogb(tol2)) / 2 : 1024);
        const int lo_w = min(E + 1023, 2047), hi_w = 480 + 1023;
        range_lo = (unsigned)lo_w << 20;
        range_len = lo_w < hi_w ? (unsigned)(hi_w - lo_w) << 20 : 0u;
    }
    template <int MODE>
    __device__ __forceinline__ void operator()(double aii, double ajj, double aij, bool trig, double &t, double &c,
                                               bool &skip, bool &bad) const
    {
        bad = MODE == kTrig  ? rotation_params_short(aii, ajj, aij, true, t, c)
              : MODE == kHyp ? rotation_params_short(aii, ajj, aij, false, t, c)
                             : rotation_params_short(aii, ajj, aij, trig, t, c);
        skip = aij * aij < tol2 * (aii * ajj);
        const unsigned ei = (unsigned)__double2hiint(aii) - range_lo, ej = (unsigned)__double2hiint(ajj) - range_lo;
        const bool odd = max(ei, ej) >= range_len;
        if (__builtin_expect(__ballot(odd) != 0ull, 0)) {
            if (odd) {
                if (!fast_range(aii, ajj)) bad = rotation_params(aii, ajj, aij, trig ? -1 : 1, t, c) != 0;
                skip = rel_orthogonal_sq(aii, ajj, aij, tol, tol2);
            }
        }
    }
};

// What the pivot wave counts over the inner steps.
struct CrossCount {
    unsigned rotated;  // lane s < b: bit b - 1 - u = slot s rotated at inner step u
    unsigned nbad;     // pairs found rank deficient (wave-uniform)
    double maxt;       // the lane's largest |t|
};

// The pivot wave; what it counts is packed into one bit per step, and the lane
// moves go through ds_bpermute.
template <typename T>
struct CrossPivot {
    T P, x01, x10, N;   // the block {lo, hi} of this lane
    int s, u0;          // slot; the inner step of step<0>
    bool up, wrap;      // block {s, s + 1} (lanes 32 ..), else {s, s}; lane 63: {0, 31}, lo = s + 1
    bool lpos;          // column L_s has sign +
    int rbase, p;       // position of R_s(0) - s
    T *ex;
    const typename SlotRot<T>::packed *plo, *phi;
    int o1, o2;         // where this lane's entries for the tiles go
    int zsrc, nsrc;     // byte addresses of the lane moves
    CrossCount n;

    static __device__ __forceinline__ float move(int src, float v)
    {
        return __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(v)));
    }
    static __device__ __forceinline__ double move(int src, double v)
    {
        return __hiloint2double(__builtin_amdgcn_ds_bpermute(src, __double2hiint(v)),
                                __builtin_amdgcn_ds_bpermute(src, __double2loint(v)));
    }

    template <int PB, int MODE>
    __device__ __forceinline__ void step(CrossLds<T> &L, const SlotRotator &rotator)
    {
        bool rot = false;
        if (!up) {
            const double pll = P, plr = x01, prr = N;
            const bool trig = MODE == kTrig || (MODE == kBothKinds && lpos == (rbase + ((s + u0 + PB) & 31) < p));
            double t, c;
            bool skip, bad;
            rotator.template operator()<MODE>(pll, prr, plr, trig, t, c, skip, bad);
            rot = !skip && !bad;
            const double tr = rot ? t : 0.0, cr = rot ? (trig ? -c : c) : 1.0;
            L.prm[PB][s] = SlotRot<T>::pack(tr, cr);
            n.maxt = fmax(n.maxt, fabs(tr));
            n.rotated = 2u * n.rotated + (rot ? 1u : 0u);
            if (MODE != kTrig) n.nbad += (unsigned)__popcll(__ballot(!skip && bad));
        }
        role_barrier();
        const T xe = ex[(PB ^ 1) * kXBuf + 2 * kXGroup + s];
        const Rot3<T> pa = unpack_rot<T>(phi[PB * kB]), pq = unpack_rot<T>(plo[PB * kB]);
        // the entry from the tiles, read before (first step: from the staged A_P): M(s, s + 1)
        x01 = up && !wrap ? xe : x01;
        x10 = wrap ? xe : x10;
        rotate_block(P, x01, x10, N, pa, pq);
        const T Mu = rot ? T(0) : (wrap ? x10 : x01);  // M(s, s), M(s, s + 1)
        // the diagonal tiles' entries: M(2i, 2i), M(2i + 1, 2i), N(2i, 2i + 1)
        // (the other lanes write to words of their own that nothing reads)
        ex[PB * kXBuf + o1] = up ? x10 : Mu;
        ex[PB * kXBuf + o2] = N;
        // {s, s} takes M(s, s + 1); {s, s + 1} takes M(s + 1, s + 1) as the one
        // entry and M(s, s + 2), from its tile, as the other
        x01 = x10 = move(zsrc, Mu);
        N = move(nsrc, N);
    }

    template <int MODE>
    __device__ __forceinline__ void run(CrossLds<T> &L, const SlotRotator &rotator, int nsteps)
    {
#pragma unroll 1
        for (u0 = 0; u0 < nsteps; u0 += 2) {
            step<0, MODE>(L, rotator);
            step<1, MODE>(L, rotator);
        }
    }
};

template <typename T>
__device__ __forceinline__ CrossCount cross_pivot_wave(const BlockArgsT<T> &a, int2 IJ, CrossLds<T> &L, int nsteps)
{
    const double *const buf = L.buf;
    CrossPivot<T> w;
    const int lane = threadIdx.x & 63;
    w.ex = reinterpret_cast<T *>(L.buf);
    const int s = w.s = lane & 31, s1 = (s + 1) & 31;
    w.up = lane >= 32;
    const int s2 = w.up ? s1 : s;
    const int lo = min(s, s2), hi = max(s, s2);
    w.wrap = lane == 63;
    w.p = a.p;
    w.lpos = IJ.x * kB + s < a.p;
    w.rbase = IJ.y * kB;
    const SlotRotator rotator(a.tol);
    w.plo = &L.prm[0][lo];
    w.phi = &L.prm[0][hi];
    const int i = s >> 1, dummy = 2 * kXGroup + kB + lane;
    const bool even = (s & 1) == 0;
    w.o1 = even ? (w.up ? kXPart : 0) + 8 * 16 + i : dummy;
    w.o2 = even && w.up ? 2 * kXPart + 8 * 16 + i : dummy + 64;
    w.zsrc = 4 * (w.up ? s1 : s + 32);
    w.nsrc = 4 * ((lane & 32) | s1);
    w.P = (T)buf[lo * kLd + hi];
    w.x01 = (T)buf[lo * kLd + kB + hi];
    w.x10 = (T)buf[hi * kLd + kB + lo];
    w.N = (T)buf[(kB + lo) * kLd + kB + hi];
    w.n = CrossCount{0u, 0u, 0.0};
    role_barrier();  // the staging area becomes the exchange area
    // as if exchanged by a step before the first
    if (w.up) w.ex[kXBuf + 2 * kXGroup + s] = w.wrap ? w.x10 : w.x01;
    const bool li = IJ.x * kB + kB <= a.p, lj = IJ.y * kB + kB <= a.p;  // all +
    const bool ni = IJ.x * kB >= a.p, nj = IJ.y * kB >= a.p;            // all -
    const int mode = (li && lj) || (ni && nj) ? kTrig : ((li && nj) || (ni && lj) ? kHyp : kBothKinds);
    __builtin_amdgcn_s_setprio(2);
    if (mode == kTrig)
        w.template run<kTrig>(L, rotator, nsteps);
    else if (mode == kHyp)
        w.template run<kHyp>(L, rotator, nsteps);
    else
        w.template run<kBothKinds>(L, rotator, nsteps);
    __builtin_amdgcn_s_setprio(0);
    return w.n;
}

template <typename T>
struct CrossTile {
    T P[2][2], U[2][2], D[2][2], N[2][2];  // [q][h]: slots lo = 2 ti + q, hi = 2 tj + h; U = M(lo, hi), D = M(hi, lo)
    T *ex;
    int ti, tj, e1, e2, own;
    int xe;     // the pivot wave's entries M(s, s + 2), s = 2 i, 2 i + 1 (tiles next to the diagonal; else unread)
    bool wrap;  // {15, 0}: they are below the diagonal

    template <int PB>
    __device__ __forceinline__ void step(CrossLds<T> &L)
    {
        role_barrier();
        const typename SlotRot<T>::packed *const prm = L.prm[PB];
        const typename SlotRot<T>::packed rq0 = prm[2 * ti], rq1 = prm[2 * ti + 1], rh0 = prm[2 * tj], rh1 = prm[2 * tj + 1];
        const T *const in = ex + (PB ^ 1) * kXBuf;
        U[0][1] = in[e1];
        U[1][1] = in[e1 + kXPart];
        N[0][1] = in[e1 + 2 * kXPart];
        D[1][0] = in[e2];
        D[1][1] = in[e2 + kXPart];
        N[1][0] = in[e2 + 2 * kXPart];
        const Rot3<T> q0 = unpack_rot<T>(rq0), q1 = unpack_rot<T>(rq1), h0 = unpack_rot<T>(rh0), h1 = unpack_rot<T>(rh1);
        rotate_block(P[0][0], U[0][0], D[0][0], N[0][0], h0, q0);
        rotate_block(P[1][0], U[1][0], D[1][0], N[1][0], h0, q1);
        rotate_block(P[0][1], U[0][1], D[0][1], N[0][1], h1, q0);
        rotate_block(P[1][1], U[1][1], D[1][1], N[1][1], h1, q1);
        T *const out = ex + PB * kXBuf;
        out[own] = U[0][0];
        out[own + kXPart] = U[1][0];
        out[own + 2 * kXPart] = N[1][0];
        out[kXGroup + own] = D[0][0];
        out[kXGroup + own + kXPart] = D[0][1];
        out[kXGroup + own + 2 * kXPart] = N[0][1];
        out[xe] = wrap ? D[0][0] : U[0][0];
        out[xe + 1] = wrap ? D[1][1] : U[1][1];
        U[0][0] = U[0][1];
        U[1][0] = U[1][1];
        D[0][0] = D[1][0];
        D[0][1] = D[1][1];
        const T n00 = N[0][0];
        N[0][0] = N[1][1];
        N[1][1] = row_next(n00);
    }
};

template <typename T, int WR>
__device__ __forceinline__ void cross_tile_wave(CrossLds<T> &L, int nsteps, int wave, int wrow, T *__restrict__ Wg)
{
    const double *const buf = L.buf;
    const int lane = threadIdx.x & 63;
    const int row = (wave - 1) * 4 + (lane >> 4), i = lane & 15;  // tile diagonal row + 1
    const int y = (i + row + 1) & 15;
    CrossTile<T> w;
    w.ex = reinterpret_cast<T *>(L.buf);
    const int ti = w.ti = min(i, y), tj = w.tj = max(i, y);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int x = 2 * ti + q, z = 2 * tj + h;
            w.P[q][h] = (T)buf[x * kLd + z];
            w.U[q][h] = (T)buf[x * kLd + kB + z];
            w.D[q][h] = (T)buf[z * kLd + kB + x];
            w.N[q][h] = (T)buf[(kB + x) * kLd + kB + z];
        }
    w.e1 = cross_source(ti, (tj + 1) & 15);
    w.e2 = cross_source(tj, (ti + 1) & 15);
    w.own = row * 16 + i;
    w.wrap = row == 0 && i == 15;
    w.xe = row == 0 ? 2 * kXGroup + 2 * i : 2 * kXGroup + kB + 128 + 2 * w.own;
    WRows<T, WR> wr;
    wr.init(wrow, i);
    role_barrier();
    {
        // the entries of the first step, as if exchanged by a step before it
        T *const in = w.ex + kXBuf;
        in[w.e1] = w.U[0][1];
        in[w.e1 + kXPart] = w.U[1][1];
        in[w.e1 + 2 * kXPart] = w.N[0][1];
        in[w.e2] = w.D[1][0];
        in[w.e2 + kXPart] = w.D[1][1];
        in[w.e2 + 2 * kXPart] = w.N[1][0];
    }
#pragma unroll 1
    for (int u = 0; u < nsteps; u += 2) {
        w.template step<0>(L);
        if (WR > 0) wr.step(unpack_rot<T>(L.prm[0][2 * i]), unpack_rot<T>(L.prm[0][2 * i + 1]));
        w.template step<1>(L);
        if (WR > 0) wr.step(unpack_rot<T>(L.prm[1][2 * i]), unpack_rot<T>(L.prm[1][2 * i + 1]));
    }
    if (WR > 0) wr.store(Wg, wrow, i);
}

template <typename T, int RG>
__device__ __forceinline__ void cross_w_wave(CrossLds<T> &L, int nsteps, int wrow, T *__restrict__ Wg)
{
    const int j = threadIdx.x & 15;
    WRows<T, RG> w;
    w.init(wrow, j);
    role_barrier();
#pragma unroll 1
    for (int u = 0; u < nsteps; u += 2) {
        role_barrier();
        w.step(unpack_rot<T>(L.prm[0][2 * j]), unpack_rot<T>(L.prm[0][2 * j + 1]));
        role_barrier();
        w.step(unpack_rot<T>(L.prm[1][2 * j]), unpack_rot<T>(L.prm[1][2 * j + 1]));
    }
    w.store(Wg, wrow, j);
}

// Every thread must call it (barriers).
template <typename T, int NT>
__device__ __forceinline__ void inner_cross_pair(const BlockArgsT<T> &a, int k, CrossLds<T> &L, int &live, int tid)
{
    static_assert(NT == 256 || NT == 512, "thread count");
    double *const buf = L.buf;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int2 IJ = outer_pair(a, k);
    // the sweep's counters so far, read ahead of their update at the end
    SweepSoFar so_far;
    if (tid == 0) so_far.read(a, k);
    stage_gram<T, NT>(a, k, tid, [&](int x, int y, double v) { buf[x * kLd + y] = v; });
    if (tid == 0) live = 0;
    __syncthreads();
    {
        // Every cross pair (x, b + y) of the block pair is the pivot of one
        // inner step.  If none fails the skip test (2.3) on A_P as staged, the
        // first step rotates nothing, A_P stays as it is, and by induction no
        // step rotates: the whole solve is skipped (W = I).  The test takes the
        // entries as the loop holds them (rounded to T).
        constexpr int K = (kB * kB) / NT;
        const double tol = a.tol, tol2 = tol * tol;
        int fails = 0;
        const int y = tid & 31;
        const double ayy = (T)buf[(kB + y) * kLd + kB + y];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int x = (tid + NT * q) >> 5;
            fails |= rel_orthogonal_sq((T)buf[x * kLd + x], ayy, (T)buf[x * kLd + kB + y], tol, tol2) ? 0 : 1;
        }
        if (__ballot(fails) != 0ull && lane == 0) live = 1;
    }
    __syncthreads();
    const int nsteps = __builtin_amdgcn_readfirstlane(live) ? kB : 0;  // the same in every thread
    T *const Wg = a.W + (size_t)k * (kB2 * kB2);
    constexpr int kWWave = NT / 64 - 4;  // first of the four W waves (NT >= 512)
    if (wave == 0) {
        const CrossCount o = cross_pivot_wave<T>(a, IJ, L, nsteps);
        double maxt = o.maxt;
        // touched columns: L_s, and R_s(u) = b + ((s + u) mod b) for the steps
        // u in which slot s rotated
        const unsigned by_step = __brev(o.rotated);  // bit u
        const int sh = lane & 31;
        unsigned mlo = o.rotated ? 1u << sh : 0u, mhi = (by_step << sh) | (sh ? by_step >> (32 - sh) : 0u);
        unsigned rot_sum = (unsigned)__popc(o.rotated);
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) {
            maxt = fmax(maxt, __shfl_xor(maxt, m, 64));
            mlo |= __shfl_xor(mlo, m, 64);
            mhi |= __shfl_xor(mhi, m, 64);
            rot_sum += __shfl_xor(rot_sum, m, 64);
        }
        // eq. (4.2) codes of the applied rotations, OR-ed
        if (tid == 0)
            so_far.write(a, k, rot_sum > 0 ? (maxt > a.tthresh ? 3 : 1) : 0, (int)o.nbad, maxt, rot_sum,
                         (unsigned)(kB * kB) - rot_sum - o.nbad, ((unsigned long long)mhi << 32) | mlo);
    } else if (wave == 1 || wave == 2) {
        cross_tile_wave<T, NT == 256 ? 4 : 0>(L, nsteps, wave, 4 * ((wave - 1) * 4 + (lane >> 4)), Wg);
    } else if (NT == 256) {
        cross_w_wave<T, 8>(L, nsteps, kB + 8 * (lane >> 4), Wg);
    } else if (wave >= kWWave) {
        cross_w_wave<T, 4>(L, nsteps, 4 * ((wave - kWWave) * 4 + (lane >> 4)), Wg);
    } else {
        for (int u = 0; u <= nsteps; ++u) role_barrier();
    }
}

// The barriers of inner_cross_pair, for threads of the workgroup without a
// block pair.
__device__ __forceinline__ void inner_cross_idle(const int &live)
{
    __syncthreads();
    __syncthreads();
    const int nsteps = __builtin_amdgcn_readfirstlane(live) ? kB : 0;
    for (int u = 0; u <= nsteps; ++u) role_barrier();
}


// ---------------------------------------------------------------------------
// Inner solve of one block pair over all pairs of its 2b columns: sweeps of the
// circle method over 2b indices (2b - 1 inner steps of b pairs each).  One
// sweep in the first outer step of a sweep of the block-oriented method;
// repeated until a sweep applies no rotation (at most a.inner_sweeps) in every
// outer step of the full-block method.
//
// At an inner step every local index sits in one slot s, on its left or its
// right (L_s, R_s); the slots' indices then move on by one place of the circle
// (L_0 stays, L_1 -> R_0, L_k -> L_{k-1}, R_k -> R_{k+1}, R_{b-1} -> L_{b-1}).
// A_P sits in LDS by places, one 2 x 2 block (L, R) x (L, R) per slot pair
// {sl <= sh}: one thread reads the block, turns it (columns of slot sh first,
// then rows of slot sl) and writes each entry to the place where the next step
// reads it.  The moves are the same in every step, so all addresses are
// settled before the loop, and the entries of consecutive blocks are
// consecutive.  The first wave evaluates the b rotations from the diagonal
// blocks, oriented to (L, R).  W is held by rows in registers: lane j of a
// 16-lane row has the columns of slots 2 j and 2 j + 1, and the same moves are
// lane moves within the row.  Two barriers per inner step: rotations out (the
// blocks have been read by then), blocks written.
//
// What bounds it: the rotation wave's chain (read, rotate, write: about 650
// cycles of 1500) and then the block waves' one (parameters, rotation, writes),
// a barrier between them; with four pairs per compute unit the vector
// instructions.  Launches over 64 pairs (FP64, one sweep): 45 us at 1024
// threads, 70 at 256; 1024 pairs at 256 threads: 120 us.  With A_P by indices
// (addresses computed anew in every step) 72, 113 and 241 us; with every block
// held twice, W in LDS and 32-byte parameters 107 us at 1024.
// Where the persistent batched kernel's last pair of a slot had few touched
// columns, steps without a rotation turn nothing (circle_block_wave): batches
// of 200 / 300 / 500 problems of order 1 to 8, where most steps are such ones,
// take 1.21 / 1.27 / 1.38 ms instead of 1.30 / 1.32 / 1.42 (1.21 / 1.25 / 1.36
// with A_P by indices, which had nothing to move then; round-robin, one circle
// solve a sweep, 300 problems 1.20, 1.28 and 1.10).
// ---------------------------------------------------------------------------
constexpr int kCircleBlocks = kB * (kB + 1) / 2;
struct CircleLds {
    // entries LL, LR, RL, RR of the blocks (a diagonal block's LR stands for its RL too)
    double X[4][kCircleBlocks];
    double2 prm[kB];   // (t, c) of each slot, as in the cross solve, L the first index
    unsigned rotated;  // slots that rotate in this step
};

// A place is 2 s + side (0: L_s, 1: R_s).  Address of entry (u, v) of A_P, u
// and v places of the slots sl <= sh (block item (sh - sl) mod b, the shorter
// way round, times b, plus the slot it starts from).
__device__ __forceinline__ int circle_at(int u, int v)
{
    const int su = u >> 1, sv = v >> 1, lo = min(su, sv), hi = max(su, sv), d = hi - lo;
    const int item = d <= kB / 2 ? d * kB + lo : (kB - d) * kB + hi;
    const int first = su <= sv ? u : v, second = su <= sv ? v : u;
    const int entry = d == 0 ? (u & 1) + (v & 1) + ((u & v) & 1) : 2 * (first & 1) + (second & 1);
    return entry * kCircleBlocks + item;
}
// Where the index at place u moves.
__device__ __forceinline__ int circle_next(int u)
{
    if (u & 1) return u == 2 * kB - 1 ? u - 1 : u + 2;
    return u == 0 ? 0 : (u == 2 ? 1 : u - 2);
}
// The place of local index i at the first step.
__device__ __forceinline__ int circle_place(int i) { return i < kB ? 2 * i : 2 * (kB2 - 1 - i) + 1; }

// The two indices of slot s at inner step u (roundrobin_pair without its
// ordering), and their next values.
struct CircleSlot {
    int l, r;
    __device__ __forceinline__ void start(int s)
    {
        l = s;
        r = kB2 - 1 - s;
    }
    __device__ __forceinline__ void next()
    {
        l = l == 0 ? 0 : (l == kB2 - 1 ? 1 : l + 1);  // index 0 stays in slot 0
        r = r == kB2 - 1 ? 1 : r + 1;
    }
};

// W of RG rows and the slots 2 j, 2 j + 1.
template <int RG>
struct CircleW {
    typedef double vec __attribute__((ext_vector_type(RG)));
    vec l0, r0, l1, r1;
    __device__ __forceinline__ void init(int row, int j)
    {
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            l0[q] = row + q == 2 * j ? 1.0 : 0.0;
            r0[q] = row + q == kB2 - 1 - 2 * j ? 1.0 : 0.0;
            l1[q] = row + q == 2 * j + 1 ? 1.0 : 0.0;
            r1[q] = row + q == kB2 - 2 - 2 * j ? 1.0 : 0.0;
        }
    }
    template <int kCtrl>
    static __device__ __forceinline__ double shifted(double edge, double v)
    {
        return __hiloint2double(
            __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), kCtrl, 0xf, 0xf, false),
            __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), kCtrl, 0xf, 0xf, false));
    }
    __device__ __forceinline__ void rotate(const double2 &w0, const double2 &w1)
    {
        const Rot3<double> p0 = unpack_rot<double>(w0), p1 = unpack_rot<double>(w1);
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const double a0 = l0[q], a1 = l1[q];
            l0[q] = fma(p0.z, r0[q], a0) * p0.y;
            r0[q] = fma(p0.x, a0, r0[q]) * p0.y;
            l1[q] = fma(p1.z, r1[q], a1) * p1.y;
            r1[q] = fma(p1.x, a1, r1[q]) * p1.y;
        }
    }
    __device__ __forceinline__ void move(int j)
    {
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const double nl0 = l0[q], nr0 = r0[q], nl1 = l1[q], nr1 = r1[q];
            l0[q] = j == 0 ? nl0 : nl1;
            l1[q] = shifted<0x101>(nr1, nl0);  // row_shl:1, lane 15 from its own R
            r0[q] = shifted<0x111>(nl1, nr1);  // row_shr:1, lane 0 from its own L
            r1[q] = nr0;
        }
    }
    template <typename T>
    __device__ __forceinline__ void store(T *__restrict__ Wg, int row, int j) const
    {
        typedef T v2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            *reinterpret_cast<v2 *>(Wg + (row + q) * kB2 + 2 * j) = v2{(T)l0[q], (T)l1[q]};
            *reinterpret_cast<v2 *>(Wg + (row + q) * kB2 + kB2 - 2 - 2 * j) = v2{(T)r1[q], (T)r0[q]};
        }
    }
};

// What the rotation wave counts, per lane (slot).
struct CircleCount {
    unsigned nrot, nskip, rank;
    double maxt;
    unsigned long long tmask;
};

template <int MODE, bool kWTurn>
__device__ __forceinline__ CircleCount circle_rotation_wave(const SlotRotator &rotator, int p, int2 IJ, CircleLds &L,
                                                            int nsweeps, CircleW<4> &w)
{
    const int lane = threadIdx.x & 63, s = lane & 31, j = lane & 15;
    const bool own = lane < kB;
    CircleSlot sl;
    sl.start(s);
    CircleCount n{0u, 0u, 0u, 0.0, 0ull};
    // ascending pair: L_s < R_s; else the smaller index is R_s
    auto is_trig = [&] {
        return MODE == kTrig || (local_pos(sl.l, IJ.x, IJ.y) < p) == (local_pos(sl.r, IJ.x, IJ.y) < p);
    };
    bool trig = is_trig();
    __builtin_amdgcn_s_setprio(2);
    for (int sw = 0; sw < nsweeps; ++sw) {
        unsigned any = 0;
#pragma unroll 1
        for (int u = 0; u < kB2 - 1; ++u) {
            const double ll = L.X[0][s], lr = L.X[1][s], rr = L.X[3][s];
            const bool asc = sl.l < sl.r;
            double t, c;
            bool skip, bad;
            rotator.template operator()<MODE>(asc ? ll : rr, asc ? rr : ll, lr, trig, t, c, skip, bad);
            const bool rot = !skip && !bad;
            const double tr = rot ? t : 0.0;
            const unsigned mask = (unsigned)__ballot(rot);  // lanes 0 .. b - 1
            // the smaller index takes h = -+t, the other t: oriented to (L, R)
            if (own) L.prm[s] = make_double2(trig && !asc ? -tr : tr, rot ? (trig ? -c : c) : 1.0);
            if (lane == 0) L.rotated = mask;
            role_barrier();
            any |= mask;
            n.nrot += rot ? 1u : 0u;
            n.nskip += skip ? 1u : 0u;
            if (MODE != kTrig) n.rank |= !skip && bad ? 1u : 0u;
            n.maxt = fmax(n.maxt, fabs(tr));
            n.tmask |= rot ? (1ull << sl.l) | (1ull << sl.r) : 0ull;
            sl.next();
            trig = is_trig();
            if (kWTurn) {
                if (mask) w.rotate(L.prm[2 * j], L.prm[2 * j + 1]);
                w.move(j);
            }
            role_barrier();
        }
        if (!any) break;  // a sweep without rotations: the block is diagonal
    }
    __builtin_amdgcn_s_setprio(0);
    return n;
}

// NB blocks of A_P per thread (items tid0 + nthreads q), and W when kWTurn.
// kSparse: a step without a rotation turns nothing and only moves the entries.
// The others then wait for the step's mask before they turn: with few problems
// per compute unit, where the chain counts, up to 2% of a solve (300 problems of
// order 100 to 128: 5.52 -> 5.60 ms), and in the 1024-thread form more than it
// saves (three full-block sweeps of n = 1024: 28.3 -> 32.3 ms).
template <int NB, bool kWTurn, bool kSparse>
__device__ __forceinline__ void circle_block_wave(CircleLds &L, int nsweeps, int tid0, int nthreads, CircleW<4> &w)
{
    const int j = threadIdx.x & 15;
    double *const X = &L.X[0][0];
    int item[NB], to[NB][4];
    const double2 *pa[NB], *pq[NB];
    bool have[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        have[q] = tid0 + nthreads * q < kCircleBlocks;
        item[q] = have[q] ? tid0 + nthreads * q : 0;
        const int s = item[q] & 31, s2 = (s + (item[q] >> 5)) & 31, sl = min(s, s2), sh = max(s, s2);
        pa[q] = &L.prm[sh];
        pq[q] = &L.prm[sl];
#pragma unroll
        for (int v = 0; v < 4; ++v) to[q][v] = circle_at(circle_next(2 * sl + (v >> 1)), circle_next(2 * sh + (v & 1)));
    }
    const bool diag = item[0] < kB;  // only a first block can be a diagonal one
    for (int sw = 0; sw < nsweeps; ++sw) {
        unsigned any = 0;
#pragma unroll 1
        for (int u = 0; u < kB2 - 1; ++u) {
            double e[NB][4];
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) e[q][v] = L.X[v][item[q]];
            role_barrier();
            double2 ra, rq;  // kSparse: on their way beside the mask
            if (kSparse) {
                ra = *pa[0];
                rq = *pq[0];
            }
            const unsigned mask = L.rotated;
            any |= mask;
            e[0][2] = diag ? e[0][1] : e[0][2];
            auto rotate = [&](int q) {
                rotate_block(e[q][0], e[q][1], e[q][2], e[q][3], unpack_rot<double>(kSparse && q == 0 ? ra : *pa[q]),
                             unpack_rot<double>(kSparse && q == 0 ? rq : *pq[q]));
                if (q == 0 && diag) e[0][1] = e[0][2] = (mask >> item[0]) & 1u ? 0.0 : e[0][1];
            };
            const bool turn = !kSparse || __builtin_amdgcn_readfirstlane(mask) != 0;
            if (kSparse && turn)
#pragma unroll
                for (int q = 0; q < NB; ++q) rotate(q);
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                if (!kSparse) rotate(q);
                if (have[q])
#pragma unroll
                    for (int v = 0; v < 4; ++v) X[to[q][v]] = e[q][v];
            }
            if (kWTurn) {
                if (turn) w.rotate(L.prm[2 * j], L.prm[2 * j + 1]);
                w.move(j);
            }
            role_barrier();
        }
        if (!__builtin_amdgcn_readfirstlane(any)) break;
    }
}

// Touched columns of the pair that the slot worked on before, up to which most
// steps are taken to rotate nothing: m columns have at most m (m - 1) / 2 pairs
// for 63 steps, and few of them rotate in the last sweeps.
constexpr int kFewTouched = 16;

// NT threads.  kSparse: a.active[k] holds the last pair's touched columns, and
// with few of them steps without a rotation turn nothing.  Every thread must
// call it (barriers).
template <typename T, int NT, bool kSparse = false>
__device__ __forceinline__ void inner_circle_pair(const BlockArgsT<T> &a, int k, CircleLds &L, int tid)
{
    static_assert(NT == 256 || (NT == 1024 && !kSparse), "thread count");
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int2 IJ = outer_pair(a, k);
    const unsigned long long last = kSparse ? a.active[k] : 0ull;  // read ahead of its use
    // the sweep's counters so far, read ahead of their update at the end
    SweepSoFar so_far;
    if (tid == 0) so_far.read(a, k);
    stage_gram<T, NT>(a, k, tid, [&](int x, int y, double v) {
        if (x <= y) (&L.X[0][0])[circle_at(circle_place(x), circle_place(y))] = v;
    });
    __syncthreads();
    const int nsweeps = a.inner_sweeps > 0 ? a.inner_sweeps : 1;
    const bool few = kSparse && __builtin_amdgcn_readfirstlane(__popcll(last)) <= kFewTouched;
    // W, four rows a lane: every wave of 256 threads, else the last four
    constexpr int kWWave = NT / 64 - 4;
    const bool wturn = wave >= kWWave;
    const int wrow = 4 * ((wave - kWWave) * 4 + (lane >> 4)), j = lane & 15;
    CircleW<4> w;
    w.init(wrow, j);
    // the blocks of A_P: 528 over the waves after the first
    constexpr int kA = NT - 64, kNB = (kCircleBlocks + kA - 1) / kA;
    if (wave == 0) {
        const SlotRotator rotator(a.tol);
        const bool same = (IJ.x * kB + kB <= a.p && IJ.y * kB + kB <= a.p) || (IJ.x * kB >= a.p && IJ.y * kB >= a.p);
        const double tthresh = a.tthresh;
        CircleCount o = same ? circle_rotation_wave<kTrig, kWWave == 0>(rotator, a.p, IJ, L, nsweeps, w)
                             : circle_rotation_wave<kBothKinds, kWWave == 0>(rotator, a.p, IJ, L, nsweeps, w);
        unsigned mlo = (unsigned)o.tmask, mhi = (unsigned)(o.tmask >> 32);
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) {
            o.rank |= __shfl_xor(o.rank, m, 64);
            o.nrot += __shfl_xor(o.nrot, m, 64);
            o.nskip += __shfl_xor(o.nskip, m, 64);
            o.maxt = fmax(o.maxt, __shfl_xor(o.maxt, m, 64));
            mlo |= __shfl_xor(mlo, m, 64);
            mhi |= __shfl_xor(mhi, m, 64);
        }
        // eq. (4.2) codes of the applied rotations, OR-ed
        if (tid == 0)
            so_far.write(a, k, o.nrot > 0 ? (o.maxt > tthresh ? 3 : 1) : 0, (int)o.rank, o.maxt, o.nrot, o.nskip,
                         ((unsigned long long)mhi << 32) | mlo);
    } else if (few) {
        if constexpr (kSparse) circle_block_wave<kNB, kWWave == 0, true>(L, nsweeps, tid - 64, kA, w);
    } else if (wturn) {
        circle_block_wave<kNB, true, false>(L, nsweeps, tid - 64, kA, w);
    } else {
        circle_block_wave<kNB, false, false>(L, nsweeps, tid - 64, kA, w);
    }
    if (wturn) w.store(a.W + (size_t)k * (kB2 * kB2), wrow, j);
}

// The barriers of inner_circle_pair with one sweep, for threads of the
// workgroup without a block pair.
__device__ __forceinline__ void inner_circle_idle()
{
    __syncthreads();
    for (int u = 0; u < 2 * (kB2 - 1); ++u) role_barrier();
}

// ---------------------------------------------------------------------------
// Update: [G_P | V_P] <- [G_P | V_P] W.
//
// Computed transposed, (X W)^T = W^T X^T for each 16-row strip X of G_P (or
// V_P): the MFMA B operand (k = column x, j = row) is then 16 consecutive rows
// of one column per 16 lanes, read straight from HBM, and the result lanes
// (i = output column, j = row) store 16 consecutive rows likewise -- no LDS
// staging of the data.  W sits in LDS for all strips of the workgroup.
// ---------------------------------------------------------------------------
// One strip per wave: 64 rows per 256-thread workgroup.  Every workgroup then
// runs one chain -- column list and W, the strip's rows, 64 products, stores --
// and the many short workgroups of a compute unit overlap theirs.  Longer
// tiles kept W for several strips (FP64: in 128 registers) at a fraction of
// the waves: with 256 rows the FP64 launch of a graded n = 1024 solve took
// 18 us against 10.2, at n = 4096 33.7 us against 31.1; with 128 rows the FP32
// launch at n = 1024 took 15.8 us against 13.7 (n = 4096: the same).
template <typename T>
struct UpdCfg {
    static constexpr int ld = sizeof(T) == 4 ? kB2 + 16 : kB2 + 8;  // LDS row stride of W: a read's 4 row groups in distinct banks
};
constexpr int kUpdRows = 64;

// Compact update of a block pair whose rotations touched only m <= NC of its
// 2b local columns (list tl, physical columns cols): the other columns of W
// are unit columns and every touched column of W is zero outside the touched
// rows (rotations only combine touched columns), so [G_T | V_T] <- [G_T | V_T]
// W_TT is the whole update.  Same MFMA formulation as the full update with NC
// columns, W_TT zero-padded to NC x NC; only the m touched columns are read
// and written.  NT threads.
template <typename T, int NC, int NT>
__device__ __forceinline__ void update_compact(const BlockArgsT<T> &a, int k, T *M, T *M2, int row_base,
                                               int nstrips, T *Wl, const int *cols, const int *tl, int m, int tid)
{
    constexpr int NW = NT / 64;
    const T *Wg = a.W + (size_t)k * (kB2 * kB2);
    for (int idx = tid; idx < NC * NC; idx += NT) {
        const int i = idx / NC, j = idx % NC;
        Wl[idx] = (i < m && j < m) ? Wg[tl[i] * kB2 + tl[j]] : T(0);
    }
    __syncthreads();
    constexpr int KK = NC / 4, YT = NC / 16;
    const int lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const unsigned row_off = (unsigned)(row_base + lr) * (unsigned)sizeof(T);
    const unsigned col_bytes = (unsigned)a.ldg * (unsigned)sizeof(T);
#pragma unroll 1
    for (int at = wave; at < (M2 ? 2 * nstrips : nstrips); at += NW) {
        const int strip = at < nstrips ? at : at - nstrips;
        char *const base = reinterpret_cast<char *>(at < nstrips ? M : M2);
        const unsigned rb = (unsigned)(strip * 16) * (unsigned)sizeof(T) + row_off;
        T bv[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const int x = 4 * kk + lk;
            bv[kk] = x < m ? *reinterpret_cast<const T *>(base + ((unsigned)cols[x] * col_bytes + rb)) : T(0);
        }
        typename MF<T>::acc acc[YT];
#pragma unroll
        for (int yt = 0; yt < YT; ++yt) acc[yt] = MF<T>::zero();
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int yt = 0; yt < YT; ++yt)
                acc[yt] = MF<T>::mma(Wl[(4 * kk + lk) * NC + yt * 16 + lr], bv[kk], acc[yt]);
#pragma unroll
        for (int yt = 0; yt < YT; ++yt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int y = yt * 16 + MF<T>::row(lane, v);
                if (y < m) *reinterpret_cast<T *>(base + ((unsigned)cols[y] * col_bytes + rb)) = acc[yt][v];
            }
    }
}

// Rows [row_base, row_base + 16 nstrips) of the 2b columns of block pair k in
// M (G or V), and in M2 when it is not null, <- themselves times W, by NT
// threads; mask = the pair's touched local columns (nonzero).  kOne: one
// matrix and at most one strip per wave (nstrips <= NT / 64), no loop; else W
// is re-read from LDS for every strip.  kLd: LDS row stride of W.
// kUpdateBarriers workgroup barriers.
constexpr int kUpdateBarriers = 2;
template <typename T, int NT, int kLd, bool kOne>
__device__ __forceinline__ void update_rows(const BlockArgsT<T> &a, int k, T *M, T *M2, int row_base, int nstrips,
                                            unsigned long long mask, T *Wl, int *cols, int *tl, int tid)
{
    constexpr int NW = NT / 64;
    const int2 IJ = outer_pair(a, k);
    const int m = __popcll(mask);
    if (m <= 32) {
        // compact list of the touched local columns, in increasing order
        if (tid < kB2 && ((mask >> tid) & 1ull)) {
            const int i = __popcll(mask & ((1ull << tid) - 1ull));
            tl[i] = tid;
            cols[i] = a.rho[local_pos(tid, IJ.x, IJ.y)];
        }
        __syncthreads();
        if (m <= 16)
            update_compact<T, 16, NT>(a, k, M, M2, row_base, nstrips, Wl, cols, tl, m, tid);
        else
            update_compact<T, 32, NT>(a, k, M, M2, row_base, nstrips, Wl, cols, tl, m, tid);
        return;
    }
    // W on its way while the column list is made; the first strip's rows on
    // theirs while W goes to LDS
    typedef T v4 __attribute__((ext_vector_type(4)));
    constexpr int kW4 = kB2 * kB2 / 4 / NT;
    static_assert(kW4 * NT * 4 == kB2 * kB2, "thread count");
    const v4 *Wg = reinterpret_cast<const v4 *>(a.W + (size_t)k * (kB2 * kB2));
    v4 wreg[kW4];
#pragma unroll
    for (int q = 0; q < kW4; ++q) wreg[q] = Wg[tid + q * NT];
    if (tid < kB2) cols[tid] = a.rho[local_pos(tid, IJ.x, IJ.y)];
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    // 32-bit byte offsets from the uniform base (r, ldg <= 16448: below 2^32 bytes).
    // Loads: B(k = x, j = row) = G(row0 + lr, column x = 4kk + lk).
    // Stores: D(i = y, j = row), y = 16yt + MF::row(lane, v).
    const unsigned row_off = (unsigned)(row_base + lr) * (unsigned)sizeof(T);
    const unsigned col_bytes = (unsigned)a.ldg * (unsigned)sizeof(T);
    auto at_matrix = [&](int at) { return reinterpret_cast<char *>(kOne || at < nstrips ? M : M2); };
    auto at_row = [&](int at) {
        return (unsigned)((kOne || at < nstrips ? at : at - nstrips) * 16) * (unsigned)sizeof(T) + row_off;
    };
    auto load = [&](int at, T *bv, const int *cp) {
        const char *base = at_matrix(at);
        const unsigned rb = at_row(at);
#pragma unroll
        for (int kk = 0; kk < 16; ++kk)
            bv[kk] = *reinterpret_cast<const T *>(base + ((unsigned)cp[4 * kk + lk] * col_bytes + rb));
    };
    const int total = !kOne && M2 ? 2 * nstrips : nstrips;
    T bv[16];
    if (wave < total) load(wave, bv, cols);
#pragma unroll
    for (int q = 0; q < kW4; ++q) {
        const int idx = (tid + q * NT) * 4;
        T *const w = Wl + (idx / kB2) * kLd + idx % kB2;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = wreg[q][e];
    }
    __syncthreads();
#pragma unroll 1
    for (int at = wave; at < total; at += kOne ? total : NW) {
        // With several strips, the opaque zero wz keeps the compiler from
        // hoisting the column offsets and the 64 W operands into registers
        // across strips.
        int wz = 0;
        if (!kOne) asm volatile("" : "+v"(wz));
        if (!kOne && at != wave) load(at, bv, cols + wz);
        const T *Wp = Wl + wz + lk * kLd + lr;
        typename MF<T>::acc acc[4];
#pragma unroll
        for (int yt = 0; yt < 4; ++yt) acc[yt] = MF<T>::zero();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk)
#pragma unroll
            for (int yt = 0; yt < 4; ++yt) {
                // A(i = y, k = x) = W(x, y), x = 4kk + lk, y = 16yt + lr
                const T aw = Wp[4 * kk * kLd + yt * 16];
                acc[yt] = MF<T>::mma(aw, bv[kk], acc[yt]);
            }
        const int *cp = cols + wz;
        char *const base = at_matrix(at);
        const unsigned rb = at_row(at);
#pragma unroll
        for (int yt = 0; yt < 4; ++yt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<T *>(base + ((unsigned)cp[yt * 16 + MF<T>::row(lane, v)] * col_bytes + rb)) =
                    acc[yt][v];
    }
}


}  // namespace hsvd
