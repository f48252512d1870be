// Pairwise sweeps of the modified modulus ordering in tiles of 4 x 4 pairs.
//
// At step sigma of a sweep (sigma = r - 1 .. 2 r - 2) every position i meets
// the position j with i + j = sigma (mod r); when sigma is even the two
// positions with 2 i = sigma (mod r) meet each other, i with i + r / 2.  A
// column's partners thus follow one another in increasing order, and pair
// (i, j) needs (i, j - 1) and (i - 1, j) only.  Two runs of four consecutive
// positions, I and J, can therefore do all their pairs in one go, by
// antidiagonals -- 7 steps of up to four pairs -- and the runs themselves meet
// in the same ordering one level up: I and J when I + J = S (mod nb), with the
// two runs 2 I = S (mod nb), r / 2 positions apart, doing the pairs inside
// themselves and the pairs (i, i + r / 2).  Every pair sees the columns that
// the step-by-step order shows it and rounds the same operations, so the
// results are bit-identical to one launch per step.
//
// One launch per S, one workgroup per tile: the columns of I in the registers
// of four waves, one on each SIMD (wave m holds column m of I for all its
// pairs), those of J in LDS.  V's columns only take the tile's rotations and
// have no part in the chain: further workgroups of the next launch apply them,
// a row per thread, all eight columns of the tile in registers.
//
// What bounds it: the chain of the 7 steps -- column from LDS, dot product,
// rotation, update, norms: 250 to 350 instructions of one wave, 1600 cycles a
// step at n = 140, 2550 at n = 1024 -- and 4 us per launch (start, columns in
// and out).  It replaces four launches, each with three dependent trips to
// memory and, at n = 1024, 34 MB moved.  Solves, launches only: n = 129 5.5 ->
// 3.0 ms, n = 301 12.9 -> 6.9, n = 513 29.1 -> 16.8, graded n = 1024 198 ->
// 95 ms, three sweeps of n = 2048 133 -> 62 ms.  Tiles of 8 x 8 (15 steps of
// eight waves, two to a SIMD) took 3.2, 7.1, 17.9 and 94 ms.
#include <algorithm>

#include "pair_device.h"

namespace hsvd {

namespace {

constexpr int kW = kTileW;

// One run of positions [start, start + size).
struct Run {
    int start, size;
};
__device__ __forceinline__ Run run_of(int I, int h, int r)
{
    const int k = I < h ? I : I - h;
    return Run{(I < h ? 0 : r / 2) + k * kW, min(kW, r / 2 - k * kW)};
}

// The tile q of tile step S: the runs I < J (twin: J = I + nb / 2, all pairs
// inside I and inside J and the pairs (i, i + r / 2)), and the antidiagonals
// s0 .. s1 of it that belong to this sweep's part of S (none: s0 > s1).
struct Tile {
    Run I, J;
    bool twin;
    int s0, s1;
};
__device__ __forceinline__ Tile tile_of(int S, int q, int r)
{
    const int h = (r / 2 + kW - 1) / kW, nb = 2 * h, sb = S < nb ? S : S - nb;  // S < 2 nb
    Tile t;
    int i = (sb + 1) / 2 + q, j = sb / 2 - q;
    if ((sb & 1) == 0 && q == 0) j += h;
    i = i >= nb ? i - nb : i;
    j = j < 0 ? j + nb : j;
    const int lo = min(i, j), hi = max(i, j);
    t.I = run_of(lo, h, r);
    t.J = run_of(hi, h, r);
    t.twin = (sb & 1) == 0 && q == 0;
    t.s0 = 0;
    t.s1 = t.I.size + t.J.size - 2;
    // pairs with i + j >= r - 1 come first in a sweep (S = I + J), the others
    // after them (S = I + J + nb); inside a run of the first half all sums are
    // below r - 1, inside one of the second half none is
    const int base = t.I.start + t.J.start;
    if (t.twin) {
        if (2 * lo + nb != S) t.s1 = -1;
    } else if (lo + hi == S) {
        t.s0 = max(0, r - 1 - base);
    } else if (lo + hi + nb == S) {
        t.s1 = min(t.s1, r - 2 - base);
    } else {
        t.s1 = -1;
    }
    return t;
}

// v + v rotated inside the 16-lane rows (mov_dpp: the unrotated value is not
// copied first).
template <int kCtrl>
__device__ __forceinline__ double ror_add(double v)
{
    return v + __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xf, 0xf, false),
                                __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xf, 0xf, false));
}
// a + b after the exchange of a's upper with b's lower half wave: the first
// stage (l ^ 32) of two wave sums at once, a's in the lower half.
__device__ __forceinline__ double halves_add(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// The same for the 16-lane rows (l ^ 16): a's sums in the even rows.
__device__ __forceinline__ double rows_add(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The butterflies (l ^ 32, 16, 8, 4, 2, 1) of the NV waves' sums of the
// per-step kernel: wave v's sum ends in every lane of row 2 (v % 2) + v / 2.
// Inside a row the values repeat with the period of the stage before, so a
// rotation by the stage's distance pairs the same two.
template <int NV>
__device__ __forceinline__ double wave_sums(const double *s)
{
    static_assert(NV == 1 || NV == 2 || NV == 4, "waves of the per-step kernel");
    double v = halves_add(s[0], s[NV == 1 ? 0 : 1]);
    v = rows_add(v, NV == 4 ? halves_add(s[2], s[3]) : v);
    v = ror_add<0x128>(v);
    v = ror_add<0x124>(v);
    v = ror_add<0x122>(v);
    return ror_add<0x121>(v);
}
// Two of them for NV < 4: s's in rows 0 and 2, u's in rows 1 and 3.
template <int NV>
__device__ __forceinline__ double wave_sums2(const double *s, const double *u)
{
    double v = rows_add(halves_add(s[0], s[NV - 1]), halves_add(u[0], u[NV - 1]));
    v = ror_add<0x128>(v);
    v = ror_add<0x124>(v);
    v = ror_add<0x122>(v);
    return ror_add<0x121>(v);
}
// The waves' sums in wave order, as the per-step kernel adds them.
template <int NV>
__device__ __forceinline__ double in_order(double s0, double s1, double s2, double s3)
{
    return NV == 1 ? s0 : (NV == 2 ? s0 + s1 : ((s0 + s1) + s2) + s3);
}

template <int R>
struct TileLds {
    double col[2 * kW][64 * R];  // runs I (twin tiles) and J
    double d[2 * kW][4];         // a column's squared norm: the sums of the per-step kernel's waves, by rows
    double2 prm[kW][kW];  // stored at the end: a store in flight holds up the step's barrier
    unsigned touched;
    unsigned rot[kW], skip[kW];
    double maxt[kW];
    __device__ __forceinline__ double2 d2(int c, int h) const { return *reinterpret_cast<const double2 *>(&d[c][2 * h]); }
    template <int NV>
    __device__ __forceinline__ double norm(int c) const
    {
        return in_order<NV>(d[c][0], d[c][2], d[c][1], d[c][3]);
    }
};
struct VLds {
    double2 prm[kW * kW];
};

// What a wave did.
struct WaveCount {
    unsigned rmask, touched, visits;
    double maxt;
};

// The antidiagonals of a tile, wave m; x: column m of I (not used by a twin
// tile).  kTrig: every pair is trigonometric.
template <int NV, int E, bool kTwin, bool kTrig>
__device__ __forceinline__ WaveCount g_steps(const TileArgs &a, const Tile &t, int m, int lane, double *x,
                                             TileLds<NV * E> &L)
{
    constexpr int R = NV * E;
    const double tol = a.tol, tol2 = tol * tol;
    const bool tol_ok = tol2 >= 0x1p-200 && tol2 <= 1.0;
    WaveCount n{0u, 0u, 0u, 0.0};
    const int nb = m < t.I.size ? t.J.size : 0;  // pairs of this wave
    __builtin_amdgcn_s_setprio(2);  // V's waves may share the compute unit
#pragma unroll 1
    for (int s = t.s0; s <= t.s1; ++s) {
        const int b = s - m;
        if ((unsigned)b < (unsigned)nb) {
            // the pair's columns: slot m of I and b of J; of a twin tile also
            // (m, b) inside I, and (b, m) inside J by the wave of the larger
            int cx = m, cy = kW + b;
            if (kTwin && m < b) cy = b;
            if (kTwin && m > b) {
                cx = kW + b;
                cy = kW + m;
            }
            double *const ly = &L.col[cy][lane], *const lx = &L.col[cx][lane];
            double y[R];
#pragma unroll
            for (int e = 0; e < R; ++e) y[e] = ly[64 * e];
            if (kTwin) {
#pragma unroll
                for (int e = 0; e < R; ++e) x[e] = lx[64 * e];
            }
            const double2 dx0 = L.d2(cx, 0), dx1 = L.d2(cx, 1), dy0 = L.d2(cy, 0), dy1 = L.d2(cy, 1);
            double part[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                part[v] = 0.0;
#pragma unroll
                for (int e = 0; e < E; ++e) part[v] = fma(x[v + NV * e], y[v + NV * e], part[v]);
            }
            const double sums = wave_sums<NV>(part);
            const double aij = in_order<NV>(lane_value(sums, 0), NV > 1 ? lane_value(sums, 32) : 0.0,
                                            NV > 2 ? lane_value(sums, 16) : 0.0, NV > 2 ? lane_value(sums, 48) : 0.0);
            const double aii = in_order<NV>(dx0.x, dx1.x, dx0.y, dx1.y), ajj = in_order<NV>(dy0.x, dy1.x, dy0.y, dy1.y);
            bool trig = true;
            if (!kTrig) {
                const int i = cx < kW ? t.I.start + cx : t.J.start + cx - kW;
                const int j = cy < kW ? t.I.start + cy : t.J.start + cy - kW;
                trig = (i < a.p) == (j < a.p);
            }
            const SlotRotation w = slot_rotation(aii, ajj, aij, trig, true, !kTrig, tol, tol2, tol_ok);
            ++n.visits;
            if (__builtin_amdgcn_readfirstlane(!w.skip && !w.bad)) {
                const double tt = w.t, ht = trig ? -w.t : w.t, c = w.c;
                double nx[NV], ny[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) nx[v] = ny[v] = 0.0;
#pragma unroll
                for (int e = 0; e < R; ++e) {
                    const double xn = fma(ht, y[e], x[e]) * c;
                    const double yn = fma(tt, x[e], y[e]) * c;
                    x[e] = xn;
                    ly[64 * e] = yn;
                    if (kTwin) lx[64 * e] = xn;
                    nx[e % NV] = fma(xn, xn, nx[e % NV]);
                    ny[e % NV] = fma(yn, yn, ny[e % NV]);
                }
                // a row of lanes per entry: rows 0 .. 3 of each norm, or rows 0 and 2 of both
                if constexpr (NV == 4) {
                    const double sx = wave_sums<NV>(nx), sy = wave_sums<NV>(ny);
                    if ((lane & 15) == 0) {
                        L.d[cx][lane >> 4] = sx;
                        L.d[cy][lane >> 4] = sy;
                    }
                } else {
                    const double sxy = wave_sums2<NV>(nx, ny);
                    if ((lane & 15) == 0) L.d[lane & 16 ? cy : cx][(lane >> 4) & 2] = sxy;
                }
                if (lane == 0) L.prm[m][b] = make_double2(tt, trig ? -c : c);
                n.rmask |= 1u << b;
                n.touched |= (1u << cx) | (1u << cy);
                n.maxt = fmax(n.maxt, fabs(tt));
            } else if (!kTrig && !w.skip) {
                if (lane == 0) atomicOr(&a.ctl->rank, 1);
            }
        }
        __syncthreads();
    }
    return n;
}

// The tile's rotations, its columns of G and its part of d.  A column's rows
// 64 (v + NV e) + lane are those of the per-step kernel's wave v, element e.
template <int NV, int E>
__device__ __forceinline__ void g_tile(const TileArgs &a, TileLds<NV * E> &L)
{
    constexpr int R = NV * E;
    const int q = blockIdx.x, r = a.r, lane = threadIdx.x & 63;
    const int m = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Tile t = tile_of(a.S, q, r);
    if (t.s0 > t.s1) {
        if (threadIdx.x < kW) a.rmask[q * kW + threadIdx.x] = 0u;
        return;
    }
    const int nch = a.ldg / 64;  // 64-row pieces of a column
    const bool in_i = m < t.I.size, in_j = m < t.J.size;
    const int pi = t.I.start + (in_i ? m : 0), pj = t.J.start + (in_j ? m : 0);
    double *const gi = a.G + (size_t)a.rho[pi] * a.ldg + lane;
    double *const gj = a.G + (size_t)a.rho[pj] * a.ldg + lane;
    const double di = a.d[pi], dj = a.d[pj];
    // the tile's counters of the sweep so far, read ahead of their update
    int code = 0;
    unsigned nrot = 0u, nskip = 0u;
    double maxt = 0.0;
    if (threadIdx.x == 0) {
        code = a.C[q];
        nrot = a.nrot[q];
        nskip = a.nskip[q];
        maxt = a.maxt[q];
    }
    double x[R];
    {
        double y[R];
#pragma unroll
        for (int e = 0; e < R; ++e) {
            const int k = 64 * min(e, nch - 1);
            const double u = gi[k], w = gj[k];
            x[e] = e < nch ? u : 0.0;
            y[e] = e < nch ? w : 0.0;
        }
#pragma unroll
        for (int e = 0; e < R; ++e) {
            if (t.twin) L.col[m][64 * e + lane] = x[e];
            L.col[kW + m][64 * e + lane] = y[e];
        }
        if (lane < 4) {
            // the first of the sums; the others -0.0, which adds nothing
            L.d[m][lane] = lane == 0 ? di : -0.0;
            L.d[kW + m][lane] = lane == 0 ? dj : -0.0;
        }
        if (threadIdx.x == 0) L.touched = 0u;
    }
    __syncthreads();
    const int i0 = t.I.start, i1 = i0 + t.I.size, j0 = t.J.start, j1 = j0 + t.J.size;
    const bool trig = j1 <= a.p || i0 >= a.p;
    WaveCount n;
    if (t.twin) n = trig ? g_steps<NV, E, true, true>(a, t, m, lane, x, L) : g_steps<NV, E, true, false>(a, t, m, lane, x, L);
    else n = trig ? g_steps<NV, E, false, true>(a, t, m, lane, x, L) : g_steps<NV, E, false, false>(a, t, m, lane, x, L);
    if (lane == 0) {
        a.rmask[q * kW + m] = n.rmask;
        if (n.touched) atomicOr(&L.touched, n.touched);
        L.rot[m] = __popc(n.rmask);
        L.skip[m] = n.visits - __popc(n.rmask);
        L.maxt[m] = n.maxt;
    }
    if (lane < kW && ((n.rmask >> lane) & 1u)) a.prm[(q * kW + m) * kW + lane] = L.prm[m][lane];
    __syncthreads();
    if (threadIdx.x == 0) {
        // launches of a sweep follow one another: tile q's counters are its own
        unsigned rot = 0u;
        double mx = 0.0;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
            rot += L.rot[w];
            nskip += L.skip[w];
            mx = fmax(mx, L.maxt[w]);
        }
        if (rot) a.C[q] = code | rotation_code(mx, a.tthresh);
        a.nrot[q] = nrot + rot;
        a.nskip[q] = nskip;
        a.maxt[q] = fmax(maxt, mx);
    }
    const unsigned all = __builtin_amdgcn_readfirstlane(L.touched);
    if ((all >> m) & 1u) {
#pragma unroll
        for (int e = 0; e < R; ++e)
            if (e < nch) gi[64 * e] = t.twin ? L.col[m][64 * e + lane] : x[e];
        if (lane == 0) a.d[pi] = L.template norm<NV>(m);
    }
    if ((all >> (kW + m)) & 1u) {
#pragma unroll
        for (int e = 0; e < R; ++e)
            if (e < nch) gj[64 * e] = L.col[kW + m][64 * e + lane];
        if (lane == 0) a.d[pj] = L.template norm<NV>(kW + m);
    }
}

// The rotations of tile q of step SV on V, every a.vparts-th run of 64 kW rows,
// pairs in row order, which keeps the order of every column's rotations.
__device__ __forceinline__ void v_tile(const TileArgs &a, int q, int part, VLds &L)
{
    unsigned mask[kW], any = 0u;
#pragma unroll
    for (int m = 0; m < kW; ++m) {
        mask[m] = __builtin_amdgcn_readfirstlane(a.rmask_v[q * kW + m]);
        any |= mask[m];
    }
    if (any == 0u) return;
    const Tile t = tile_of(a.SV, q, a.r);
    if (threadIdx.x < kW * kW) L.prm[threadIdx.x] = a.prm_v[q * kW * kW + threadIdx.x];
    // lane c of a wave fetches column c's number
    const int cl = threadIdx.x & (2 * kW - 1), k = cl & (kW - 1);
    const Run u = cl < kW ? t.I : t.J;
    const int phys = a.rho[u.start + (k < u.size ? k : 0)];
    __syncthreads();
#pragma unroll 1
    for (int row0 = part * 64 * kW; row0 < a.ldg; row0 += a.vparts * 64 * kW) {
        const int row = min(row0 + (int)threadIdx.x, a.ldg - 1);
        double v[2 * kW];
        double *at[2 * kW];
#pragma unroll
        for (int c = 0; c < 2 * kW; ++c) {
            at[c] = a.V + (size_t)__builtin_amdgcn_readlane(phys, c) * a.ldg + row;
            v[c] = *at[c];
        }
        // an opaque zero: the rotations are not kept in registers from run to run
        int z = 0;
        asm volatile("" : "+v"(z));
        unsigned touched = 0u;
        auto turn = [&](int e, int cx, int cy) {
            const double2 w = L.prm[e + z];
            const double tt = w.x, c = fabs(w.y), ht = w.y < 0.0 ? -w.x : w.x;
            const double xn = fma(ht, v[cy], v[cx]) * c;
            const double yn = fma(tt, v[cx], v[cy]) * c;
            v[cx] = xn;
            v[cy] = yn;
            touched |= (1u << cx) | (1u << cy);
        };
        if (t.twin) {
#pragma unroll
            for (int m = 0; m < kW; ++m) {
                if ((mask[m] >> m) & 1u) turn(m * kW + m, m, kW + m);
#pragma unroll
                for (int b = m + 1; b < kW; ++b) {
                    if ((mask[m] >> b) & 1u) turn(m * kW + b, m, b);
                    if ((mask[b] >> m) & 1u) turn(b * kW + m, kW + m, kW + b);
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m < kW; ++m)
#pragma unroll
                for (int b = 0; b < kW; ++b)
                    if ((mask[m] >> b) & 1u) turn(m * kW + b, m, kW + b);
        }
        if (row0 + (int)threadIdx.x < a.ldg)
#pragma unroll
            for (int c = 0; c < 2 * kW; ++c)
                if ((touched >> c) & 1u) *at[c] = v[c];
    }
}

}  // namespace

// Workgroups 0 .. tiles - 1: the tiles of step S (S < 0: none); the others: V's
// tiles of step SV (SV < 0: none), a.vparts workgroups each.
template <int NV, int E>
__global__ __launch_bounds__(64 * kW, 1) void pair_tile_kernel(TileArgs a)
{
    __shared__ union {
        TileLds<NV * E> g;
        VLds v;
    } L;
    const int tiles = (a.r / 2 + kW - 1) / kW;
    if ((int)blockIdx.x < tiles) {
        if (a.S >= 0) g_tile<NV, E>(a, L.g);
    } else if (a.SV >= 0) {
        const int k = blockIdx.x - tiles;
        v_tile(a, k / a.vparts, k % a.vparts, L.v);
    }
}

hipError_t launch_pair_tiles(hipStream_t st, TileArgs a, int step)
{
    const int tiles = tile_count(a.r), steps = tile_steps(a.r);
    const int first = 2 * tiles - 1 - (steps - (2 * tiles + 1));
    double2 *const prm = a.prm;
    unsigned *const rmask = a.rmask;
    const int cur = step & 1;
    a.S = step < steps ? first + step : -1;
    a.SV = a.V && step > 0 ? first + step - 1 : -1;
    a.prm = prm + cur * tiles * kW * kW;
    a.rmask = rmask + cur * tiles * kW;
    a.prm_v = prm + (cur ^ 1) * tiles * kW * kW;
    a.rmask_v = rmask + (cur ^ 1) * tiles * kW;
    a.vparts = std::min(2, (a.ldg + 64 * kW - 1) / (64 * kW));
    const dim3 grid(tiles + (a.SV >= 0 ? tiles * a.vparts : 0)), wg(64 * kW);
    // the waves and elements of the per-step kernel at this height, less the
    // elements that no row has
    const int nch = a.ldg / 64;
    if (nch <= 3) pair_tile_kernel<1, 3><<<grid, wg, 0, st>>>(a);
    else if (nch <= 4) pair_tile_kernel<1, 4><<<grid, wg, 0, st>>>(a);
    else if (nch <= 6) pair_tile_kernel<2, 3><<<grid, wg, 0, st>>>(a);
    else if (nch <= 8) pair_tile_kernel<2, 4><<<grid, wg, 0, st>>>(a);
    else if (nch <= 12) pair_tile_kernel<4, 3><<<grid, wg, 0, st>>>(a);
    else if (nch <= 16) pair_tile_kernel<4, 4><<<grid, wg, 0, st>>>(a);
    else if (nch <= 24) pair_tile_kernel<4, 6><<<grid, wg, 0, st>>>(a);
    else if (nch <= kTileMaxLdg / 64) pair_tile_kernel<4, 8><<<grid, wg, 0, st>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace hsvd
