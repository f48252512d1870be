// Pairwise solves of small orders (r <= 128, modified modulus ordering) in one
// workgroup: set-up, every sweep (Algs. 4.1 - 4.5), the sort, the stop rule
// and the outputs in one launch.
//
// A parallel step of such an order is far too little work for a launch of its
// own: what it cost there was the launch and three dependent trips to memory.
// Here G and V stay in registers.  Lane k of every wave is slot k of the step
// (r / 2 <= 64 slots); the rows are spread over the waves, eight for G and
// seven for V: G's wave w holds rows w + 8 m + 64 e of the slot's two columns.
// So
// - dot products need no lane moves: each wave adds up its rows' products, and
//   the eight partial sums meet in LDS;
// - one wave, with no rows of its own, evaluates all rotations of the step at
//   once, a slot per lane;
// - from step to step every slot keeps one column and passes the other on to
//   the slot before it, around the ring of slots: a one-lane move inside each
//   wave, no barrier;
// - V's waves apply a step's rotations while the next step's are evaluated.
//
// The sums run in the order of the per-step kernel (fma chain over e, then
// the butterfly over 64 rows: l ^ 32, l ^ 16, l ^ 8 inside a wave, l ^ 4, l ^ 2,
// l ^ 1 over the waves), and slot_rotation rounds the operations of
// rotation_params, so the results are bit-identical to the per-step launches.
//
// What bounds it: the dependent chain of a step -- partial sums, eight-way
// sum, rotation (about 95 instructions of one wave), barriers -- up to n = 64
// (2900 cycles a step there, 2230 at n = 16), and the FP64 issue rate of the
// one compute unit at n = 128 (4160 cycles: G's 16 rows per wave and V's 19).
// Whole calls: n = 16 883 us in per-step launches, 167 us here; n = 128 5.35
// ms and 2.08 ms.
#include "pair_device.h"

namespace hsvd {

namespace {

constexpr int kSlots = 64;       // slots at most
constexpr int kGWaves = 8;       // waves that hold G
constexpr int kRotWave = 8;      // the wave that evaluates the rotations
constexpr int kVWave = 9;        // first of the waves that hold V
constexpr int kVWaves = 7;

// Steps of a sweep start on the antidiagonal (slot k: positions k and r - 1 -
// k) every time: after r steps the slots hold the antidiagonal pairs again,
// in reverse slot order (Alg. 4.4), and the sort moves every column anyway.
// In between, slot k's first position moves up to step T = r - 1 - 2 k, where
// it wraps to r/2 - 1 - k; from there on the second one moves.
__device__ __forceinline__ int2 slot_pair(int k, int t, int r)
{
    const int T = r - 1 - 2 * k;
    if (t < T) return make_int2(k + t, r - 1 - k);
    return make_int2(r / 2 - 1 - k, t == T ? r - 1 - k : t + k - r / 2);
}

struct SmallLds {
    double part[3][kGWaves][kSlots];  // partial sums: dot product, the two norms
    double pa[kSlots], pb[kSlots], pc[kSlots];
    double d[kSmallMaxOrder];         // by position
    double dnew[kSmallMaxOrder];
    int rho[kSmallMaxOrder], src[kSmallMaxOrder], rnew[kSmallMaxOrder];
    double row[16][kSmallMaxOrder];  // column moves of one row, per wave
    int stop;
};

// Where a lane stands.  kRing (the number of slots divides 64): the slots are
// repeated across the wave's lanes, and its first lanes are the slots' own.
// Otherwise the last lanes hold the slots, the others none.
template <bool kRing>
struct Lane {
    int slot, base;
    bool act, own;  // has a slot; is the slot's own lane
    __device__ __forceinline__ Lane(int lane, int r)
    {
        const int slots = r / 2;
        base = kRing ? 0 : kSlots - slots;
        slot = kRing ? lane & (slots - 1) : lane - base;
        act = kRing || slot >= 0;
        own = kRing ? lane < slots : slot >= 0;
    }
    // Every slot takes the next slot's value, the last one slot 0's: a
    // rotation of the wave, or a shift with slot 0's value moving in at its
    // end.  (A DPP move costs a wave about 5 cycles, a ds_bpermute of the same
    // word 6 cycles of the compute unit's one LDS pipe.)
    __device__ __forceinline__ int next(int v) const
    {
        if (kRing) return __builtin_amdgcn_update_dpp(v, v, 0x134, 0xf, 0xf, false);  // wave_rol:1
        return __builtin_amdgcn_update_dpp(__builtin_amdgcn_readlane(v, base), v, 0x130, 0xf, 0xf, false);  // wave_shl:1
    }
    __device__ __forceinline__ double next(double v) const
    {
        return __hiloint2double(next(__double2hiint(v)), next(__double2loint(v)));
    }
};

// Eight waves' partial sums in butterfly order (l ^ 4, l ^ 2, l ^ 1).
__device__ __forceinline__ double sum8(const double (*p)[kSlots], int lane)
{
    const double p0 = p[0][lane], p1 = p[1][lane], p2 = p[2][lane], p3 = p[3][lane];
    const double p4 = p[4][lane], p5 = p[5][lane], p6 = p[6][lane], p7 = p[7][lane];
    return ((p0 + p4) + (p2 + p6)) + ((p1 + p5) + (p3 + p7));
}

// a <-> b in the active lanes, one instruction per word.
__device__ __forceinline__ void swap_words(double &a, double &b)
{
    int al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
    asm("v_swap_b32 %0, %1" : "+v"(al), "+v"(bl));
    asm("v_swap_b32 %0, %1" : "+v"(ah), "+v"(bh));
    a = __hiloint2double(ah, al);
    b = __hiloint2double(bh, bl);
}

// R rows of the slots' columns, in one wave: a, the column that moves on, and
// b, the one that stays.
template <int R>
struct Cols {
    double a[R], b[R];

    __device__ __forceinline__ void rotate(double pa, double pb, double c)
    {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const double x = fma(pa, b[q], a[q]) * c;
            b[q] = fma(pb, a[q], b[q]) * c;
            a[q] = x;
            if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // a few rows at a time: no room for more
        }
    }
    // From step t to the next.  kOdd: t is odd, and slot (r - 1 - t) / 2 has
    // reached the step from where its other column moves.
    template <bool kOdd, bool kRing>
    __device__ __forceinline__ void exchange(const Lane<kRing> &l, int t, int r)
    {
        if (kOdd) {
            if (l.slot == (r - 1 - t) / 2) {
#pragma unroll
                for (int q = 0; q < R; ++q) swap_words(a[q], b[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) a[q] = l.next(a[q]);
    }
    // every column from position `from` to the first step's slots
    template <bool kRing>
    __device__ __forceinline__ void reorder(SmallLds &L, int wave, const Lane<kRing> &l, int from, int r)
    {
        const bool act = l.act, aj = from > r - 1 - 2 * l.slot;
        const int2 f = slot_pair(l.slot, from, r), to = slot_pair(l.slot, 0, r);
        const int pa = aj ? f.y : f.x, pb = aj ? f.x : f.y;
        const int s0 = act ? L.src[to.x] : 0, s1 = act ? L.src[to.y] : 0;
        double *const buf = L.row[wave];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (act) {
                buf[pa] = a[q];
                buf[pb] = b[q];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (act) {
                a[q] = buf[s0];
                b[q] = buf[s1];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    // out[:, c] for the slots' columns, divided by sa and sb when kDiv; this
    // wave's rows are row0 + step q
    template <bool kDiv, int kStep, bool kRing>
    __device__ __forceinline__ void store(const SmallLds &L, double *out, int ld, int n, int r, const Lane<kRing> &l,
                                          int row0) const
    {
        if (!l.own || !out) return;
        const int2 ij = slot_pair(l.slot, 0, r);
        const int ca = L.rho[ij.x], cb = L.rho[ij.y];
        const double sa = kDiv ? sqrt(L.d[ij.x]) : 1.0, sb = kDiv ? sqrt(L.d[ij.y]) : 1.0;
        double *const oa = out + (size_t)min(ca, n - 1) * ld + row0, *const ob = out + (size_t)min(cb, n - 1) * ld + row0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (row0 + kStep * q >= n) continue;
            if (ca < n) oa[kStep * q] = kDiv ? a[q] / sa : a[q];
            if (cb < n) ob[kStep * q] = kDiv ? b[q] / sb : b[q];
        }
    }
};

// Sum over a G wave's rows w + 8 m + 64 e (q = m + NM e) of term(q, .): fma
// chain over e in [E0, E), then l ^ 32, l ^ 16, l ^ 8.
template <int NM, int E0, int E, typename F>
__device__ __forceinline__ double tree(F term)
{
    double s[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        s[m] = 0.0;
#pragma unroll
        for (int e = E0; e < E; ++e) s[m] = term(e * NM + m, s[m]);
    }
    if constexpr (NM == 8) return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
    else if constexpr (NM == 4) return (s[0] + s[2]) + (s[1] + s[3]);
    else return s[0] + s[1];
}

// The waves' loops; every wave meets the same barriers.  Barriers of a solve:
// two per 64 rows (set-up norms) and one, the sort (two), then per sweep one,
// three per step (rotations out, norms in, dot products in), one, and the
// sort's two.

// Stable sort of the two sign segments (Alg. 4.1) by the first waves' threads
// tid < r: src, and d and rho in the new order.
__device__ __forceinline__ void sort_positions(const SmallArgs &g, SmallLds &L, int tid)
{
    const int r = g.r, p = g.p;
    if (tid < r) {
        int dst = tid;
        if (g.sort) {
            const long long kq = sort_key(L.d[tid]);
            const bool pos = tid < p;
            const int lo = pos ? 0 : p, hi = pos ? p : r;
            int cnt = 0;
            for (int u = lo; u < hi; ++u) {
                const long long kv = sort_key(L.d[u]);
                const bool before = pos ? (kv > kq) : (kv < kq);
                cnt += (before || (kv == kq && u < tid)) ? 1 : 0;
            }
            dst = lo + cnt;
        }
        L.src[dst] = tid;
        L.dnew[dst] = L.d[tid];
        L.rnew[dst] = L.rho[tid];
    }
    role_barrier();
    if (tid < r) {
        L.d[tid] = L.dnew[tid];
        L.rho[tid] = L.rnew[tid];
    }
}

template <int NM, int E, bool kRing>
__device__ __forceinline__ void g_wave(const SmallArgs &g, SmallLds &L, int wave, int lane)
{
    constexpr int R = NM * E;
    const int r = g.r, n = g.n;
    const Lane<kRing> l(lane, r);
    Cols<R> x;
    {
        // the columns of the first step, bordered (eq. 4.1); lanes without a
        // slot (whose pair means nothing) hold zeros and read nothing
        const bool act = l.act;
        const int2 ij = slot_pair(l.slot, 0, r);
        const int ca = act ? ij.x : n, cb = act ? ij.y : n;
        const double *const ga = g.G + (size_t)min(ca, n - 1) * g.lda + wave;
        const double *const gb = g.G + (size_t)min(cb, n - 1) * g.lda + wave;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int at = 8 * (q % NM) + 64 * (q / NM), row = wave + at;
            double va = act && row == ca ? 1.0 : 0.0, vb = act && row == cb ? 1.0 : 0.0;
            if (ca < n) va = row < n ? ga[at] : 0.0;
            if (cb < n) vb = row < n ? gb[at] : 0.0;
            x.a[q] = va;
            x.b[q] = vb;
        }
    }
    // d = diag(G^T G): rows 0 .. 63 and 64 .. 127 summed on their own, as the
    // set-up of the other paths does
    auto sq_a = [&](int q, double s) { return fma(x.a[q], x.a[q], s); };
    auto sq_b = [&](int q, double s) { return fma(x.b[q], x.b[q], s); };
    auto dot = [&](int q, double s) { return fma(x.a[q], x.b[q], s); };
    L.part[1][wave][lane] = tree<NM, 0, 1>(sq_a);
    L.part[2][wave][lane] = tree<NM, 0, 1>(sq_b);
    role_barrier();
    role_barrier();
    if (E > 1) {
        L.part[1][wave][lane] = tree<NM, E - 1, E>(sq_a);
        L.part[2][wave][lane] = tree<NM, E - 1, E>(sq_b);
        role_barrier();
        role_barrier();
    }
    role_barrier();
    int from = 0;
    for (;;) {
        sort_positions(g, L, 64 * wave + lane);
        x.reorder(L, wave, l, from, r);
        role_barrier();
        if (L.stop) break;
        L.part[0][wave][lane] = tree<NM, 0, E>(dot);
        role_barrier();
        auto rotate = [&] {
            role_barrier();
            x.rotate(L.pa[lane], L.pb[lane], L.pc[lane]);
            L.part[1][wave][lane] = tree<NM, 0, E>(sq_a);
            L.part[2][wave][lane] = tree<NM, 0, E>(sq_b);
            role_barrier();
        };
        auto dots = [&] {
            L.part[0][wave][lane] = tree<NM, 0, E>(dot);
            role_barrier();
        };
        for (int t = 0; t < r - 2; t += 2) {
            rotate();
            x.template exchange<false>(l, t, r);
            dots();
            rotate();
            x.template exchange<true>(l, t + 1, r);
            dots();
        }
        rotate();
        x.template exchange<false>(l, r - 2, r);
        dots();
        rotate();
        role_barrier();
        role_barrier();
        from = r - 1;
    }
    // U = G Sigma^{-1}
    if constexpr (E == 1) {
        x.template store<true, 8>(L, g.U, g.ldu, n, r, l, wave);
    } else {
        Cols<NM> h;
#pragma unroll
        for (int e = 0; e < E; ++e) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                h.a[m] = x.a[e * NM + m];
                h.b[m] = x.b[e * NM + m];
            }
            h.template store<true, 8>(L, g.U, g.ldu, n, r, l, wave + 64 * e);
        }
    }
}

template <int E, bool kRing>
__device__ __forceinline__ void rotation_wave(const SmallArgs &g, SmallLds &L, int lane)
{
    const int r = g.r, slots = r / 2;
    const Lane<kRing> l(lane, r);
    const bool act = l.act;
    const int T = r - 1 - 2 * l.slot;  // the slot's second position moves from this step on
    double da = 0.0, db = 0.0;       // squared norms of the slot's columns
#pragma unroll
    for (int e = 0; e < E; ++e) {
        role_barrier();
        const double sa = sum8(L.part[1], lane), sb = sum8(L.part[2], lane);
        da = e ? da + sa : sa;
        db = e ? db + sb : sb;
        role_barrier();
    }
    const int2 first = slot_pair(l.slot, 0, r), last = slot_pair(l.slot, r - 1, r);
    if (act) {
        L.d[first.x] = da;
        L.d[first.y] = db;
    }
    const int inval = __ballot(act && (!isfinite(da) || !isfinite(db))) != 0ull ? 1 : 0;
    int rank = __ballot(act && ((isfinite(da) && !(da > 0.0)) || (isfinite(db) && !(db > 0.0)))) != 0ull ? 1 : 0;
    int sweeps = 0, code = 0;
    unsigned long long nrot = 0;
    double maxt = 0.0;
    if (lane == 0) L.stop = inval || rank || g.max_sweeps < 1;
    role_barrier();
    const double tol = g.tol, tol2 = tol * tol;
    const bool tol_ok = tol2 >= 0x1p-200 && tol2 <= 1.0;
    __builtin_amdgcn_s_setprio(2);
    for (;;) {
        role_barrier();
        role_barrier();
        if (L.stop) break;
        da = act ? L.d[first.x] : 1.0;
        db = act ? L.d[first.y] : 1.0;
        int nr = 0, bad = 0;
        maxt = 0.0;
        bool aj = false;  // a is the pair's second column
        bool trig = !act || (first.x < g.p) == (first.y < g.p);
        bool any_hyp = __ballot(!trig) != 0ull;
        double di = da, dj = db;
        role_barrier();
#pragma unroll 1
        for (int t = 0; t < r; ++t) {
            const double aij = sum8(L.part[0], lane);
            const SlotRotation s = slot_rotation(di, dj, aij, trig, act, any_hyp, tol, tol2, tol_ok);
            const bool rot = act && !s.skip && !s.bad;
            const double tt = rot ? s.t : 0.0, ht = trig ? -tt : tt;
            L.pa[lane] = aj ? tt : ht;
            L.pb[lane] = aj ? ht : tt;
            L.pc[lane] = rot ? s.c : 1.0;
            role_barrier();
            nr += __popcll(__ballot(rot && l.own));
            bad |= __ballot(act && !s.skip && s.bad) != 0ull ? 1 : 0;
            maxt = fmax(maxt, fabs(tt));
            aj = t + 1 > T;
            const int2 next = slot_pair(l.slot, t + 1, r);
            trig = !act || (next.x < g.p) == (next.y < g.p);
            any_hyp = __ballot(!trig) != 0ull;
            role_barrier();
            // the norms after this step's rotations, then its exchange
            const double na = sum8(L.part[1], lane), nb = sum8(L.part[2], lane);
            da = rot ? na : da;
            db = rot ? nb : db;
            if (t + 1 < r) {
                const bool flip = t == T;
                const double out = flip ? db : da;
                db = flip ? da : db;
                da = l.next(out);
            }
            di = aj ? db : da;
            dj = aj ? da : db;
            role_barrier();
        }
        if (act) {
            const bool after = r - 1 > T;
            L.d[after ? last.y : last.x] = da;
            L.d[after ? last.x : last.y] = db;
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) maxt = fmax(maxt, __shfl_xor(maxt, m, 64));
        // eq. (4.2) codes of the sweep's rotations, OR-ed
        code = nr > 0 ? (maxt > g.tthresh ? 3 : 1) : 0;
        rank = bad;
        nrot += (unsigned long long)nr;
        ++sweeps;
        if (lane == 0) L.stop = rank || (code & 2) == 0 || sweeps >= g.max_sweeps;
        role_barrier();
    }
    __builtin_amdgcn_s_setprio(0);
    if (lane == 0) {
        Ctl c;
        c.code = code;
        c.rank = rank;
        c.inval = inval;
        c.sweeps = sweeps;
        c.rot = nrot;
        c.skip = (unsigned long long)sweeps * r * slots - nrot;
        c.act = 0;
        c.tcol = 0;
        c.maxt = maxt;
        c.nsres = 0.0;
        *g.ctl = c;
    }
    // Sigma, lambda = sigma^2 j, perm (Sec. 2)
    for (int q = lane; q < r; q += 64) {
        const int c = L.rho[q];
        if (c >= g.n) continue;
        const double dq = L.d[q];
        g.sigma[c] = sqrt(dq);
        if (g.lambda) g.lambda[c] = q < g.p ? dq : -dq;
        if (g.perm) {
            int real = 0;  // border columns are dropped
            for (int u = 0; u < q; ++u) real += L.rho[u] < g.n ? 1 : 0;
            g.perm[real] = c;
        }
    }
}

template <int R, int E, bool kRing>
__device__ __forceinline__ void v_wave(const SmallArgs &g, SmallLds &L, int wave, int lane)
{
    constexpr int kRows = (8 * R + kVWaves - 1) / kVWaves;
    const int r = g.r, row0 = wave - kVWave;
    const Lane<kRing> l(lane, r);
    Cols<kRows> x;
    const int2 ij = slot_pair(l.slot, 0, r);
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
        x.a[q] = l.act && row0 + kVWaves * q == ij.x ? 1.0 : 0.0;
        x.b[q] = l.act && row0 + kVWaves * q == ij.y ? 1.0 : 0.0;
    }
    for (int e = 0; e < 2 * E + 1; ++e) role_barrier();
    int from = 0;
    for (;;) {
        role_barrier();
        x.reorder(L, wave, l, from, r);
        role_barrier();
        if (L.stop) break;
        role_barrier();
        // a step's rotations are applied while the next one's are evaluated
        auto rotate = [&] {
            role_barrier();
            const double pa = L.pa[lane], pb = L.pb[lane], pc = L.pc[lane];
            role_barrier();
            role_barrier();
            x.rotate(pa, pb, pc);
        };
        for (int t = 0; t < r - 2; t += 2) {
            rotate();
            x.template exchange<false>(l, t, r);
            rotate();
            x.template exchange<true>(l, t + 1, r);
        }
        rotate();
        x.template exchange<false>(l, r - 2, r);
        rotate();
        role_barrier();
        from = r - 1;
    }
    x.template store<false, kVWaves>(L, g.V, g.ldv, g.n, r, l, row0);
}

}  // namespace

// kV: V accumulated; kRing: r / 2 divides 64.
template <int NM, int E, bool kV, bool kRing>
__global__ __launch_bounds__(kV ? 1024 : 576) void pair_small_kernel(SmallArgs g)
{
    __shared__ SmallLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < g.r) L.rho[tid] = tid;
    if (wave < kGWaves)
        g_wave<NM, E, kRing>(g, L, wave, lane);
    else if (wave == kRotWave)
        rotation_wave<E, kRing>(g, L, lane);
    else
        v_wave<NM * E, E, kRing>(g, L, wave, lane);
}

template <int NM, int E, bool kRing>
static hipError_t small_as(hipStream_t st, const SmallArgs &a)
{
    if (a.want_v)
        pair_small_kernel<NM, E, true, kRing><<<1, 1024, 0, st>>>(a);
    else
        pair_small_kernel<NM, E, false, kRing><<<1, 576, 0, st>>>(a);
    return hipGetLastError();
}

template <int NM, int E>
static hipError_t small_as(hipStream_t st, const SmallArgs &a)
{
    return kSlots % (a.r / 2) == 0 ? small_as<NM, E, true>(st, a) : small_as<NM, E, false>(st, a);
}

hipError_t launch_pair_small(hipStream_t st, const SmallArgs &a)
{
    if (a.r < 2 || a.r > kSmallMaxOrder || (a.r & 1) || a.n < 1 || a.n > a.r || a.lda < a.n) return hipErrorInvalidValue;
    if (a.r <= 16) return small_as<2, 1>(st, a);
    if (a.r <= 32) return small_as<4, 1>(st, a);
    if (a.r <= 64) return small_as<8, 1>(st, a);
    return small_as<8, 2>(st, a);
}

}  // namespace hsvd
