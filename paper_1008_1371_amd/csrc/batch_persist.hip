// Batched solves in one persistent launch.
//
// Each workgroup takes whole problems from a device work queue (problem
// indices ordered by n, largest first, so that the long solves start first
// and the short ones fill in at the end) and runs the complete block-oriented
// solve of each one on its own: set-up and bordering (eq. 4.1), the kept
// diagonal and the sort (Alg. 4.1), then sweeps of outer steps -- for every
// block pair the Gram on MFMA, the inner rotations (eqs. 2.2-2.5), the
// update of the pair's columns of G and V on MFMA -- each sweep closed by
// fresh column norms, the sort and the stop rule of eq. (4.2), decided in the
// workgroup; finally Sigma, U, lambda and V into the caller's packed outputs.
// No host round trip and no other launch happens between the first problem
// and the last.
//
// A workgroup holds one, two or four groups of 256 threads, each with a block
// pair of the outer step; whatever the width, 16 waves share a compute unit:
// four problems side by side, whose phases interleave (while one runs the
// latency-bound inner solve the others keep the matrix cores busy), or one
// problem with its (up to four) pairs at a time, which then takes a third of
// the time.  What bounds it, at n = 256, FP64, 88 outer steps: one problem of
// 1024 threads per compute unit spends 3.5 ms on Grams, 4.4 on inner solves
// and 6.3 on updates (16.1 in all), of which 7.0 are the matrix cores' time;
// four problems of 256 threads take 12.7 ms per problem.  The earlier form --
// all threads on one pair, the pairs one after the other, two workgroups of
// 256 threads per compute unit -- took 18 ms per problem and compute unit.
//
// The building blocks are those of the per-launch kernels (block_device.h),
// called with the same arguments and 256 threads per block pair (one row
// split), and the set-up, norm, sort and stop-rule steps repeat the grouped
// batched path's arithmetic in the same order: for the same problems the
// results are bit-identical to it.
//
// Mixed precision runs the whole mixed solve of a problem in its workgroup
// too: FP32 block sweeps on FP32 copies (the same building blocks with
// T = float) until the problem's own switch rule, the Newton-Schulz
// J-re-orthogonalisation of V on FP64 MFMA inside the workgroup, G1 = G X,
// then the FP64 sweeps (or, after a rank flag in FP32 or a residual above
// the accepted bound, the FP64 sweeps from G).
//
// Each workgroup works in a slot of device memory of its own (working copies
// of G and V, partial Grams, W, the kept diagonal, rho, stepper state and
// counters; FP32 copies and FP64 product scratch for mixed precision), sized
// for the largest order the kernel takes (n <= 256).
#include "block_device.h"
#include "gemm_device.h"

namespace hsvd {

namespace {

constexpr int kPMaxR = kPersistMaxOrder;       // largest bordered order
constexpr int kPMaxPairs = kPMaxR / kB2;        // block pairs per step at most
constexpr int kPUpdLd = UpdCfg<double>::ld, kPUpdLd32 = UpdCfg<float>::ld;  // LDS row strides of W in the update
constexpr int kPTile = 64;                      // tile of the re-orthogonalisation's products

// LDS of one group of 256 threads: the phases of a block pair run one after
// the other, so they share one area.
union GroupLds {
    CircleLds circle;
    CrossLds<double> cross;
    CrossLds<float> cross32;
    gemm::GemmLds<kPTile> gemm;
    double red[kGramRed];
    struct {
        double Wl[kB2 * kPUpdLd];
        int cols[kB2];
        int tl[kB2];
    } upd;
};

// LDS of a workgroup of GR groups.
template <int GR>
union PersistLds {
    GroupLds group[GR];
    double red[4 * GR];
    struct {
        long long key[kPMaxR];
        double dv[kPMaxR];
        int val[kPMaxR];
    } sort;
    double colsum[4][kPMaxR];
};

// The workgroup's LDS and the block pair arguments of the problem it works
// on.  The phases below are separate (not inlined) functions that reach both
// by name: compiled as one function, the whole solve kept so many values live
// at once that it no longer fitted the registers of four waves per SIMD; as
// calls, each phase is allocated on its own.
__shared__ PersistLds<1> g_lds1;
__shared__ PersistLds<2> g_lds2;
__shared__ PersistLds<4> g_lds4;
template <int GR>
__device__ __forceinline__ PersistLds<GR> &lds()
{
    if constexpr (GR == 1) return g_lds1;
    else if constexpr (GR == 2) return g_lds2;
    else return g_lds4;
}
__shared__ int g_live;  // some cross pair of the workgroup's block pairs fails the skip test
// raw storage: the argument struct has default member initialisers
__shared__ __align__(16) unsigned char g_args[sizeof(BlockArgsT<double>)];

__shared__ __align__(16) unsigned char g_args32[sizeof(BlockArgsT<float>)];
__shared__ __align__(16) unsigned char g_gemm[sizeof(GemmArgs)];

__device__ __forceinline__ BlockArgsT<double> &pargs() { return *reinterpret_cast<BlockArgsT<double> *>(g_args); }
__device__ __forceinline__ BlockArgsT<float> &pargs32() { return *reinterpret_cast<BlockArgsT<float> *>(g_args32); }
__device__ __forceinline__ GemmArgs &pgemm() { return *reinterpret_cast<GemmArgs *>(g_gemm); }

// A workgroup is GR groups of 256 threads (GR 1, 2 or 4), each with one block
// pair of the outer step at a time: the inner solve of a pair is a serial
// chain that a few waves fill, so further threads work on further pairs.  The
// groups pass the same workgroup barriers; one without a pair only those.
__device__ __forceinline__ int group_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8); }
// The thread's index in its group.  Group g starts its waves g places further
// on, so that the rotation waves of the groups (the first of each) sit on
// different SIMDs.
__device__ __forceinline__ int group_tid() { return ((int)threadIdx.x - 64 * group_index()) & 255; }
template <int N>
__device__ __forceinline__ void idle_barriers()
{
#pragma unroll
    for (int u = 0; u < N; ++u) __syncthreads();
}

template <typename T>
__device__ __forceinline__ BlockArgsT<T> &args_of();
template <>
__device__ __forceinline__ BlockArgsT<double> &args_of<double>()
{
    return pargs();
}
template <>
__device__ __forceinline__ BlockArgsT<float> &args_of<float>()
{
    return pargs32();
}
template <typename T>
__device__ __forceinline__ CrossLds<T> &cross_of(GroupLds &L)
{
    if constexpr (sizeof(T) == 8) return L.cross;
    else return L.cross32;
}

// The phases of an outer step for block pairs q0 .. q0 + GR - 1 (of `pairs`).
template <typename T, int GR>
__device__ __noinline__ void phase_gram(int q0, int pairs)
{
    const int g = group_index(), q = __builtin_amdgcn_readfirstlane(q0) + g;
    if (q < __builtin_amdgcn_readfirstlane(pairs))
        gram_pair<T>(args_of<T>(), q, 0, reinterpret_cast<T *>(lds<GR>().group[g].red), group_tid());
    else
        idle_barriers<kGramBarriers>();
}
template <typename T, int GR>
__device__ __noinline__ void phase_circle(int q0, int pairs)
{
    const int g = group_index(), q = __builtin_amdgcn_readfirstlane(q0) + g;
    if (q < __builtin_amdgcn_readfirstlane(pairs))
        inner_circle_pair<T, 256, true>(args_of<T>(), q, lds<GR>().group[g].circle, group_tid());
    else
        inner_circle_idle();
}
template <typename T, int GR>
__device__ __noinline__ void phase_cross(int q0, int pairs)
{
    const int g = group_index(), q = __builtin_amdgcn_readfirstlane(q0) + g;
    if (q < __builtin_amdgcn_readfirstlane(pairs))
        inner_cross_pair<T, 256>(args_of<T>(), q, cross_of<T>(lds<GR>().group[g]), g_live, group_tid());
    else
        inner_cross_idle(g_live);
}
template <typename T, int GR>
__device__ __noinline__ void phase_update(int q0, int pairs)
{
    const BlockArgsT<T> &a = args_of<T>();
    const int g = group_index(), q = __builtin_amdgcn_readfirstlane(q0) + g;
    const unsigned long long mask = q < __builtin_amdgcn_readfirstlane(pairs) ? a.active[q] : 0ull;
    if (__builtin_amdgcn_readfirstlane(mask != 0ull)) {
        GroupLds &L = lds<GR>().group[g];
        update_rows<T, 256, sizeof(T) == 8 ? kPUpdLd : kPUpdLd32, false>(
            a, q, a.G, a.V, 0, a.ldg / 16, mask, reinterpret_cast<T *>(L.upd.Wl), L.upd.cols, L.upd.tl, group_tid());
    } else {
        idle_barriers<kUpdateBarriers>();
    }
}

// One outer step.
template <typename T, int GR>
__device__ __forceinline__ void outer_step(int pairs, bool first)
{
    for (int q0 = 0; q0 < pairs; q0 += GR) {
        phase_gram<T, GR>(q0, pairs);
        __syncthreads();
        if (first)
            phase_circle<T, GR>(q0, pairs);
        else
            phase_cross<T, GR>(q0, pairs);
        __syncthreads();
        phase_update<T, GR>(q0, pairs);
        __syncthreads();
    }
}

// One r x r FP64 product of the re-orthogonalisation, C = op(A) S B
// (arguments in pgemm(); S = diag(+1 x p, -1 x (r - p)) on the rows of B when
// SGN), tile by tile with the grid-wide product kernel's tile code
// (gemm_device.h), GR tiles at a time: the same arithmetic as the grouped
// launches' products.  SYM: the tiles on and above the diagonal, each written
// to both triangles.
template <bool TA, bool SGN, bool SYM, int GR>
__device__ __noinline__ void phase_gemm()
{
    const GemmArgs &a = pgemm();
    const int tiles = __builtin_amdgcn_readfirstlane(a.M) / kPTile, g = group_index();
    const int total = SYM ? tiles * (tiles + 1) / 2 : tiles * tiles;
    for (int i0 = 0; i0 < total; i0 += GR) {
        const int i = i0 + g;
        if (i < total) {
            int tm = i % tiles, tn = i / tiles;
            if (SYM) {
                tn = 0;
                for (int left = i; left > tn; ++tn) left -= tn + 1;
                tm = i - tn * (tn + 1) / 2;
            }
            gemm::gemm_tile<TA, SGN, SYM, kPTile>(a, 0, 0, 0, tm, tn, lds<GR>().group[g].gemm, group_tid());
        } else {
            for (int u = 0; u <= __builtin_amdgcn_readfirstlane(a.K) / gemm::kTK; ++u) __syncthreads();
        }
    }
    __syncthreads();
}

// Byte offsets of the parts of a slot.
struct SlotLayout {
    size_t G, V, P, W, d, rho, S, C, nrot, nskip, nact, ntc, maxt, active, ctl, G32, V32, T1, T2, bytes;
};

__host__ __device__ inline SlotLayout slot_layout(bool mixed)
{
    SlotLayout s;
    size_t o = 0;
    auto take = [&o](size_t bytes) {
        const size_t at = o;
        o = (o + bytes + 255) / 256 * 256;
        return at;
    };
    const size_t mat = sizeof(double) * (size_t)kPMaxR * kPMaxR, bb = sizeof(double) * kB2 * kB2;
    s.G = take(mat);
    s.V = take(mat);
    s.P = take(bb * kPMaxPairs);
    s.W = take(bb * kPMaxPairs);
    s.d = take(sizeof(double) * kPMaxR);
    s.rho = take(sizeof(int) * kPMaxR);
    s.S = take(sizeof(int4) * kPMaxPairs);
    s.C = take(sizeof(int) * kPMaxPairs);
    s.nrot = take(sizeof(unsigned) * kPMaxPairs);
    s.nskip = take(sizeof(unsigned) * kPMaxPairs);
    s.nact = take(sizeof(unsigned) * kPMaxPairs);
    s.ntc = take(sizeof(unsigned) * kPMaxPairs);
    s.maxt = take(sizeof(double) * kPMaxPairs);
    s.active = take(sizeof(unsigned long long) * kPMaxPairs);
    s.ctl = take(sizeof(Ctl));
    // mixed precision: FP32 working copies, FP64 product scratch
    const size_t mat32 = mixed ? sizeof(float) * (size_t)kPMaxR * kPMaxR : 0;
    s.G32 = take(mat32);
    s.V32 = take(mat32);
    s.T1 = take(mixed ? mat : 0);
    s.T2 = take(mixed ? mat : 0);
    s.bytes = o;
    return s;
}

// d[q] = ||G[:, rho[q]]||^2 for q < r: a group per column, its thread `row`
// squares its entry, the waves add in butterfly order, the four wave sums are
// added in wave order (the order of the grouped path's norm kernel for
// ldg <= 256 rows).
template <int GR, typename T>
__device__ __forceinline__ void persist_colnorm(const T *G, int ldg, int r, const int *rho, bool init,
                                                double *d, PersistLds<GR> &L)
{
    const int row = threadIdx.x & 255, lane = row & 63, wave = row >> 6;
    for (int q = group_index(); q < r; q += GR) {
        const int c = init ? q : rho[q];
        const double x = row < ldg ? (double)G[(size_t)c * ldg + row] : 0.0;  // ldg <= 256
        const double s = wave_sum(fma(x, x, 0.0));
        if (lane == 0) L.colsum[wave][q] = s;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < r; q += 256 * GR) {
        double s = L.colsum[0][q];
#pragma unroll
        for (int w = 1; w < 4; ++w) s += L.colsum[w][q];
        d[q] = s;
    }
    __syncthreads();
}

// Stable sort of positions [0, p) by d decreasing and [p, r) by d increasing,
// rho carried along (as the grouped path's sort).
template <int GR>
__device__ __forceinline__ void persist_sort(double *d, int *rho, int r, int p, PersistLds<GR> &L)
{
    const int q = threadIdx.x;
    if (q < r) {
        L.sort.dv[q] = d[q];
        L.sort.key[q] = sort_key(L.sort.dv[q]);
        L.sort.val[q] = rho[q];
    }
    __syncthreads();
    if (q < r) {
        const long long kq = L.sort.key[q];
        const bool pos = q < p;
        const int lo = pos ? 0 : p, hi = pos ? p : r;
        int cnt = 0;
        for (int u = lo; u < hi; ++u) {
            const long long kv = L.sort.key[u];
            const bool before = pos ? (kv > kq) : (kv < kq);
            cnt += (before || (kv == kq && u < q)) ? 1 : 0;
        }
        d[lo + cnt] = L.sort.dv[q];
        rho[lo + cnt] = L.sort.val[q];
    }
    __syncthreads();
}

// One problem, by the whole workgroup; A is the LDS copy of its block pair
// arguments that the phases read.
template <int GR>
__device__ void persist_solve(const PersistArgs &pa, int z, char *slot, PersistLds<GR> &L, BlockArgsT<double> &A)
{
    constexpr int NT = 256 * GR;
    const int tid = threadIdx.x;
    const SlotLayout sl = slot_layout(pa.mixed != 0);
    const int n = pa.n[z], p = pa.p[z];
    const int r = (n + kB2 - 1) / kB2 * kB2, ldg = r, nb = r / kB, pairs = nb / 2;
    const int steps_per_sweep = pa.ordering == HSVD_ORD_MODMOD ? nb : nb - 1;
    const double tol = pa.tol > 0.0 ? pa.tol : 1e-15 * n;
    const double tth = pa.tthresh > 0.0 ? pa.tthresh : sqrt(tol) / 2.0;
    double *G = reinterpret_cast<double *>(slot + sl.G);
    // the mixed path carries V through its FP32 phase even when it is not returned
    double *V = (pa.want_v || pa.mixed) ? reinterpret_cast<double *>(slot + sl.V) : nullptr;
    double *d = reinterpret_cast<double *>(slot + sl.d);
    int *rho = reinterpret_cast<int *>(slot + sl.rho);
    int4 *S = reinterpret_cast<int4 *>(slot + sl.S);
    Ctl *ctl = reinterpret_cast<Ctl *>(slot + sl.ctl);

    if (tid == 0) {
        BlockArgsT<double> a;
        a.G = G;
        a.V = V;
        a.ldg = ldg;
        a.r = r;
        a.p = p;
        a.nb = nb;
        a.rho = rho;
        a.S_in = S;
        a.S_out = S;
        a.ordering = pa.ordering;
        a.step = 0;
        a.partial = reinterpret_cast<double *>(slot + sl.P);
        a.splits = 1;
        a.rows_per_split = ldg;
        a.W = reinterpret_cast<double *>(slot + sl.W);
        a.active = reinterpret_cast<unsigned long long *>(slot + sl.active);
        a.C = reinterpret_cast<int *>(slot + sl.C);
        a.nrot = reinterpret_cast<unsigned *>(slot + sl.nrot);
        a.nskip = reinterpret_cast<unsigned *>(slot + sl.nskip);
        a.nact = reinterpret_cast<unsigned *>(slot + sl.nact);
        a.ntc = reinterpret_cast<unsigned *>(slot + sl.ntc);
        a.maxt = reinterpret_cast<double *>(slot + sl.maxt);
        a.ctl = ctl;
        a.tol = tol;
        a.tthresh = tth;
        a.inner_sweeps = 0;
        a.nprob = 1;
        A = a;
    }
    __syncthreads();
    const BlockArgsT<double> &a = A;

    // set-up: bordered working copy (eq. 4.1), V = I, counters
    const double *src = pa.Gin + pa.off[z];
    for (int e = tid; e < r * ldg; e += NT) {
        const int c = e / ldg, row = e - c * ldg;
        double v;
        if (c < n)
            v = row < n ? src[(size_t)c * n + row] : 0.0;
        else
            v = row == c ? 1.0 : 0.0;
        G[e] = v;
        if (V) V[e] = row == c ? 1.0 : 0.0;
    }
    if (tid < pairs) {
        a.C[tid] = 0;
        a.nrot[tid] = 0;
        a.nskip[tid] = 0;
        a.nact[tid] = 0;
        a.ntc[tid] = 0;
        a.maxt[tid] = 0.0;
        a.active[tid] = ~0ull;  // no pair before the first
        if (pa.ordering == HSVD_ORD_MODMOD) S[tid] = modmod_start(tid, nb);
    }
    if (tid == 0) {
        ctl->code = 0;
        ctl->rank = 0;
        ctl->inval = 0;
        ctl->rot = 0;
        ctl->skip = 0;
        ctl->act = 0;
        ctl->tcol = 0;
        ctl->maxt = 0.0;
    }
    if (tid < r) rho[tid] = tid;
    __syncthreads();
    persist_colnorm<GR>(G, ldg, r, rho, true, d, L);
    // a non-finite entry or a zero column ends the problem at once
    int status = HSVD_OK;
    {
        int bad_inval = 0, bad_rank = 0;
        for (int q = tid; q < r; q += NT) {
            if (!isfinite(d[q])) bad_inval = 1;
            else if (!(d[q] > 0.0)) bad_rank = 1;
        }
        bad_inval = __syncthreads_or(bad_inval);
        bad_rank = __syncthreads_or(bad_rank);
        status = bad_inval ? HSVD_E_INVAL : (bad_rank ? HSVD_E_RANK : HSVD_OK);
    }
    if (pa.sort && status == HSVD_OK) persist_sort(d, rho, r, p, L);

    int sweeps = 0, code = 0;
    double maxt = 0.0;
    unsigned long long rot_all = 0, skip_all = 0, act_all = 0;
    int sweeps32 = 0, nsiters = 0, restart = 0;
    double nsprev = 2.0;
    if (pa.mixed && status == HSVD_OK) {
        // FP32 block sweeps on FP32 copies of G and V = I, each leaving by the
        // switch rule of a single mixed solve; then V promoted and
        // J-re-orthogonalised (Newton-Schulz, FP64 MFMA products) and
        // G1 = G X, or, after a rank flag in FP32 or a residual above the
        // accepted bound, a restart from G in FP64.  The stepper goes on
        // from where the FP32 sweeps left it.
        float *G32 = reinterpret_cast<float *>(slot + sl.G32);
        float *V32 = reinterpret_cast<float *>(slot + sl.V32);
        double *T1 = reinterpret_cast<double *>(slot + sl.T1);
        double *T2 = reinterpret_cast<double *>(slot + sl.T2);
        for (int e = tid; e < r * ldg; e += NT) {
            const int c = e / ldg, row = e - c * ldg;
            G32[e] = (float)G[e];
            V32[e] = row == c ? 1.f : 0.f;
        }
        // the FP32 Gram resolves cosines down to about sqrt(r) FP32 epsilons
        const double tol32 = fmax(tol, sqrt((double)r) * 0x1p-23);
        if (tid == 0) {
            BlockArgsT<float> f;
            f.G = G32;
            f.V = V32;
            f.ldg = ldg;
            f.r = r;
            f.p = p;
            f.nb = nb;
            f.rho = rho;
            f.S_in = S;
            f.S_out = S;
            f.ordering = pa.ordering;
            f.step = 0;
            f.partial = reinterpret_cast<float *>(a.partial);
            f.splits = 1;
            f.rows_per_split = ldg;
            f.W = reinterpret_cast<float *>(a.W);
            f.active = a.active;
            f.C = a.C;
            f.nrot = a.nrot;
            f.nskip = a.nskip;
            f.nact = a.nact;
            f.ntc = a.ntc;
            f.maxt = a.maxt;
            f.ctl = ctl;
            f.tol = tol32;
            f.tthresh = sqrt(tol32) / 2.0;
            f.inner_sweeps = 0;
            f.nprob = 1;
            pargs32() = f;
        }
        __syncthreads();
        double pm = 1.0, pf = 1.0;
        for (int sw = 0; sw < pa.max_sweeps; ++sw) {
            for (int k = 0; k < steps_per_sweep; ++k) {
                if (tid == 0) pargs32().step = k;
                __syncthreads();
                outer_step<float, GR>(pairs, k == 0);
                if (pa.ordering == HSVD_ORD_MODMOD && tid < pairs) S[tid] = modmod_next(S[tid], nb);
                __syncthreads();
            }
            ++sweeps32;
            persist_colnorm<GR>(G32, ldg, r, rho, false, d, L);
            if (pa.sort) persist_sort(d, rho, r, p, L);
            int c = 0;
            unsigned long long rt = 0, sk = 0, ac = 0;
            double mx = 0.0;
            for (int q = 0; q < pairs; ++q) {
                c |= a.C[q];
                rt += a.nrot[q];
                sk += a.nskip[q];
                ac += a.nact[q];
                mx = fmax(mx, a.maxt[q]);
            }
            const int rank = __hip_atomic_load(&ctl->rank, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (tid < pairs) {
                a.C[tid] = 0;
                a.nrot[tid] = 0;
                a.nskip[tid] = 0;
                a.nact[tid] = 0;
                a.ntc[tid] = 0;
                a.maxt[tid] = 0.0;
            }
            if (tid == 0 && rank) __hip_atomic_store(&ctl->rank, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            rot_all += rt;
            skip_all += sk;
            act_all += ac;
            if (rank) {
                // a rank failure is final only in FP64
                restart = 1;
                break;
            }
            // leave FP32 at its resolution, on stagnation, when FP32 itself
            // converged, or by the fraction of rotating pair visits
            const double frac = rt + sk > 0 ? (double)rt / (double)(rt + sk) : 0.0;
            const bool stop = mx <= 3e-4 || (c & 2) == 0 || (mx < 0.1 && mx > 0.25 * pm) || frac < 0.01 ||
                              (frac <= 1.0 / 3.0 && frac >= 0.75 * pf) || sweeps32 >= pa.max_sweeps;
            pm = mx;
            pf = frac;
            if (stop) break;
        }
        if (!restart) {
            for (int e = tid; e < r * ldg; e += NT) V[e] = (double)V32[e];
            __syncthreads();
            // Newton-Schulz: X <- X (3I - J X^T J X) / 2 while the residual
            // max |J X^T J X - I| falls quadratically above its rounding floor
            const double floor_ = 16.0 * n * 0x1p-53;
            for (int it = 0; it <= 6; ++it) {
                if (tid == 0) {
                    GemmArgs g;
                    g.A = V;
                    g.B = V;
                    g.C = T2;
                    g.M = g.N = g.K = r;
                    g.lda = g.ldb = g.ldc = ldg;
                    g.p = p;
                    pgemm() = g;
                }
                __syncthreads();
                phase_gemm<true, true, true, GR>();
                double mxr = 0.0;
                for (int e = tid; e < r * ldg; e += NT) {
                    const int c = e / ldg, row = e - c * ldg;
                    const double b = T2[e];
                    const double y = row < p ? b : -b;
                    const double id = row == c ? 1.0 : 0.0;
                    mxr = fmax(mxr, fabs(y - id));
                    T2[e] = (3.0 * id - y) * 0.5;
                }
#pragma unroll
                for (int m = 32; m >= 1; m >>= 1) mxr = fmax(mxr, __shfl_xor(mxr, m, 64));
                if ((tid & 63) == 0) L.red[tid >> 6] = mxr;
                __syncthreads();
                double resid = L.red[0];
                for (int w = 1; w < NT / 64; ++w) resid = fmax(resid, L.red[w]);
                __syncthreads();
                const bool stop = it == 6 || !(resid < 1.0) || resid <= floor_ || (it > 0 && resid > 0.25 * nsprev);
                nsprev = resid;  // the residual of the current X: the final one once stopped
                if (stop) break;
                ++nsiters;
                if (tid == 0) {
                    GemmArgs g;
                    g.A = V;
                    g.B = T2;
                    g.C = T1;
                    g.M = g.N = g.K = r;
                    g.lda = g.ldb = g.ldc = ldg;
                    pgemm() = g;
                }
                __syncthreads();
                phase_gemm<false, false, false, GR>();
                for (int e = tid; e < r * ldg; e += NT) V[e] = T1[e];
                __syncthreads();
            }
            const double bound = pa.reorth_accept > 0.0 ? pa.reorth_accept : 16384.0 * n * 0x1p-53;
            if (!(nsprev <= bound)) restart = 1;
        }
        if (!restart) {
            // G1 = G X
            if (tid == 0) {
                GemmArgs g;
                g.A = G;
                g.B = V;
                g.C = T1;
                g.M = g.N = g.K = r;
                g.lda = g.ldb = g.ldc = ldg;
                pgemm() = g;
            }
            __syncthreads();
            phase_gemm<false, false, false, GR>();
            for (int e = tid; e < r * ldg; e += NT) G[e] = T1[e];
        } else {
            // FP64 from G: the bordered working copy again, V = I, rho = id
            for (int e = tid; e < r * ldg; e += NT) {
                const int c = e / ldg, row = e - c * ldg;
                double v;
                if (c < n)
                    v = row < n ? src[(size_t)c * n + row] : 0.0;
                else
                    v = row == c ? 1.0 : 0.0;
                G[e] = v;
                V[e] = row == c ? 1.0 : 0.0;
            }
            if (tid < r) rho[tid] = tid;
        }
        __syncthreads();
        // the kept diagonal of the FP64 start and the sort, as after a sweep
        persist_colnorm<GR>(G, ldg, r, rho, false, d, L);
        if (pa.sort) persist_sort(d, rho, r, p, L);
    }
    if (status == HSVD_OK) {
        status = HSVD_E_NOCONV;
        for (int sw = 0; sw < pa.max_sweeps; ++sw) {
            for (int k = 0; k < steps_per_sweep; ++k) {
                if (tid == 0) A.step = k;
                __syncthreads();
                outer_step<double, GR>(pairs, k == 0);
                if (pa.ordering == HSVD_ORD_MODMOD && tid < pairs) S[tid] = modmod_next(S[tid], nb);
                __syncthreads();
            }
            ++sweeps;
            persist_colnorm<GR>(G, ldg, r, rho, false, d, L);
            if (pa.sort) persist_sort(d, rho, r, p, L);
            // the sweep's codes and counters (eq. 4.2)
            int c = 0;
            unsigned long long rt = 0, sk = 0, ac = 0;
            double mx = 0.0;
            for (int q = 0; q < pairs; ++q) {
                c |= a.C[q];
                rt += a.nrot[q];
                sk += a.nskip[q];
                ac += a.nact[q];
                mx = fmax(mx, a.maxt[q]);
            }
            // the inner solves raise the flag with device-scope atomics
            const int rank = __hip_atomic_load(&ctl->rank, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (tid < pairs) {
                a.C[tid] = 0;
                a.nrot[tid] = 0;
                a.nskip[tid] = 0;
                a.nact[tid] = 0;
                a.ntc[tid] = 0;
                a.maxt[tid] = 0.0;
            }
            code = c;
            maxt = mx;
            rot_all += rt;
            skip_all += sk;
            act_all += ac;
            if (rank) {
                status = HSVD_E_RANK;
                break;
            }
            if ((c & 2) == 0) {
                status = HSVD_OK;
                break;
            }
        }
    }

    // Sigma, U = G Sigma^{-1}, lambda, V of the real columns
    const int lane = tid & 63, wave = tid >> 6;
    for (int q = wave; q < r; q += NT / 64) {
        const int c = rho[q];
        if (c >= n) continue;
        const double dq = d[q];
        const double s = sqrt(dq);
        const long long vo = pa.voff[z], mo = pa.off[z];
        if (lane == 0) {
            pa.sigma[vo + c] = s;
            if (pa.lambda) pa.lambda[vo + c] = q < p ? dq : -dq;
        }
        const double *gc = G + (size_t)c * ldg;
        if (pa.U)
            for (int row = lane; row < n; row += 64) pa.U[mo + (size_t)c * n + row] = gc[row] / s;
        if (pa.V && V) {
            const double *vc = V + (size_t)c * ldg;
            for (int row = lane; row < n; row += 64) pa.V[mo + (size_t)c * n + row] = vc[row];
        }
    }
    if (tid == 0 && pa.mixed) {
        pa.sweeps32[z] = sweeps32;
        pa.nsiters[z] = nsiters;
        pa.restart[z] = restart;
        pa.nsres[z] = nsprev;
    }
    if (tid == 0) {
        pa.status[z] = status;
        pa.sweeps[z] = sweeps;
        pa.code[z] = code;
        pa.maxt[z] = maxt;
        pa.rot[z] = rot_all;
        pa.skip[z] = skip_all;
        pa.act[z] = act_all;
    }
    __syncthreads();
}

}  // namespace

// Four waves per SIMD: one workgroup of four groups per compute unit, two of
// two, four of one.
template <int GR>
__global__ __launch_bounds__(256 * GR, 4) void batch_persist_kernel(PersistArgs pa)
{
    __shared__ int s_idx;
    char *slot = pa.slots + (size_t)blockIdx.x * slot_layout(pa.mixed != 0).bytes;
    for (;;) {
        if (threadIdx.x == 0) s_idx = atomicAdd(pa.next, 1);
        __syncthreads();
        const int idx = s_idx;
        __syncthreads();
        if (idx >= pa.batch) break;
        persist_solve<GR>(pa, pa.order[idx], slot, lds<GR>(), pargs());
    }
}

__global__ void persist_zero_kernel(int *next) { *next = 0; }

size_t persist_slot_bytes(bool mixed) { return slot_layout(mixed).bytes; }

int persist_blocks_per_cu(int threads)
{
    int blocks = 0;
    hipError_t e = hipErrorInvalidValue;
    if (threads == 256) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_persist_kernel<1>, 256, 0);
    if (threads == 512) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_persist_kernel<2>, 512, 0);
    if (threads == 1024) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, batch_persist_kernel<4>, 1024, 0);
    return e == hipSuccess ? blocks : 0;
}

hipError_t launch_batch_persist(hipStream_t st, const PersistArgs &pa, int threads, int workgroups)
{
    if (workgroups < 1 || pa.batch < 1) return hipErrorInvalidValue;
    if (threads != 256 && threads != 512 && threads != 1024) return hipErrorInvalidValue;
    persist_zero_kernel<<<1, 1, 0, st>>>(pa.next);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (threads == 256) batch_persist_kernel<1><<<workgroups, 256, 0, st>>>(pa);
    if (threads == 512) batch_persist_kernel<2><<<workgroups, 512, 0, st>>>(pa);
    if (threads == 1024) batch_persist_kernel<4><<<workgroups, 1024, 0, st>>>(pa);
    return hipGetLastError();
}

}  // namespace hsvd
