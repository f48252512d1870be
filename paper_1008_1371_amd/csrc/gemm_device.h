// FP64 matrix product tiles on 16x16x4 FP64 MFMA, shared by the grid-wide
// product kernel (gemm_kernels.hip; 128 x 128 tiles of C) and the persistent
// batched solver, which forms a small problem's re-orthogonalisation products
// inside one workgroup (64 x 64 tiles: 32 accumulation registers and 32 KB of
// LDS per 256 threads, so that several groups of them share a compute unit).
// C = op(A) S B, op(A) = A or A^T, S = I or diag(+1 x p, -1 x (K - p)) on the
// rows of B, all column-major FP64.  256 threads form a tile; each of their
// four waves a quarter of it as MFMA tiles of 16 x 16.  K runs in chunks of 16, staged in LDS in MFMA
// operand order (element (i, k) of a 16 x 4 operand tile at lane i + 16 k,
// so every operand read is one contiguous 512-byte LDS read), the next
// chunk's global loads in flight while the current chunk's MFMAs run (two
// LDS buffers, one barrier per chunk).  The MFMA takes the B tile as its
// first operand, so it computes the transpose of the C tile: result lanes run
// along the rows of C and each store writes 16 consecutive rows of 4 columns.
// A symmetric product (SYM) writes each tile with row <= col to both
// triangles.
#pragma once
#include "internal.h"

namespace hsvd {
namespace gemm {

typedef double gd2 __attribute__((ext_vector_type(2)));
typedef double gd4 __attribute__((ext_vector_type(4)));

constexpr int kTK = 16;   // K chunk

// Position of element (i, k) of a kT x 16 operand tile in MFMA operand
// order: operand tile (k / 4, i / 16), lane (i % 16) + 16 (k % 4).
template <int kT>
__device__ __forceinline__ int frag_pos(int i, int k)
{
    return ((((k >> 2) * (kT / 16)) + (i >> 4)) << 6) + (i & 15) + ((k & 3) << 4);
}

// kT: rows and columns of a tile of C (square: the symmetric product mirrors
// them).
template <int kT>
struct GemmLds {
    double As[2][kT * kTK];
    double Bs[2][kT * kTK];
};

// Tile (tm, tn) of problem z (zg, ks: block pair and K split of the
// block-pair form, else zg = z, ks = 0), by 256 threads, tid among them, with
// g.K / kTK + 1 workgroup barriers.
template <bool TA, bool SGN, bool SYM, int kT>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, int z, int zg, int ks, int tm, int tn, GemmLds<kT> &L,
                                          int tid)
{
    constexpr int kMt = kT / 32;               // 16 x 16 tiles of a wave per direction
    constexpr int kIt = kT * kTK / (2 * 256);  // 16-byte items per thread and operand
    constexpr int kAp = kT / 2;                // items per column of an untransposed A chunk
    double(*const As)[kT * kTK] = L.As;
    double(*const Bs)[kT * kTK] = L.Bs;
    // A and C may be the same matrix (in-place block-pair update): no
    // restrict on them
    const int mapA = g.map & 1, mapB = g.map & 2, mapC = g.map & 4;
    const size_t koff = (size_t)ks * g.K;  // rows of this K split (transposed A, B)
    const double *A = g.A + (mapA ? (TA ? koff : 0) : (size_t)z * g.sa);
    const double *__restrict__ B = g.B + (mapB ? koff : (size_t)z * g.sb);
    double *C = g.C + (mapC ? 0 : (size_t)z * g.sc);
    const int2 bij = g.blk ? g.blk[zg] : make_int2(0, 0);
    auto mcol = [&](int c) -> size_t {
        return (size_t)(c < g.bw ? bij.x * g.bw + c : bij.y * g.bw + (c - g.bw));
    };
    const int p = g.pvec ? g.pvec[zg] : g.p;
    const int M = g.M, N = g.N, K = g.K;
    const int i0 = tm * kT, j0 = tn * kT;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // global loads of one K chunk, 16 bytes per thread and item
    gd2 ra[kIt], rb[kIt];
    auto gload = [&](int k0) {
#pragma unroll
        for (int q = 0; q < kIt; ++q) {
            const int u = tid + 256 * q;
            if (!TA) {
                // A(i, k) = A[k lda + i]: kT consecutive rows of one column
                const int kk = u / kAp, ip = (u % kAp) * 2, i = i0 + ip;
                const size_t ca = mapA ? mcol(k0 + kk) : (size_t)(k0 + kk);
                ra[q] = i < M ? *reinterpret_cast<const gd2 *>(A + ca * g.lda + i) : gd2{0.0, 0.0};
            } else {
                // A(i, k) = A[i lda + k]: 8 lanes read 128 bytes of one column
                const int il = u >> 3, kp = (u & 7) * 2, i = i0 + il;
                ra[q] = i < M ? *reinterpret_cast<const gd2 *>(A + (mapA ? mcol(i) : (size_t)i) * g.lda + k0 + kp)
                              : gd2{0.0, 0.0};
            }
            const int jl = u >> 3, kp = (u & 7) * 2, j = j0 + jl;
            gd2 b = j < N ? *reinterpret_cast<const gd2 *>(B + (mapB ? mcol(j) : (size_t)j) * g.ldb + k0 + kp)
                          : gd2{0.0, 0.0};
            if (SGN) {
                if (k0 + kp >= p) b.x = -b.x;
                if (k0 + kp + 1 >= p) b.y = -b.y;
            }
            rb[q] = b;
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < kIt; ++q) {
            const int u = tid + 256 * q;
            if (!TA) {
                const int kk = u / kAp, ip = (u % kAp) * 2;
                *reinterpret_cast<gd2 *>(&As[buf][frag_pos<kT>(ip, kk)]) = ra[q];
            } else {
                const int il = u >> 3, kp = (u & 7) * 2;
                As[buf][frag_pos<kT>(il, kp)] = ra[q].x;
                As[buf][frag_pos<kT>(il, kp + 1)] = ra[q].y;
            }
            const int jl = u >> 3, kp = (u & 7) * 2;
            Bs[buf][frag_pos<kT>(jl, kp)] = rb[q].x;
            Bs[buf][frag_pos<kT>(jl, kp + 1)] = rb[q].y;
        }
    };

    gd4 acc[kMt][kMt];
#pragma unroll
    for (int m = 0; m < kMt; ++m)
#pragma unroll
        for (int n = 0; n < kMt; ++n) acc[m][n] = gd4{0.0, 0.0, 0.0, 0.0};

    const int nk = K / kTK;
    gload(0);
    sstore(0);
    __syncthreads();
    for (int kc = 0; kc < nk; ++kc) {
        const int cur = kc & 1;
        if (kc + 1 < nk) gload((kc + 1) * kTK);
#pragma unroll
        for (int kt = 0; kt < kTK / 4; ++kt) {
            double a[kMt], b[kMt];
#pragma unroll
            for (int m = 0; m < kMt; ++m) a[m] = As[cur][((kt * (kT / 16) + wm * kMt + m) << 6) + lane];
#pragma unroll
            for (int n = 0; n < kMt; ++n) b[n] = Bs[cur][((kt * (kT / 16) + wn * kMt + n) << 6) + lane];
#pragma unroll
            for (int m = 0; m < kMt; ++m)
#pragma unroll
                for (int n = 0; n < kMt; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[n], a[m], acc[m][n], 0, 0, 0);
        }
        if (kc + 1 < nk) sstore(cur ^ 1);
        __syncthreads();
    }

    // register v of lane l holds C(i0 + 16 (kMt wm + m) + l % 16, j0 + 16 (kMt wn + n) + l / 16 + 4 v)
#pragma unroll
    for (int m = 0; m < kMt; ++m)
#pragma unroll
        for (int n = 0; n < kMt; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = i0 + 16 * (kMt * wm + m) + (lane & 15);
                const int col = j0 + 16 * (kMt * wn + n) + (lane >> 4) + 4 * v;
                if (row >= M || col >= N) continue;
                const double x = acc[m][n][v];
                if (!SYM) {
                    C[(mapC ? mcol(col) : (size_t)col) * g.ldc + row] = x;
                } else if (row <= col) {
                    // both triangles from the entry with row <= col
                    C[(size_t)col * g.ldc + row] = x;
                    C[(size_t)row * g.ldc + col] = x;
                }
            }
}

}  // namespace gemm
}  // namespace hsvd
