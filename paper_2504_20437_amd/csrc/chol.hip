// Cholesky factorisation of the k x k Gram matrices (fp64) and the inverse of the
// factor, for the Cholesky-based orthonormalisation (Q = Y R^-1 with
// R^T R = Y^T Y) that keeps the sketch well conditioned between the products
// of the randomized subspace iteration (Halko et al. 2011, §4.5 re-orthonormal-
// ises after every application of A or A^T), and for the square factor the
// small SVD works on.
//
// Right-looking, blocked by CB = 64 rows; every launch covers all matrices of
// the batch (grid y = matrix), so the chip is filled by (tiles x batch)
// workgroups rather than one workgroup per matrix. The inverse X = R'^-1 is
// built alongside, column block by column block (X R' = I gives
// X_IJ = -(sum_{U<J} X_IU R_UJ) D_J), its partial sums P_IJ accumulated by the
// trailing launches in X's own upper blocks, so no separate inverse phase runs:
//   diag 0   factor the 64 x 64 diagonal block 0 (fp64, by block rows of 16)
//            and invert it (D_0 = R'_00^-1, kept in X's diagonal block);
//   for each block row J:
//     panel+X  R_JT = D_J^T C_JT for every block column T > J, and block column J
//              of the inverse, X_IJ = -P_IJ D_J for I < J (fp64 and fp32, the
//              fp32 copy's lower tiles zero for the GEMM that applies it);
//     trailing C_T1T2 -= R_JT1^T R_JT2 on the upper tiles J < T1 <= T2, and
//              P_IT (+)= X_IJ R_JT for I <= J < T; the workgroup of tile
//              (J + 1, J + 1) then factors and inverts that diagonal block
//              (step J + 1's diagonal), whose last update it just made.
// The panel, inverse, trailing and partial-sum tiles are 64 x 64 x 64 products
// on the fp64 matrix cores, operands loaded from memory straight into
// registers. Two launches per block row (with the factor's inverse or without).
// R overwrites the upper triangle of C; the lower triangle is not used.
//
// Semi-definite inputs: a pivot d <= tau_rel * (original diagonal) marks the
// column as numerically dependent on the previous ones. Its row of R is set to
// zero (R^T R still reproduces the Gram), and for the inverse that row is
// replaced by the unit row so that R' stays invertible; the caller replaces the
// corresponding column of Q by a generic unit vector (fill_deficient).
#include "common.hpp"

namespace galore {
namespace {

constexpr int CB = 64;     // block size
constexpr int CT = 256;    // threads per workgroup (4 waves)

__device__ __forceinline__ void zero_acc(f64x4 acc[2][2]) {
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = f64x4{0.0, 0.0, 0.0, 0.0};
}

typedef double f64x2 __attribute__((ext_vector_type(2)));

// (M[row * ld + col], M[row * ld + col + 1]) with zeros outside row < nr,
// col < nc; one 16-byte load when vec (even ld and offsets)
__device__ __forceinline__ f64x2 ld_pair(const double* M, int64_t ld, int row, int col, int nr, int nc,
                                         bool vec) {
    f64x2 p = {0.0, 0.0};
    if (row < nr) {
        const double* q = M + static_cast<int64_t>(row) * ld + col;
        if (vec && col + 1 < nc) {
            p = *reinterpret_cast<const f64x2*>(q);
        } else {
            if (col < nc) p[0] = q[0];
            if (col + 1 < nc) p[1] = q[1];
        }
    }
    return p;
}

// Register-direct 64 x 64 x 64 product for the tile kernels: wave (wm, wn)
// owns output rows 32 wm + 2 i + bi and columns 32 wn + 2 j + bj (i, j < 16,
// bi, bj < 2), so each lane's A (B) operands for the two row (column) blocks
// are one 16-byte pair; step s of the contraction takes rows 4 s + (lane >> 4)
// of the two row-major operand panels Ap (t x rows) and Bp (t x cols).
// Accumulator register v of block (bi, bj) holds row 32 wm + 2 (4 v + (lane >> 4)) + bi,
// column 32 wn + 2 (lane & 15) + bj.
__device__ __forceinline__ void mma64_pairs(const double* Ap, const double* Bp, int64_t ld, int nt, int na,
                                            int nbc, bool vec, f64x4 acc[2][2], int wm, int wn, int lane) {
    const int l16 = lane & 15, lk = lane >> 4;
    // four groups of four steps, the next group's operands in flight while the
    // current one is multiplied (keeps the kernels within 128 registers)
    f64x2 av[2][4], bv[2][4];
    auto load = [&](int g, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = 4 * (4 * g + i) + lk;
            av[buf][i] = ld_pair(Ap, ld, t, 32 * wm + 2 * l16, nt, na, vec);
            bv[buf][i] = ld_pair(Bp, ld, t, 32 * wn + 2 * l16, nt, nbc, vec);
        }
    };
    load(0, 0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g + 1 < 4) load(g + 1, (g + 1) & 1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int bj = 0; bj < 2; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[g & 1][i][bi], bv[g & 1][i][bj],
                                                                       acc[bi][bj], 0, 0, 0);
    }
}

// fp64 value of one lane, in every lane
__device__ __forceinline__ double lane_value(double v, int lane) {
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// fp64 value of the lane whose byte address (4 times its number) is a
__device__ __forceinline__ double lane_at(int a, double v) {
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_ds_bpermute(a, static_cast<int>(u));
    const uint32_t hi = __builtin_amdgcn_ds_bpermute(a, static_cast<int>(u >> 32));
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// r = sqrt(d) and y = 1 / r for d > 0: the hardware's estimate of 1 / sqrt(d),
// two Newton steps, the root's residual taken out once and the reciprocal's
// once. The last two steps round correctly (equal to sqrt and division on
// 102400 random values), at half their length.
__device__ __forceinline__ void root64(double d, double& r, double& y) {
    y = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-d * y, y, 1.0), y);
    r = d * y;
    r = fma(0.5 * y, fma(-r, r, d), r);
    y = fma(y, fma(-r, y, 1.0), y);
}

// Factor the diagonal block J and invert its factor, one workgroup per matrix.
// The 64 x 64 block sits in LDS and is worked off in four block rows of 16:
//  * wave 0 takes the block row, one column a lane (lane l: column 16 ib + l,
//    sixteen rows in registers), and eliminates it: pivot d = S_ii; d <=
//    tau_rel * (original diagonal) marks a dependent column, whose row of R is
//    zero; otherwise the row is scaled by 1 / sqrt(d) and R_ia times it is
//    taken from the rows a > i. The R_ia are lane values, so a pivot costs no
//    LDS access and no barrier;
//  * the four waves update the block rows below on the fp64 matrix cores.
// Then wave J works out block column J of D = R'^-1 (R' = R with unit rows for
// the dependent pivots) from its last row: what the rows below take from a
// block row on the matrix cores, then the block row by substitution, a column
// a lane (in all four lane groups alike).
// An fp64 matrix-core product adds its four terms one by one in the order of
// the contraction index (checked on the device against a chain of fused
// multiply-adds), so every entry sees the operations of the plain right-looking
// factorisation and of the substitution from the last row, in their order: the
// same bits as one pivot at a time, whatever the block's condition.
// Rows and columns past the matrix are those of the unit matrix.
// One barrier, square root and division per pivot and 128 dependent steps of
// the whole workgroup took 56 us a block; this form 20 us.
// (the body of one matrix's diagonal step; every thread of the workgroup calls it)
// The block (upper triangle) and lim are in LDS on entry, behind a barrier.
constexpr int DB = 16;       // block rows
struct DiagLds {
    double S[CB][CB + 1];
    double lim[CB];          // tau_rel * original diagonal
    double inv[CB];          // 1 / R'_ii
};
__device__ __forceinline__ void diag_block(DiagLds& lds, double* C, int k, int J, int* defic, double* X, float* Ri) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lk = lane >> 4;
    const int j0 = J * CB;
    const int jb = min(CB, k - j0);
    double (*S)[CB + 1] = lds.S;
    // R_ii^T (row pitch CB + 1) in the free blocks (1, 0), (2, 0), (2, 1) and
    // (3, 0) below the diagonal
    auto rt = [&](int i) { return &S[i == 0 ? DB : (i == 3 ? 3 * DB : 2 * DB)][i == 2 ? DB : 0]; };

    for (int ib = 0; ib < CB / DB; ++ib) {
        const int r0 = DB * ib;
        if (wave == 0) {
            // kept opaque per block row: the lane masks of all pivots, formed
            // once for all block rows, would not fit the scalar registers
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int c = min(r0 + ln, CB - 1);
            const double li = lds.lim[r0 + (ln & 15)];
            double s[DB];
#pragma unroll
            for (int i = 0; i < DB; ++i) s[i] = S[r0 + i][c];
            unsigned dmask = 0;
            double iv = 1.0;
#pragma unroll
            for (int i = 0; i < DB; ++i) {
                const bool def = (__builtin_amdgcn_ballot_w64(s[i] <= li) >> i) & 1;   // lane i's; NaN compares false
                const double d = lane_value(s[i], i);
                double r, y;
                root64(d, r, y);
                s[i] = (ln == i) ? (def ? 0.0 : r) : s[i] * (def ? 0.0 : y);
                iv = (ln == i) ? (def ? 1.0 : y) : iv;
                dmask |= def ? 1u << i : 0u;
#pragma unroll
                for (int a = i + 1; a < DB; ++a) s[a] = fma(-lane_value(s[i], a), s[i], s[a]);
                // pivot by pivot: left to itself the compiler puts a row's updates off
                // to its own pivot, and their lane values do not fit the scalar registers
                asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "+v"(s[4]), "+v"(s[5]), "+v"(s[6]),
                             "+v"(s[7]), "+v"(s[8]), "+v"(s[9]), "+v"(s[10]), "+v"(s[11]), "+v"(s[12]), "+v"(s[13]),
                             "+v"(s[14]));
            }
            if (r0 + ln < CB) {
#pragma unroll
                for (int i = 0; i < DB; ++i) S[r0 + i][r0 + ln] = s[i];
            }
            if (ln < DB) {
                double* t = rt(ib) + (CB + 1) * ln;
#pragma unroll
                for (int i = 0; i < DB; ++i) t[i] = s[i];
                lds.inv[r0 + ln] = iv;
                if (r0 + ln < jb) defic[j0 + r0 + ln] = (dmask >> ln) & 1;
            }
        }
        __syncthreads();
        // S_ab -= R_ia^T R_ib for the block rows below (a diagonal block's lower
        // part is not used)
        const int n = CB / DB - 1 - ib;
        for (int t = wave; t < n * (n + 1) / 2; t += CT / 64) {
            int u = 0, idx = t;
            while (idx >= n - u) {
                idx -= n - u;
                ++u;
            }
            const int a0 = DB * (ib + 1 + u), b0 = DB * (ib + 1 + u + idx);
            f64x4 acc;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] = S[a0 + 4 * v + lk][b0 + l16];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[r0 + 4 * v + lk][a0 + l16], S[r0 + 4 * v + lk][b0 + l16],
                                                           acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) S[a0 + 4 * v + lk][b0 + l16] = acc[v];
        }
        __syncthreads();
    }

    // block column `wave` of D: xb[U] = rows 16 U + 4 v + 3 - lk (right operands
    // in descending order of the row), xs[U] = rows 16 U + 4 v + lk, stored at the
    // end (between the blocks the stores held up the next one's reads); a whole
    // block (uniform) without per-entry branches, zeros below the diagonal
    double* Xd = X + static_cast<int64_t>(j0) * k + j0 + DB * wave + l16;
    double* Cd = C + static_cast<int64_t>(j0) * k + j0;
    float* Rd = Ri != nullptr ? Ri + static_cast<int64_t>(j0) * k + j0 + DB * wave + l16 : nullptr;
    auto store = [&](int U, f64x4 x) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = DB * U + 4 * v + lk;
            if (jb == CB || (r < jb && DB * wave + l16 < jb)) {
                Xd[static_cast<int64_t>(r) * k] = x[v];
                if (Rd != nullptr) Rd[static_cast<int64_t>(r) * k] = static_cast<float>(x[v]);
            }
        }
    };
    f64x4 xb[CB / DB], xs[CB / DB];
    auto pick = [&](double x0, double x1, double x2, double x3, int g) {
        const double u = (g & 1) ? x1 : x0, v = (g & 1) ? x3 : x2;
        return (g & 2) ? v : u;
    };
#pragma unroll
    for (int U = CB / DB - 1; U >= 0; --U) {
        xs[U] = xb[U] = f64x4{0.0, 0.0, 0.0, 0.0};
        if (U > wave) continue;
        double x[DB];
        if (U == wave) {
#pragma unroll
            for (int i = 0; i < DB; ++i) x[i] = (l16 == i) ? 1.0 : 0.0;
        } else {
            f64x4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int T = CB / DB - 1; T > U; --T) {
                if (T > wave) continue;
#pragma unroll
                for (int v = 3; v >= 0; --v)
                    z = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[DB * U + l16][DB * T + 4 * v + 3 - lk], xb[T][v], z, 0, 0,
                                                             0);
            }
            // all sixteen rows of the lane's column
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int g = 0; g < 4; ++g) x[4 * v + g] = lane_at(4 * (l16 + 16 * g), z[v]);
        }
        const double* t = rt(U);
#pragma unroll
        for (int i = DB - 1; i >= 0; --i) {
            x[i] *= lds.inv[DB * U + i];
#pragma unroll
            for (int a = i - 1; a >= 0; --a) x[a] = fma(-t[(CB + 1) * i + a], x[i], x[a]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            xs[U][v] = pick(x[4 * v], x[4 * v + 1], x[4 * v + 2], x[4 * v + 3], lk);
            xb[U][v] = pick(x[4 * v + 3], x[4 * v + 2], x[4 * v + 1], x[4 * v], lk);
            if (U == wave && 4 * v + lk > l16) xs[U][v] = 0.0;
        }
    }
#pragma unroll
    for (int U = 0; U < CB / DB; ++U) store(U, xs[U]);
    if (jb == CB) {
#pragma unroll 8
        for (int e = 0; e < CB * CB / CT; ++e) {
            const int a = wave + 4 * e;
            if (a <= lane) Cd[static_cast<int64_t>(a) * k + lane] = S[a][lane];
        }
    } else {
        for (int a = wave; a < jb; a += CT / 64)
            if (a <= lane && lane < jb) Cd[static_cast<int64_t>(a) * k + lane] = S[a][lane];
    }
}

// Block 0 of every matrix (blockIdx.y = 0), and the diagonal of the Gram that
// the later blocks' dependency tests compare with (blockIdx.y = 1)
__global__ __launch_bounds__(CT) void chol_diag_kernel(double* Cb, int k, int64_t strideC, double* diag0b, int* deficB,
                                                       double* Xb, float* Rib, int64_t strideInv, double tau_rel) {
    __shared__ DiagLds lds;
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    double* C = Cb + static_cast<int64_t>(b) * strideC;
    if (blockIdx.y == 1) {
        // not those of block 0: its factor overwrites them (it keeps its own)
#pragma unroll 4
        for (int i = CB + tid; i < k; i += CT) diag0b[static_cast<int64_t>(b) * k + i] = C[static_cast<int64_t>(i) * k + i];
        return;
    }
    const int jb = min(CB, k);
    if (tid < CB) {
        const double d = tid < jb ? C[static_cast<int64_t>(tid) * k + tid] : 0.0;
        if (tid < jb) diag0b[static_cast<int64_t>(b) * k + tid] = d;
        lds.lim[tid] = tau_rel * d;
    }
#pragma unroll
    for (int e = 0; e < CB * CB / CT; ++e) {
        const int a = (tid >> 6) + 4 * e, c = tid & 63;
        lds.S[a][c] = (c < jb && a <= c) ? C[static_cast<int64_t>(a) * k + c] : (a == c ? 1.0 : 0.0);
    }
    __syncthreads();
    diag_block(lds, C, k, 0, deficB + static_cast<int64_t>(b) * k, Xb + static_cast<int64_t>(b) * strideInv,
               Rib != nullptr ? Rib + static_cast<int64_t>(b) * strideInv : nullptr);
}

// acc += A B for one 64 x 64 x 64 tile with A given by rows (A[i * ld + t], t
// contiguous) and B by contraction rows (B[t * ld + c]), operands straight from
// global memory into registers: contraction step s takes t = 8 (s / 2) +
// 2 (lane >> 4) + s % 2, so a lane's A entries A[i][t], A[i][t + 1] are one
// 16-byte pair. The result lands in the pair layout of mma64_pairs (row
// 32 wm + 2 (4 v + (lane >> 4)) + bi, column 32 wn + 2 (lane & 15) + bj).
__device__ __forceinline__ void mma64_rowA(const double* Ap, const double* Bp, int64_t ld, int nar, int nt, int nbc,
                                           bool vec, f64x4 acc[2][2], int wm, int wn, int lane) {
    const int l16 = lane & 15, lk = lane >> 4;
    // four groups of four steps (two A pairs per row block), double-buffered as
    // in mma64_pairs
    f64x2 a2[2][2][2], b2[2][4];
    auto load = [&](int g, int buf) {
#pragma unroll
        for (int mm = 0; mm < 2; ++mm)
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
                a2[buf][mm][bi] = ld_pair(Ap, ld, 32 * wm + 2 * l16 + bi, 8 * (2 * g + mm) + 2 * lk, nar, nt, vec);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = 4 * g + i;
            b2[buf][i] = ld_pair(Bp, ld, 8 * (s >> 1) + 2 * lk + (s & 1), 32 * wn + 2 * l16, nt, nbc, vec);
        }
    };
    load(0, 0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (g + 1 < 4) load(g + 1, (g + 1) & 1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int bj = 0; bj < 2; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[g & 1][i >> 1][bi][i & 1], b2[g & 1][i][bj],
                                                                       acc[bi][bj], 0, 0, 0);
    }
}

// Step J, after the diagonal block J (factor R_JJ and D_J = R'_JJ^-1):
//  * blockIdx.x < n (n = nb - J - 1): the panel tile T = J + 1 + blockIdx.x,
//    R_JT = D_J^T C_JT (deficient rows zero), in place in C;
//  * with the inverse, blockIdx.x = n + I (I < J): block column J of the
//    inverse X = R'^-1, X_IJ = -P_IJ D_J, where P_IJ (held in X's block (I, J))
//    is the sum over U < J of X_IU R_UJ that the trailing steps accumulated;
//    written in fp64 and as fp32, whose mirrored (lower) tile is set to zero.
__global__ __launch_bounds__(CT, 4) void chol_panel_x_kernel(double* Cb, int k, int64_t strideC, int J, int n,
                                                          const int* deficB, double* Xb, float* Rib,
                                                          int64_t strideInv) {
    const int b = blockIdx.y;
    double* C = Cb + static_cast<int64_t>(b) * strideC;
    const int* defic = deficB + static_cast<int64_t>(b) * k;
    double* X = Xb + static_cast<int64_t>(b) * strideInv;
    const int j0 = J * CB;
    const int jb = min(CB, k - j0);
    const bool vec = (k & 1) == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lk = lane >> 4;
    f64x4 acc[2][2];
    zero_acc(acc);
    if (static_cast<int>(blockIdx.x) < n) {
        const int c0 = (J + 1 + blockIdx.x) * CB;
        const int cb = min(CB, k - c0);
        // A[i][t] = D[t][i] (rows j0 + t of the block inverse), B[t][c] = C_JT[t][c]
        mma64_pairs(X + static_cast<int64_t>(j0) * k + j0, C + static_cast<int64_t>(j0) * k + c0, k, jb, jb, cb,
                    vec, acc, wm, wn, lane);
        // the deficiency flags of the lane's eight rows, read together
        bool dfl[2][4];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int v = 0; v < 4; ++v) dfl[bi][v] = defic[j0 + min(32 * wm + 2 * (4 * v + lk) + bi, jb - 1)] != 0;
        __syncthreads();   // every wave has its operands before the tile is overwritten
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 32 * wm + 2 * (4 * v + lk) + bi;
                if (r >= jb) continue;
                const bool def = dfl[bi][v];
                const int c = 32 * wn + 2 * l16;
                double* dst = C + static_cast<int64_t>(j0 + r) * k + c0 + c;
                const double o0 = def ? 0.0 : acc[bi][0][v], o1 = def ? 0.0 : acc[bi][1][v];
                if (vec && c + 1 < cb) {
                    *reinterpret_cast<f64x2*>(dst) = f64x2{o0, o1};
                } else {
                    if (c < cb) dst[0] = o0;
                    if (c + 1 < cb) dst[1] = o1;
                }
            }
        return;
    }
    const int I = blockIdx.x - n;
    const int i0 = I * CB;
    // A = P_IJ (rows i0.., columns j0..), B = D_J (rows j0 + t)
    mma64_rowA(X + static_cast<int64_t>(i0) * k + j0, X + static_cast<int64_t>(j0) * k + j0, k, CB, jb, jb, vec, acc,
               wm, wn, lane);
    __syncthreads();       // P_IJ is overwritten by X_IJ below
    float* Ri = Rib + static_cast<int64_t>(b) * strideInv;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 32 * wm + 2 * (4 * v + lk) + bi;
                const int c = 32 * wn + 2 * l16 + bj;
                if (c < jb) {
                    const double val = -acc[bi][bj][v];
                    X[static_cast<int64_t>(i0 + r) * k + j0 + c] = val;
                    Ri[static_cast<int64_t>(i0 + r) * k + j0 + c] = static_cast<float>(val);
                }
                // the mirrored (lower) tile of the fp32 inverse is zero
                if (r < jb) Ri[static_cast<int64_t>(j0 + r) * k + i0 + c] = 0.0f;
            }
}

// Step J's updates, after the panel:
//  * blockIdx.x < n (n + 1) / 2: C_T1T2 -= R_JT1^T R_JT2 on the upper tiles
//    J < T1 <= T2; the workgroup of tile (J + 1, J + 1) then factors that
//    diagonal block (step J + 1's diagonal), whose last update this was;
//  * with the inverse, the rest: P_IT (+)= X_IJ R_JT for I <= J < T, the
//    partial sums block column T of the inverse needs (I = J starts the sum).
__global__ __launch_bounds__(CT, 4) void chol_trailing_p_kernel(double* Cb, int k, int64_t strideC, int J, int nb,
                                                             double* diag0b, int* deficB, double* Xb, float* Rib,
                                                             int64_t strideInv, double tau_rel) {
    __shared__ DiagLds lds;   // the diagonal tile's workgroup only
    const int b = blockIdx.y;
    double* C = Cb + static_cast<int64_t>(b) * strideC;
    double* X = Xb + static_cast<int64_t>(b) * strideInv;
    const int n = nb - J - 1;
    const int ntrail = n * (n + 1) / 2;
    const int j0 = J * CB;
    const int jb = min(CB, k - j0);
    const bool vec = (k & 1) == 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lk = lane >> 4;
    f64x4 acc[2][2];
    zero_acc(acc);
    if (static_cast<int>(blockIdx.x) < ntrail) {
        // blockIdx.x -> (u, vt) with 0 <= u <= vt < n, row-major over the upper triangle
        int idx = blockIdx.x, u = 0;
        while (idx >= n - u) {
            idx -= n - u;
            ++u;
        }
        const int vt = u + idx;
        const int r0 = (J + 1 + u) * CB, rb = min(CB, k - r0);
        const int c0 = (J + 1 + vt) * CB, cb = min(CB, k - c0);
        if (blockIdx.x == 0) {
            // tile (J + 1, J + 1): its last update, into LDS, then step J + 1's
            // diagonal (the entries' original diagonal fetched beside the product)
            const bool live = threadIdx.x < CB && static_cast<int>(threadIdx.x) < rb;
            const double d0 = live ? diag0b[static_cast<int64_t>(b) * k + r0 + threadIdx.x] : 0.0;
            const int c = 32 * wn + 2 * l16;
            const bool need = wm <= wn;   // the quadrant below the diagonal is not
            if (need)
                mma64_pairs(C + static_cast<int64_t>(j0) * k + r0, C + static_cast<int64_t>(j0) * k + c0, k, jb, rb, cb,
                            vec, acc, wm, wn, lane);
            f64x2 o[2][4];
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    o[bi][v] = need ? ld_pair(C + static_cast<int64_t>(r0) * k + c0, k,
                                              32 * wm + 2 * (4 * v + lk) + bi, c, rb, cb, vec)
                                    : f64x2{0.0, 0.0};
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 32 * wm + 2 * (4 * v + lk) + bi;
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        lds.S[r][c + e] = (r < rb && c + e < cb) ? o[bi][v][e] - acc[bi][e][v] : (r == c + e ? 1.0 : 0.0);
                }
            if (threadIdx.x < CB) lds.lim[threadIdx.x] = tau_rel * d0;
            __syncthreads();
            diag_block(lds, C, k, J + 1, deficB + static_cast<int64_t>(b) * k, X,
                       Rib != nullptr ? Rib + static_cast<int64_t>(b) * strideInv : nullptr);
            return;
        }
        // on a diagonal tile the quadrant below the diagonal is not needed
        if (!(u == vt && wm > wn)) {
            // operands: rows j0 + t of the block row J just finished (R_JT1, R_JT2);
            // the tile updated lies in a later block row, so no wave reads what
            // another one writes
            mma64_pairs(C + static_cast<int64_t>(j0) * k + r0, C + static_cast<int64_t>(j0) * k + c0, k, jb, rb, cb,
                        vec, acc, wm, wn, lane);
            if (vec && rb == CB && cb == CB && u != vt) {
                // an interior tile off the diagonal (uniform): the lane's eight
                // pairs are read together, then written (read-modify-write one
                // pair at a time waited a memory latency per pair)
                const int c = 32 * wn + 2 * l16;
                f64x2 o[2][4];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        o[bi][v] = *reinterpret_cast<const f64x2*>(
                            C + static_cast<int64_t>(r0 + 32 * wm + 2 * (4 * v + lk) + bi) * k + c0 + c);
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        *reinterpret_cast<f64x2*>(C + static_cast<int64_t>(r0 + 32 * wm + 2 * (4 * v + lk) + bi) * k +
                                                  c0 + c) =
                            f64x2{o[bi][v][0] - acc[bi][0][v], o[bi][v][1] - acc[bi][1][v]};
            } else {
#pragma unroll
            for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 32 * wm + 2 * (4 * v + lk) + bi;
                    if (r >= rb) continue;
                    const int c = 32 * wn + 2 * l16;
                    const bool k0 = c < cb && (u != vt || c >= r);
                    const bool k1 = c + 1 < cb && (u != vt || c + 1 >= r);
                    double* dst = C + static_cast<int64_t>(r0 + r) * k + c0 + c;
                    if (vec && k0 && k1) {
                        f64x2 o = *reinterpret_cast<f64x2*>(dst);
                        o[0] -= acc[bi][0][v];
                        o[1] -= acc[bi][1][v];
                        *reinterpret_cast<f64x2*>(dst) = o;
                    } else {
                        if (k0) dst[0] -= acc[bi][0][v];
                        if (k1) dst[1] -= acc[bi][1][v];
                    }
                }
            }
        }
        return;
    }
    const int p = blockIdx.x - ntrail;
    const int I = p / n, T = J + 1 + p % n;
    const int i0 = I * CB;
    const int c0 = T * CB, cb = min(CB, k - c0);
    // A = X_IJ (rows i0.., columns j0..), B = R_JT (rows j0 + t of C)
    mma64_rowA(X + static_cast<int64_t>(i0) * k + j0, C + static_cast<int64_t>(j0) * k + c0, k, CB, jb, cb, vec, acc,
               wm, wn, lane);
    const bool first = (I == J);
    if (vec && i0 + CB <= k && cb == CB) {
        // a whole tile (uniform): the lane's eight pairs read together first
        const int c = 32 * wn + 2 * l16;
        f64x2 o[2][4];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                o[bi][v] = first ? f64x2{0.0, 0.0}
                                 : *reinterpret_cast<const f64x2*>(
                                       X + static_cast<int64_t>(i0 + 32 * wm + 2 * (4 * v + lk) + bi) * k + c0 + c);
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<f64x2*>(X + static_cast<int64_t>(i0 + 32 * wm + 2 * (4 * v + lk) + bi) * k + c0 + c) =
                    f64x2{o[bi][v][0] + acc[bi][0][v], o[bi][v][1] + acc[bi][1][v]};
        return;
    }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 32 * wm + 2 * (4 * v + lk) + bi;
            if (i0 + r >= k) continue;
            const int c = 32 * wn + 2 * l16;
            double* dst = X + static_cast<int64_t>(i0 + r) * k + c0 + c;
            if (vec && c + 1 < cb) {
                f64x2 o = first ? f64x2{0.0, 0.0} : *reinterpret_cast<f64x2*>(dst);
                o[0] += acc[bi][0][v];
                o[1] += acc[bi][1][v];
                *reinterpret_cast<f64x2*>(dst) = o;
            } else {
                if (c < cb) dst[0] = (first ? 0.0 : dst[0]) + acc[bi][0][v];
                if (c + 1 < cb) dst[1] = (first ? 0.0 : dst[1]) + acc[bi][1][v];
            }
        }
}

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    // splitmix64 finaliser (Steele, Lea, Flood 2014)
    z += 0x9E3779B97F4A7C15ULL;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void fill_deficient_kernel(float* Qb, int rows, int k,
                                                             int64_t strideQ, const int* deficB) {
    const int b = blockIdx.y;
    const int j = blockIdx.x;
    if (!deficB[static_cast<int64_t>(b) * k + j]) return;
    float* Q = Qb + static_cast<int64_t>(b) * strideQ;
    const float scale = 1.0f / sqrtf(static_cast<float>(rows));
    for (int i = threadIdx.x; i < rows; i += blockDim.x) {
        const uint64_t h = mix64((static_cast<uint64_t>(j) << 32) | static_cast<uint32_t>(i));
        Q[static_cast<int64_t>(i) * k + j] = (h & 1ULL) ? scale : -scale;
    }
}

// The same generic unit vector written as the three bf16 planes of column j
// (plane row j, transposed layout of GemmArgs::planes), for a Q that exists
// only as its planes; rows past `rows` keep the zeros the product wrote.
__global__ __launch_bounds__(256) void fill_deficient_planes_kernel(uint16_t* planesb, int64_t ldpl, int64_t planeStride,
                                                                    int64_t stridePl, int rows, int k,
                                                                    const int* deficB) {
    const int b = blockIdx.y;
    const int j = blockIdx.x;
    if (!deficB[static_cast<int64_t>(b) * k + j]) return;
    uint16_t* pl = planesb + static_cast<int64_t>(b) * stridePl + static_cast<int64_t>(j) * ldpl;
    const float scale = 1.0f / sqrtf(static_cast<float>(rows));
    for (int i = threadIdx.x; i < rows; i += blockDim.x) {
        const uint64_t h = mix64((static_cast<uint64_t>(j) << 32) | static_cast<uint32_t>(i));
        uint16_t h1, h2, h3;
        split3_rn((h & 1ULL) ? scale : -scale, h1, h2, h3);
        pl[i] = h1;
        pl[planeStride + i] = h2;
        pl[2 * planeStride + i] = h3;
    }
}

}  // namespace

hipError_t launch_cholesky(double* C, int k, int64_t strideC, float* rinv32, double* xinv,
                           int64_t strideInv, int* defic, double* diag0, double tau_rel, int batch,
                           hipStream_t stream) {
    const int nb = (k + CB - 1) / CB;
    const bool inv = rinv32 != nullptr;
    hipLaunchKernelGGL(chol_diag_kernel, dim3(batch, k > CB ? 2 : 1), dim3(CT), 0, stream, C, k, strideC, diag0, defic,
                       xinv, rinv32, strideInv, tau_rel);
    for (int J = 0; J < nb; ++J) {
        const int n = nb - J - 1;
        const int px = n + (inv ? J : 0);
        if (px > 0)
            hipLaunchKernelGGL(chol_panel_x_kernel, dim3(px, batch), dim3(CT), 0, stream, C, k, strideC, J, n, defic,
                               xinv, rinv32, strideInv);
        if (n > 0)
            hipLaunchKernelGGL(chol_trailing_p_kernel, dim3(n * (n + 1) / 2 + (inv ? (J + 1) * n : 0), batch),
                               dim3(CT), 0, stream, C, k, strideC, J, nb, diag0, defic, xinv, rinv32, strideInv,
                               tau_rel);
    }
    return hipGetLastError();
}

hipError_t launch_fill_deficient(float* Q, int rows, int k, int64_t strideQ, const int* defic,
                                 int batch, hipStream_t stream) {
    hipLaunchKernelGGL(fill_deficient_kernel, dim3(k, batch), dim3(256), 0, stream, Q, rows, k,
                       strideQ, defic);
    return hipGetLastError();
}

hipError_t launch_fill_deficient_planes(uint16_t* planes, int64_t ldpl, int64_t planeStride, int64_t stridePl,
                                        int rows, int k, const int* defic, int batch, hipStream_t stream) {
    hipLaunchKernelGGL(fill_deficient_planes_kernel, dim3(k, batch), dim3(256), 0, stream, planes, ldpl, planeStride,
                       stridePl, rows, k, defic);
    return hipGetLastError();
}

}  // namespace galore
