// Small SVD of the projected matrix B = Q^T A (k x l) in the randomized SVD
// (Halko et al. 2011, direct SVD of the small matrix; paper §4.1.2).
//
// The left singular vectors of B are the eigenvectors of B B^T = Z^T Z with
// Z = A^T Q = B^T. The host factors that Gram in fp64 as R^T R (Cholesky), so
// they are also the left singular vectors of Y = R^T (k x k). One-sided
// (Hestenes) Jacobi rotates the columns of Y until they are mutually
// orthogonal: Y W = U Sigma, so sigma_j is the norm of column j and u_j the
// column divided by it; no rotation needs to be accumulated. Y is stored by
// columns (column c contiguous), which is exactly the row-major upper
// triangle of R.
//
// Blocked for the GPU: the k columns form blocks of 32; a round-robin
// tournament pairs the blocks so that every step is a set of disjoint pairs
// (with an odd number of blocks, the pair with the padding block is not
// launched). A step is one launch, one workgroup per pair and matrix, which
//   1. forms the 64 x 64 Gram of its two blocks: 32-row chunks split exactly
//      into three bf16 planes in LDS, six plane products per tile on the bf16
//      matrix cores (v_mfma_f32_16x16x32_bf16) summed in fp32 per chunk and
//      in fp64 across chunks;
//   2. skips the pair if every column pair is already orthogonal to the
//      tolerance (relative off-diagonal), otherwise
//   3. if every rotation the Gram asks for is small, takes them all at once
//      (Theta = polar factor of I + E, four small matrix-core products), else
//      reduces the small Gram by one sweep of two-sided Jacobi held in
//      registers (fp32 entries, fp64 diagonal and angles; 63 rounds of 32
//      disjoint rotations, accumulating the rotation Theta), and
//   4. applies Theta to the pair's 64 columns of Y on the bf16 matrix cores,
//      Theta and the 32-row chunks of Y split into three planes as in 1.
// A launch of few workgroups runs them with four groups of four waves, the
// row chunks of phases 1 and 4 dealt out to the groups (same bits).
// A sweep is nb - 1 steps; the matrix has converged when a whole sweep
// rotates nothing (rotation counts per sweep live in device memory, so no
// host synchronisation is needed).
//
// Rank deficiency: a pivot the Cholesky found dependent zeroes a row of R,
// i.e. a column of Y; zero columns are never rotated and stay exactly zero.
// If one of them is among the r leading columns, the finalize kernel replaces
// it by an orthonormal completion (unit vectors orthogonalised twice against
// the columns already kept), the singular value staying 0.
#include <float.h>

#include <type_traits>

#include "common.hpp"
#include "dispatch.hpp"

namespace galore {
namespace {

constexpr int JB = kJacobiBlock;   // columns per block
constexpr int JW = 2 * JB;         // columns per pair (64)
constexpr int JT = 256;            // threads (4 waves)
constexpr int PD = JW + 1;         // padded LDS row

static_assert(JW == 64, "the pair kernels assume 64 columns per pair");

__device__ __forceinline__ int ring_slot(int pos, int step, int n) {
    // circle method: slot 0 fixed, the others rotate by one per step
    if (pos == 0) return 0;
    int v = (pos - 1 - step) % (n - 1);
    if (v < 0) v += n - 1;
    return 1 + v;
}

// Power-of-two exponent e of each matrix with 2^e sqrt(max_j d_j) in [1/2, 1),
// d = the diagonal of the Gram Z^T Z that R factors (the squared column norms
// of B^T). Y = R^T enters the sweeps as 2^e R^T: the fp32 columns and the
// fp32 matrix-core partial sums of their Gram then neither underflow nor
// overflow whatever the gradient's scale (a gradient with singular values near
// 1e-20 would otherwise give partial products below the fp32 range and pass
// as converged), and sigma is scaled back by 2^-e, exactly. A zero or
// non-finite maximum gives e = 0.
__global__ __launch_bounds__(256) void jacobi_scale_kernel(const double* diagb, int k, int* expb) {
    const int b = blockIdx.x;
    const double* d = diagb + static_cast<int64_t>(b) * k;
    __shared__ double red[4];
    double mx = 0.0;
    for (int i = threadIdx.x; i < k; i += blockDim.x) mx = fmax(mx, d[i]);   // fmax drops NaN
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        int e = 0;
        if (mx > 0.0 && mx <= DBL_MAX) {
            int ex;
            frexp(sqrt(mx), &ex);      // sqrt(mx) = f 2^ex, f in [1/2, 1)
            e = -ex;
        }
        expb[b] = e;
    }
}

__global__ __launch_bounds__(256) void jacobi_prepare_kernel(const double* Rb, int k,
                                                             int64_t strideR, float* Ytb,
                                                             int64_t strideX, int* rotb,
                                                             int max_sweeps, const int* expb) {
    const int b = blockIdx.y;
    const double* R = Rb + static_cast<int64_t>(b) * strideR;
    float* Yt = Ytb + static_cast<int64_t>(b) * strideX;
    const int e = expb[b];
    if (blockIdx.x == 0 && threadIdx.x < static_cast<unsigned>(max_sweeps))
        rotb[static_cast<int64_t>(b) * max_sweeps + threadIdx.x] = 0;
    const int64_t total = static_cast<int64_t>(k) * k;
    // column c of Y = R^T is row c of R
    for (int64_t pos = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; pos < total;
         pos += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int c = static_cast<int>(pos / k);
        const int i = static_cast<int>(pos - static_cast<int64_t>(c) * k);
        Yt[pos] = (i >= c) ? static_cast<float>(ldexp(R[pos], e)) : 0.0f;
    }
}

// Jacobi rotation (c, s) that zeroes the off-diagonal of [[a, g], [g, b]]
// under column p' = c p - s q, q' = s p + c q: t = tan(theta) is the smaller
// root of t^2 + 2 zeta t - 1 = 0, zeta = (b - a) / (2 g) (Rutishauser's
// form), b - a taken in fp64. The rotation is applied to fp32 entries, so
// fp32 suffices for the rest: the hardware reciprocal, square root and
// reciprocal square root (c = 1 / sqrt(1 + t^2), s = c t: c^2 + s^2 = 1 to a
// few fp32 ulp). The angle only has to be close: a residual off-diagonal is
// removed by later sweeps, and every visit recomputes the pair's Gram from the
// columns in fp64. |zeta| past the fp32 range gives t = 0.
__device__ __forceinline__ void rotation(double a, double b, float g, float& c, float& s) {
    const float zf = static_cast<float>(b - a) * 0.5f * __builtin_amdgcn_rcpf(g);
    const float az = fabsf(zf);
    float tf = __builtin_amdgcn_rcpf(az + __builtin_amdgcn_sqrtf(fmaf(az, az, 1.0f)));   // |zeta| huge: 0
    tf = (zf >= 0.0f) ? tf : -tf;                                                         // sign(0) = +1
    c = __builtin_amdgcn_rsqf(fmaf(tf, tf, 1.0f));
    s = c * tf;
}

// ---- bf16 planes of the pair's columns (Gram and rotation phases) ----------
// A 32-row chunk of the pair's 64 columns is held in LDS as three bf16 planes
// (h, m, l with x = h + m + l exactly: each plane takes the leading 8
// significant bits of what the previous ones left, by truncation, and an fp32
// significand has 24). Plane p of buffer s starts at s * kChunkBytes +
// p * kPlaneBytes; column c is 64 bytes (32 rows), its row octet o stored at
// 16-byte slot o ^ ((c >> 2) & 3), which keeps the 16-byte fragment reads, the
// transposing reads and the stores free of bank conflicts.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int PC = 32;                         // rows per plane chunk
constexpr int kPlaneBytes = JW * PC * 2;
constexpr int kChunkBytes = 3 * kPlaneBytes;
// plane products kept: h h, h m, m h, m m, h l, l h (the others are below
// 2^-25 of |a| |b|)
constexpr int kPlanePairs[6][2] = {{0, 0}, {0, 1}, {1, 0}, {1, 1}, {0, 2}, {2, 0}};

__device__ __forceinline__ void split8(f32x4 a, f32x4 b, bf16x8& h, bf16x8& m, bf16x8& l) {
    const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    u32x4 ph, pm, pl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned u0 = __float_as_uint(x[2 * i]), u1 = __float_as_uint(x[2 * i + 1]);
        const float r0 = x[2 * i] - __uint_as_float(u0 & 0xffff0000u);
        const float r1 = x[2 * i + 1] - __uint_as_float(u1 & 0xffff0000u);
        const unsigned v0 = __float_as_uint(r0), v1 = __float_as_uint(r1);
        const float q0 = r0 - __uint_as_float(v0 & 0xffff0000u);
        const float q1 = r1 - __uint_as_float(v1 & 0xffff0000u);
        // the upper halves of two words in one
        ph[i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        pm[i] = __builtin_amdgcn_perm(v1, v0, 0x07060302u);
        pl[i] = __builtin_amdgcn_perm(__float_as_uint(q1), __float_as_uint(q0), 0x07060302u);
    }
    h = __builtin_bit_cast(bf16x8, ph);
    m = __builtin_bit_cast(bf16x8, pm);
    l = __builtin_bit_cast(bf16x8, pl);
}

struct Rows8 {
    f32x4 a, b;
};
// entries 0 .. 7 of src (zeros past `left` of them); vec: 16-byte aligned
__device__ __forceinline__ Rows8 pair_fetch(const float* src, int left, bool vec) {
    if (vec && left >= 8)
        return Rows8{*reinterpret_cast<const f32x4*>(src), *reinterpret_cast<const f32x4*>(src + 4)};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (e < left) ? src[e] : 0.0f;
    return Rows8{f32x4{v[0], v[1], v[2], v[3]}, f32x4{v[4], v[5], v[6], v[7]}};
}

// thread t stages rows 8 (t & 3) .. + 7 of the chunk of pair column t >> 2
__device__ __forceinline__ void pair_stash(unsigned char* lds, int s, int tid, Rows8 r) {
    bf16x8 h, m, l;
    split8(r.a, r.b, h, m, l);
    const int c = tid >> 2, o = tid & 3;
    unsigned char* dst = lds + s * kChunkBytes + c * 64 + 16 * (o ^ ((c >> 2) & 3));
    *reinterpret_cast<bf16x8*>(dst) = h;
    *reinterpret_cast<bf16x8*>(dst + kPlaneBytes) = m;
    *reinterpret_cast<bf16x8*>(dst + 2 * kPlaneBytes) = l;
}

// Gram operand (A and B alike) of 16-column block blk: lane l holds column
// 16 blk + (l & 15), rows 8 (l >> 4) .. + 7 of the chunk
__device__ __forceinline__ bf16x8 gram_frag(const unsigned char* lds, int s, int p, int blk, int lane) {
    const int c = 16 * blk + (lane & 15), o = lane >> 4;
    return *reinterpret_cast<const bf16x8*>(lds + s * kChunkBytes + p * kPlaneBytes + c * 64 +
                                            16 * (o ^ ((c >> 2) & 3)));
}

// Rotation operand A (rows of Y_P): lane l holds row 16 tm + (l & 15) of the
// chunk, columns 32 ks + 8 (l >> 4) .. + 7. Two transposing reads: in each
// group of 16 lanes, lane j receives element j % 4 of the 8 bytes that lane
// 4 e + j / 4 points at (e = 0..3); lane L points at column w0 + L / 4, rows
// 16 tm + 4 (L % 4) .. + 3, so lane j gets row 16 tm + j, columns w0 .. w0 + 3.
__device__ __forceinline__ bf16x8 apply_frag(const unsigned char* lds, int s, int p, int tm, int ks, int lane) {
    const int L = lane & 15;
    const int t = 16 * tm + 4 * (L & 3);
    bf16x4 q[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int w = 32 * ks + 8 * (lane >> 4) + 4 * h + (L >> 2);
        const int off = s * kChunkBytes + p * kPlaneBytes + w * 64 + 16 * ((t >> 3) ^ ((w >> 2) & 3)) + 2 * (t & 7);
        q[h] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(
            reinterpret_cast<__attribute__((address_space(3))) unsigned char*>(reinterpret_cast<size_t>(lds)) + off));
    }
    return __builtin_shufflevector(q[0], q[1], 0, 1, 2, 3, 4, 5, 6, 7);
}

// The inner sweep's Gram and accumulated rotation are fp32: the rotation is
// applied to fp32 columns (split exactly into planes), and the sweep only has to
// produce an orthogonal Theta that reduces the pair's off-diagonal. The pair
// Gram, the convergence test, the diagonal the sweep carries and the rotation
// angles' differences stay fp64, so pairs are judged converged (and the last
// sweeps are steered) at fp64 accuracy.

// Angles at and below which a pair's rotations are taken all at once: every
// |E_ij| <= kSmallAngle and the sum of E_ij^2 over i < j <= kSmallSum. The terms
// are cut off to units of 2^-24, so the true sum may be 2016 units, 1.2e-4, larger:
// |E|_2^2 <= 0.02262, |E|_2 <= 0.1504 (an antisymmetric matrix's singular values
// come in pairs).
constexpr float kSmallAngle = 0.1f;
constexpr float kSmallSum = 0.0225f;
// below (|P|_2 <= 2.43e-4 with the cut-off): two products give Theta to fp32
// rounding, off an orthogonal matrix by 3/8 |P|^2 < 2.3e-8
constexpr float kTinySum = 1.0f / 8192.0f;
constexpr int SP = JW + 4;                   // row pitch of E and S (fp32): 16-byte rows, fragment reads on distinct banks

// LDS of one group of four waves, reused phase by phase: two plane chunks, the
// fp64 Gram, the inner sweep's exchange arrays, E and S, Theta
constexpr int kPairLds = 2 * JW * SP * static_cast<int>(sizeof(float));
static_assert(2 * kChunkBytes <= kPairLds && JW * PD * static_cast<int>(sizeof(double)) <= kPairLds, "phases fit");

// Row chunks of segment g of four: [seg_begin(n, g), seg_begin(n, g + 1)). The
// Gram is summed segment by segment (fp64), in the same order whether one
// group of waves walks all four or four groups take one each.
__device__ __forceinline__ int seg_begin(int nchunk, int g) { return (g * nchunk) >> 2; }

// A step's rotations all at once. For columns i, j of the pair with Gram G a
// Jacobi rotation of angle E_ij = g_ij / (g_jj - g_ii) removes g_ij to first
// order; when all of them are small their joint rotation is the orthogonal
// polar factor of I + E (E antisymmetric),
//   Theta = (I + E)(I - E^2)^(-1/2) = (I + E)(I + S),
//   S = P/2 + 3/8 P^2 + 5/16 P^3 + ...,  P = E^2,
// off an orthogonal matrix by 35/128 |P|^4 < 7.2e-8. Second-order terms are left
// for the next sweep, as a sweep of single rotations leaves them: in a CPU
// model of these sweeps (six spectra, k = 136 .. 528, the exact SVD among
// them) the number of sweeps is unchanged and the number of pair rotations
// grows by 0-2%, and 40-60% of the pair visits take this form, the later
// sweeps nearly all. fp32 matrix-core products (v_mfma_f32_16x16x4_f32), every
// operand read by rows: P and S are symmetric and E is antisymmetric. On entry
// E is in LDS; on exit Theta (fp32, row pitch PD) is. `tiles` of the 64 x 64
// outputs: row tile wr, column tiles wc .. wc + NT - 1 of this wave.
template <int NT>
__device__ __forceinline__ void small_angle_theta(unsigned char* smem, int wr, int wc, int lane, bool tiny) {
    float (*E)[SP] = reinterpret_cast<float (*)[SP]>(smem);
    float (*S)[SP] = reinterpret_cast<float (*)[SP]>(smem + JW * SP * sizeof(float));
    const int l15 = lane & 15, lk = lane >> 4;
    float fe[16], fp[16];   // row 16 wr + l15 of E and of P, entries 4 s + lk
    f32x4 acc[NT];
    auto product = [&](const float* fa, const float (*B)[SP]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 16; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[s], B[16 * (wc + t) + l15][4 * s + lk], acc[t], 0, 0, 0);
    };
    // a tile's rows 16 wr + 4 lk + v of column 16 (wc + t) + l15, stored as the
    // four consecutive entries of that row of the (symmetric) matrix
    auto store_sym = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(&S[16 * (wc + t) + l15][16 * wr + 4 * lk]) = acc[t];
    };
    auto add_diag = [&](float c) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (wr == wc + t && l15 == 4 * lk + v) acc[t][v] += c;
    };
#pragma unroll
    for (int s = 0; s < 16; ++s) fe[s] = E[16 * wr + l15][4 * s + lk];
    product(fe, E);                                   // E E^T = -P
    if (tiny) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] *= -0.5f;   // S = P / 2
        store_sym();
        __syncthreads();
    } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] *= -1.0f;
        store_sym();
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 16; ++s) fp[s] = S[16 * wr + l15][4 * s + lk];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] *= 0.3125f;
        add_diag(0.375f);
        store_sym();                                  // 3/8 + 5/16 P
        __syncthreads();
        product(fp, S);
        add_diag(0.5f);
        __syncthreads();
        store_sym();                                  // 1/2 + 3/8 P + 5/16 P^2
        __syncthreads();
        product(fp, S);
        __syncthreads();
        store_sym();                                  // S
        __syncthreads();
    }
    f32x4 keep[NT];                                   // I + E + S, in the tiles' layout
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        keep[t] = *reinterpret_cast<const f32x4*>(&S[16 * (wc + t) + l15][16 * wr + 4 * lk]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * wr + 4 * lk + v, j = 16 * (wc + t) + l15;
            keep[t][v] += E[i][j] + (i == j ? 1.0f : 0.0f);
        }
    }
    product(fe, S);                                   // E S
    __syncthreads();                                  // Theta overwrites E
    float (*Tf)[PD] = reinterpret_cast<float (*)[PD]>(smem);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) Tf[16 * wr + 4 * lk + v][16 * (wc + t) + l15] = keep[t][v] + acc[t][v];
    __syncthreads();
}

// v of lane x ^ M within each 16 lanes (M = 1, 2: quad permutations)
template <int M>
__device__ __forceinline__ float lane_xor(float v) {
    static_assert(M == 1 || M == 2, "quad permutations");
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), M == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}
template <int M>
__device__ __forceinline__ int lane_xor(int v) {
    return __builtin_amdgcn_mov_dpp(v, M == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true);
}
template <int M>
__device__ __forceinline__ double lane_xor(double v) {
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = lane_xor<M>(static_cast<int>(u)), hi = lane_xor<M>(static_cast<int>(u >> 32));
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}
// v of the lane whose byte address (4 times its number) is a
__device__ __forceinline__ int lane_at(int a, int v) { return __builtin_amdgcn_ds_bpermute(a, v); }
__device__ __forceinline__ float lane_at(int a, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(a, __float_as_int(v)));
}
__device__ __forceinline__ double lane_at(int a, double v) {
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = lane_at(a, static_cast<int>(u)), hi = lane_at(a, static_cast<int>(u >> 32));
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// One sweep of two-sided Jacobi on the 64 x 64 Gram (upper triangle, fp64, in
// LDS on entry), held in registers; on exit the accumulated rotation Theta (fp32, row pitch
// PD) is in LDS. All four waves of a group; ACTIVE = false runs the barriers
// alone.
//
// The 64 columns sit in 32 positions of two, A and B; a round rotates the 32
// pairs (A_p, B_p). Wave w holds positions 8 w .. 8 w + 7; lane x + 32 h (x <
// 32) the rows of A_x and B_x of the Gram, and rows x and 32 + x of Theta, at
// the eight columns of positions 8 w + 4 h .. + 3: both rows and both columns
// of a rotation are in one lane, so a round's rotations are 96 multiply-adds
// a lane with no lane moves. The pair's diagonal entries are carried along
// exactly (2 x 2 formulas, fp64); its off-diagonal entry is read from its
// holder (one LDS word, one barrier a round).
// Between rounds the B side is permuted by p -> p ^ m: m = 1, 2 are register
// renames for the columns and quad permutations for the rows; every fourth
// round m = 7, 15 or 16 goes through LDS. m steps through a Gray code of the
// basis {1, 2, 7, 15, 16}, so 32 rounds meet every A with every B. Then A and
// B are paired anew across bit 4 (A_p with A_p^16, B_p with B_p^16) and 16
// rounds do the same within the halves, and so on down: 32 + 16 + 8 + 4 + 2 +
// 1 = 63 rounds, in which every pair of columns meets once.
// (One row a lane, 64 odd-even rounds with a lane move per value and round,
// took 46 us of the visit in a workgroup alone on its CU; this form 30 us.)
constexpr int kSweepScratch = JW * SP * static_cast<int>(sizeof(float));   // past Theta and the exchanged columns
static_assert(JW * PD * static_cast<int>(sizeof(float)) <= kSweepScratch && 32 * 32 * 16 <= kSweepScratch &&
                  kSweepScratch + 2048 <= kPairLds, "sweep scratch");

template <bool ACTIVE>
__device__ __forceinline__ void inner_sweep(unsigned char* smem, int wave, int lane) {
    const double (*G)[PD] = reinterpret_cast<const double (*)[PD]>(smem);
    f32x4 (*Xb)[32] = reinterpret_cast<f32x4 (*)[32]>(smem);                          // exchanged columns by position
    float (*gx)[32] = reinterpret_cast<float (*)[32]>(smem + kSweepScratch);          // [2] off-diagonals, ping-pong
    float2 (*cs)[32] = reinterpret_cast<float2 (*)[32]>(smem + kSweepScratch + 256);  // [4 waves] (c, s), wave-private
    int (*ids)[32] = reinterpret_cast<int (*)[32]>(smem + kSweepScratch + 1280);      // [2] columns held by A and B
    const int x = lane & 31, h = lane >> 5;
    const int p0 = 8 * wave + 4 * h;             // this lane's first position
    const bool holder = (x >> 2) == (p0 >> 2);   // position x's columns are this lane's
    float gAA[4], gAB[4], gBA[4], gBB[4];        // Gram rows A_x, B_x at columns A_p, B_p of position p0 + j
    float t0A[4], t0B[4], t1A[4], t1B[4];        // Theta rows x, 32 + x
    double da = 0.0, db = 0.0;                   // the diagonal entries of A_x and B_x
    int ia = x, ib = 32 + x;                     // the columns they are
    if constexpr (ACTIVE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = p0 + j;
            const int lo = min(x, p), hi = max(x, p);
            gAA[j] = static_cast<float>(G[lo][hi]);
            gAB[j] = static_cast<float>(G[x][32 + p]);
            gBA[j] = static_cast<float>(G[p][32 + x]);
            gBB[j] = static_cast<float>(G[32 + lo][32 + hi]);
            t0A[j] = t1B[j] = (x == p) ? 1.0f : 0.0f;
            t0B[j] = t1A[j] = 0.0f;
        }
        da = G[x][x];
        db = G[32 + x][32 + x];
    }
    __syncthreads();                             // the exchange arrays overwrite the Gram
    int buf = 0;
    float g = 0.0f;                              // the coming round's off-diagonal of position x
    float cj[4], sj[4];                          // the round's rotations of the lane's positions
    // p' = c p - s q, q' = s p + c q
    auto turn2 = [](float& p, float& q, float cc, float ss) {
        const float u = cc * p - ss * q;
        q = ss * p + cc * q;
        p = u;
    };
    // position x's next off-diagonal, at the holder's column B_(x ^ M), to every wave
    auto put = [&](auto mc) __attribute__((always_inline)) {
        constexpr int M = decltype(mc)::value;
        if constexpr (ACTIVE) {
            const float v01 = (x & 1) ? gAB[1 ^ M] : gAB[M], v23 = (x & 1) ? gAB[3 ^ M] : gAB[2 ^ M];
            if (holder) gx[buf][x] = (x & 2) ? v23 : v01;
        }
    };
    auto get = [&]() __attribute__((always_inline)) {
        __syncthreads();
        if constexpr (ACTIVE) g = gx[buf][x];
        buf ^= 1;
    };
    auto publish = [&]() __attribute__((always_inline)) {
        put(std::integral_constant<int, 0>());
        get();
    };
    // a round's rotations: the rows and the A_x row's columns first (the next
    // off-diagonal is among them) ...
    auto rotate_a = [&]() __attribute__((always_inline)) {
        if constexpr (ACTIVE) {
            const double gd = g;
            float c, s;
            rotation(da, db, g, c, s);
            const bool turn = gd * gd > 1e-30 * (da * db);
            c = turn ? c : 1.0f;
            s = turn ? s : 0.0f;
            if (h == 0) cs[wave][x] = make_float2(c, s);
            // the wave's own LDS writes and reads are in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const f32x4 q01 = *reinterpret_cast<const f32x4*>(&cs[wave][p0]);
            const f32x4 q23 = *reinterpret_cast<const f32x4*>(&cs[wave][p0 + 2]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                turn2(gAA[j], gBA[j], c, s);
                turn2(gAB[j], gBB[j], c, s);
            }
            const double cr = c, sr = s;
            const double cs2 = 2.0 * cr * sr * gd;
            const double na = cr * cr * da - cs2 + sr * sr * db;
            db = sr * sr * da + cs2 + cr * cr * db;
            da = na;
            cj[0] = q01[0], sj[0] = q01[1], cj[1] = q01[2], sj[1] = q01[3];
            cj[2] = q23[0], sj[2] = q23[1], cj[3] = q23[2], sj[3] = q23[3];
#pragma unroll
            for (int j = 0; j < 4; ++j) turn2(gAA[j], gAB[j], cj[j], sj[j]);
        }
    };
    // ... then the B_x row's and Theta's columns
    auto rotate_b = [&]() __attribute__((always_inline)) {
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) turn2(gBA[j], gBB[j], cj[j], sj[j]);
        }
    };
    auto rotate_t = [&]() __attribute__((always_inline)) {
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                turn2(t0A[j], t0B[j], cj[j], sj[j]);
                turn2(t1A[j], t1B[j], cj[j], sj[j]);
            }
        }
    };
    auto rotate = [&]() __attribute__((always_inline)) {
        rotate_a();
        rotate_b();
        rotate_t();
    };
    auto swap1 = [](float& u, float& v) {
        const float w = u;
        u = v;
        v = w;
    };
    // B_p -> position p ^ M, M = 1 or 2
    auto flip = [&](auto mc) __attribute__((always_inline)) {
        constexpr int M = decltype(mc)::value;
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((j & M) != 0) continue;
                swap1(gAB[j], gAB[j ^ M]);
                swap1(gBB[j], gBB[j ^ M]);
                swap1(t0B[j], t0B[j ^ M]);
                swap1(t1B[j], t1B[j ^ M]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gBA[j] = lane_xor<M>(gBA[j]);
                gBB[j] = lane_xor<M>(gBB[j]);
            }
            db = lane_xor<M>(db);
            ib = lane_xor<M>(ib);
        }
    };
    // the rows of a move across positions p ^ m: `both` sides' rows change
    // places (a new pairing), or B's alone move
    auto move_rows = [&](int m, bool pairing) __attribute__((always_inline)) {
        if constexpr (ACTIVE) {
            const int src = 4 * (lane ^ m);
            const bool up = pairing && (x & m) != 0;   // these lanes give and take A, the others B
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float va = lane_at(src, (pairing && !up) ? gBA[j] : (pairing ? gAA[j] : gBA[j]));
                const float vb = lane_at(src, (pairing && !up) ? gBB[j] : (pairing ? gAB[j] : gBB[j]));
                gAA[j] = up ? va : gAA[j];
                gAB[j] = up ? vb : gAB[j];
                gBA[j] = up ? gBA[j] : va;
                gBB[j] = up ? gBB[j] : vb;
            }
            const double vd = lane_at(src, (pairing && up) ? da : db);
            const int vi = lane_at(src, (pairing && up) ? ia : ib);
            da = up ? vd : da;
            ia = up ? vi : ia;
            db = up ? db : vd;
            ib = up ? ib : vi;
        }
    };
    // a move across p ^ m, m >= 4: the columns through LDS
    auto exchange = [&](int m, bool pairing) __attribute__((always_inline)) {
        const bool up = pairing && (p0 & m) != 0;      // uniform over the lane's four positions
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                Xb[p0 + j][x] = up ? f32x4{gAA[j], gBA[j], t0A[j], t1A[j]} : f32x4{gAB[j], gBB[j], t0B[j], t1B[j]};
        }
        __syncthreads();
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 v = Xb[(p0 + j) ^ m][x];
                gAA[j] = up ? v[0] : gAA[j];
                gBA[j] = up ? v[1] : gBA[j];
                t0A[j] = up ? v[2] : t0A[j];
                t1A[j] = up ? v[3] : t1A[j];
                gAB[j] = up ? gAB[j] : v[0];
                gBB[j] = up ? gBB[j] : v[1];
                t0B[j] = up ? t0B[j] : v[2];
                t1B[j] = up ? t1B[j] : v[3];
            }
        }
        move_rows(m, pairing);
    };
    // a new pairing across bit 2 or 1 of the position: register renames
    auto pair_low = [&](auto mc) __attribute__((always_inline)) {
        constexpr int M = decltype(mc)::value;
        if constexpr (ACTIVE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((j & M) != 0) continue;            // B_j with A_(j + M)
                swap1(gAB[j], gAA[j ^ M]);
                swap1(gBB[j], gBA[j ^ M]);
                swap1(t0B[j], t0A[j ^ M]);
                swap1(t1B[j], t1A[j ^ M]);
            }
        }
        move_rows(M, true);
    };
    using std::integral_constant;
    // a round, then B_p -> position p ^ M (M = 1 or 2): the next off-diagonal
    // is written before the rest of the round's work and read behind it
    auto round_flip = [&](auto mc) __attribute__((always_inline)) {
        rotate_a();
        put(mc);
        __builtin_amdgcn_sched_barrier(0);
        rotate_b();
        get();
        __builtin_amdgcn_sched_barrier(0);
        rotate_t();
        flip(mc);
    };
    auto four_rounds = [&]() __attribute__((always_inline)) {
        round_flip(integral_constant<int, 1>());
        round_flip(integral_constant<int, 2>());
        round_flip(integral_constant<int, 1>());
        rotate();
    };
    publish();
    // moves after each four rounds, a nibble each from the lowest: 7, 15, 16, or
    // a new pairing across bit 4, 3 (value 8) or 2 (value 4); the last four
    // rounds (positions of two bits) follow
    constexpr uint64_t kMoves = 0x47A7F7B7F7E7F7ULL;
    for (int i = 0; i < 14; ++i) {
        four_rounds();
        const int mv = static_cast<int>((kMoves >> (4 * i)) & 15);
        if (mv == 0x7 || mv == 0xF) exchange(mv, false);
        else if (mv == 0xE) exchange(16, false);
        else exchange(mv == 0xB ? 16 : (mv == 0xA ? 8 : 4), true);
        publish();
    }
    four_rounds();
    pair_low(integral_constant<int, 2>());
    publish();
    round_flip(integral_constant<int, 1>());
    rotate();
    pair_low(integral_constant<int, 1>());
    publish();
    rotate();
    if constexpr (ACTIVE) {
        if (wave == 0 && h == 0) {
            ids[0][x] = ia;
            ids[1][x] = ib;
        }
    }
    __syncthreads();
    if constexpr (ACTIVE) {
        float (*Tf)[PD] = reinterpret_cast<float (*)[PD]>(smem);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ca = ids[0][p0 + j], cb = ids[1][p0 + j];
            Tf[x][ca] = t0A[j];
            Tf[x][cb] = t0B[j];
            Tf[32 + x][ca] = t1A[j];
            Tf[32 + x][cb] = t1B[j];
        }
    }
    __syncthreads();
}

// Step of the block Jacobi (one workgroup per pair and matrix): Gram of the
// pair's 64 columns, convergence test, reduction of the small Gram, rotation
// of the columns, all in one LDS buffer per group of four waves (see above).
// NG groups: 1, four workgroups per CU; or 4 (one workgroup per CU), for steps
// of few workgroups (wide_pairs in dispatch.hpp): the chunk loops of the
// two phases over memory wait a memory latency per chunk, which only other
// workgroups of the CU would hide, so four groups walk a quarter of the chunks
// each. The results are the same bits. One 4096x11008 update (k = 1056, 16
// workgroups a launch), per launch: 99 us with the inner sweep before and 61 us
// now, 36 us with small rotations only, 25 and 15 us where nothing rotates.
template <int NG>
__global__ __launch_bounds__(JT * NG, NG == 1 ? 4 : 1) void jacobi_pair_kernel(float* Xtb, int k, int64_t strideX,
                                                                               int nb, int step, int sweep, int* rotb,
                                                                               int max_sweeps, double tol,
                                                                               int skip_dummy, const int* jpermb) {
    static_assert(NG == 1 || NG == 4, "one group of four waves, or one per segment");
    const int b = blockIdx.y;
    int* rot = rotb + static_cast<int64_t>(b) * max_sweeps;
    if (sweep > 0 && rot[sweep - 1] == 0) return;     // converged in an earlier sweep
    const int tid = threadIdx.x & (JT - 1);           // thread of its group
    const int lane = threadIdx.x & 63;
    const int gwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = gwave & 3;                       // wave of its group
    const int grp = gwave >> 2;
    int h = blockIdx.x;
    if (skip_dummy) {
        // the padding block nb - 1 holds no columns: its pair is not launched
        // (every column pair inside a real block is still reduced by the inner
        // sweeps of that block's other pairs)
        const int pos = 1 + (step + nb - 2) % (nb - 1);
        const int hd = (pos < nb / 2) ? pos : nb - 1 - pos;
        h += (h >= hd) ? 1 : 0;
    }
    const int bi = ring_slot(h, step, nb);
    const int bj = ring_slot(nb - 1 - h, step, nb);
    const float* Xt = Xtb + static_cast<int64_t>(b) * strideX;

    __shared__ __attribute__((aligned(16))) unsigned char smem[NG * kPairLds];
    double (*G)[PD] = reinterpret_cast<double (*)[PD]>(smem);
    __shared__ int col[JW];
    __shared__ int sum_s;

    if (threadIdx.x < JW) {
        // logical column c of the sweep's order -> stored column jperm[c]
        const int blk = (tid < JB) ? bi : bj;
        const int c = blk * JB + (tid & (JB - 1));
        col[tid] = (c < k) ? jpermb[static_cast<int64_t>(b) * k + c] : -1;
        if (tid == 0) sum_s = 0;
    }
    __syncthreads();

    unsigned char* lds = smem + grp * kPairLds;
    const int nchunk = (k + PC - 1) / PC;
    // this group's chunks, and the loop length common to all groups
    const int ch0 = NG == 1 ? 0 : seg_begin(nchunk, grp);
    const int nch = NG == 1 ? nchunk : seg_begin(nchunk, grp + 1) - ch0;
    const int nit = NG == 1 ? nchunk : (nchunk + 3) / 4;
    // this thread's column and its first row in a chunk (none for a padding column)
    const int mycol = col[tid >> 2];
    const int myrow = ch0 * PC + 8 * (tid & 3);
    const int myrows = mycol >= 0 ? k - myrow : 0;   // rows from there on
    const int64_t myoff = static_cast<int64_t>(max(mycol, 0)) * k + myrow;
    const bool vec4 = (k & 3) == 0;
    Rows8 pre;   // the next chunk, in flight
    auto fetch = [&](const float* src, int it) {
        if (it < nch) pre = pair_fetch(src + myoff + it * PC, myrows - it * PC, vec4);
    };

    // ---- 1. Gram of the pair's columns on the bf16 matrix cores: every
    //         32-row chunk of the 64 columns is split exactly into three bf16
    //         planes (x = h + m + l, 8 significant bits each, so the split of
    //         an fp32 value loses nothing) and staged in LDS, double-buffered,
    //         the next chunk in flight in registers. A 16 x 16 tile of the Gram
    //         sums the six plane products h h, h m, m h, m m, h l, l h
    //         (v_mfma_f32_16x16x32_bf16; the three left out are below 2^-25 of
    //         |y_p| |y_q|) in fp32 per chunk, each chunk's sum added into fp64.
    //         Tiles per wave: waves 0 and 1 the three upper tiles of blocks
    //         {0, 1} and {2, 3}, waves 2 and 3 the tiles (0, 2), (1, 2) and
    //         (0, 3), (1, 3), so a wave reads the fragments of at most three
    //         16-column blocks.
    {
        f64x4 acc[3], tot[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) acc[x] = tot[x] = f64x4{0.0, 0.0, 0.0, 0.0};
        fetch(Xt, 0);
        if (nch > 0) pair_stash(lds, 0, tid, pre);
        __syncthreads();
        const bool diag = wave < 2;
        const int a0 = (wave == 1) ? 2 : 0, a1 = a0 + 1, bb = wave;     // bb: third block of waves 2, 3
        for (int it = 0; it < nit; ++it) {
            const int s = it & 1;
            fetch(Xt, it + 1);
            if (NG == 1 || it < nch) {
                bf16x8 f0[3], f1[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    f0[p] = gram_frag(lds, s, p, a0, lane);
                    f1[p] = gram_frag(lds, s, p, a1, lane);
                }
                if (diag) {
                    f32x4 part[3];
#pragma unroll
                    for (int x = 0; x < 3; ++x) part[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        const int pa = kPlanePairs[q][0], pb = kPlanePairs[q][1];
                        part[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0[pa], f0[pb], part[0], 0, 0, 0);
                        part[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0[pa], f1[pb], part[1], 0, 0, 0);
                        part[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f1[pa], f1[pb], part[2], 0, 0, 0);
                    }
#pragma unroll
                    for (int x = 0; x < 3; ++x) acc[x] += __builtin_convertvector(part[x], f64x4);
                } else {
                    bf16x8 f2[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) f2[p] = gram_frag(lds, s, p, bb, lane);
                    f32x4 part[2];
#pragma unroll
                    for (int x = 0; x < 2; ++x) part[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int q = 0; q < 6; ++q) {
                        const int pa = kPlanePairs[q][0], pb = kPlanePairs[q][1];
                        part[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0[pa], f2[pb], part[0], 0, 0, 0);
                        part[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f1[pa], f2[pb], part[1], 0, 0, 0);
                    }
#pragma unroll
                    for (int x = 0; x < 2; ++x) acc[x] += __builtin_convertvector(part[x], f64x4);
                }
            }
            if constexpr (NG == 1) {
                // end of a segment: add its sum to the total
                const int e = it + 1;
                if (e == seg_begin(nchunk, 1) || e == seg_begin(nchunk, 2) || e == seg_begin(nchunk, 3) || e == nchunk) {
#pragma unroll
                    for (int x = 0; x < 3; ++x) {
                        tot[x] += acc[x];
                        acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
                    }
                }
            }
            if (it + 1 < nch) pair_stash(lds, s ^ 1, tid, pre);
            __syncthreads();
        }
        // 16 x 16 block layout: lane holds column (lane & 15); accumulator
        // register v holds row 4 (lane >> 4) + v. The planes are dead: the
        // last barrier above ends every read of them.
        double (*Gp)[PD] = reinterpret_cast<double (*)[PD]>(lds);
        const int ntile = diag ? 3 : 2;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            if (x < ntile) {
                const int ti = diag ? ((x == 2) ? a1 : a0) : ((x == 0) ? a0 : a1);
                const int tj = diag ? ((x == 0) ? a0 : a1) : bb;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + 4 * (lane >> 4) + v;
                    const int j = 16 * tj + (lane & 15);
                    const double g = NG == 1 ? tot[x][v] : acc[x][v];
                    Gp[i][j] = g;
                    Gp[j][i] = g;
                }
            }
        }
        __syncthreads();
        if constexpr (NG == 4) {
            const double (*G1)[PD] = reinterpret_cast<const double (*)[PD]>(smem + kPairLds);
            const double (*G2)[PD] = reinterpret_cast<const double (*)[PD]>(smem + 2 * kPairLds);
            const double (*G3)[PD] = reinterpret_cast<const double (*)[PD]>(smem + 3 * kPairLds);
            for (int idx = threadIdx.x; idx < JW * JW; idx += JT * NG) {
                const int i = idx >> 6, j = idx & 63;
                G[i][j] = ((G[i][j] + G1[i][j]) + G2[i][j]) + G3[i][j];
            }
            __syncthreads();
        }
    }

    // ---- 2. convergence test: every column pair orthogonal to the tolerance?
    //         |g_pq| <= tol sqrt(g_pp g_qq), compared squared; a pair with a
    //         zero column never counts, a pair with a NaN or Inf entry always
    //         does (non-finite input must not pass as converged: such a matrix
    //         runs every sweep and reports the sweep limit)
    // The same pass forms the angles E of the joint rotation (a coupling of
    // columns of nearly equal norm has a large angle however small it is and
    // calls for the sweep: left unrotated at 1e-7 of the norms, it turned such
    // columns by up to 0.02) and their squares' sum, in whole units of 2^-24 so that the
    // sum does not depend on its order. E goes into the Gram's lower triangle,
    // which nothing reads from here on.
    bool small, tiny;
    {
        const double tol2 = tol * tol;
        int need = 0, big = 0, fsum = 0;
#pragma unroll 2
        for (int idx = threadIdx.x; idx < JW * JW; idx += JT * NG) {
            const int p = idx >> 6, q = idx & 63;
            if (q > p) {
                float ev = 0.0f;
                const double a = G[p][p], c = G[q][q];
                const double dd = a * c;
                const double gpq = G[p][q];
                if (dd != 0.0) {
                    const bool ok = dd <= DBL_MAX && gpq * gpq <= tol2 * dd;
                    if (!ok) need = 1;
                    const double d = c - a;
                    const bool fits = fabs(gpq) <= static_cast<double>(kSmallAngle) * fabs(d);
                    if (!fits) {
                        big = 1;
                    } else if (gpq != 0.0) {
                        if (!(fabs(d) > 1e-30 && fabs(d) < 1e30)) {
                            big = 1;
                        } else {
                            ev = static_cast<float>(gpq) * __builtin_amdgcn_rcpf(static_cast<float>(d));
                            fsum += static_cast<int>(ev * ev * 16777216.0f);
                        }
                    }
                }
                G[q][p] = ev;
            }
        }
        need = __syncthreads_or(need);
        if (threadIdx.x == 0 && need) atomicAdd(&rot[sweep], 1);
        if (!need) return;
        for (int o = 32; o > 0; o >>= 1) fsum += __shfl_xor(fsum, o);
        if (lane == 0 && fsum != 0) atomicAdd(&sum_s, fsum);
        big = __syncthreads_or(big);
        const int total = sum_s;
        small = !big && total <= static_cast<int>(kSmallSum * 16777216.0f);
        tiny = total <= static_cast<int>(kTinySum * 16777216.0f);
    }

    if (small) {
        float (*E)[SP] = reinterpret_cast<float (*)[SP]>(smem);
        float ev[16 / NG];
#pragma unroll
        for (int e = 0; e < 16 / NG; ++e) {
            const int idx = static_cast<int>(threadIdx.x) + e * JT * NG;
            const int p = idx >> 6, q = idx & 63;
            const float v = static_cast<float>(G[max(p, q)][min(p, q)]);
            ev[e] = (q > p) ? v : ((q < p) ? -v : 0.0f);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16 / NG; ++e) {
            const int idx = static_cast<int>(threadIdx.x) + e * JT * NG;
            E[idx >> 6][idx & 63] = ev[e];
        }
        __syncthreads();
        small_angle_theta<4 / NG>(smem, wave, NG == 1 ? 0 : grp, lane, tiny);
    } else if (NG > 1 && grp > 0) {
        // the inner sweep is the first group's; the others keep its barriers
        inner_sweep<false>(smem, wave, lane);
    } else {
        // ---- 3. one sweep of two-sided Jacobi on the 64 x 64 Gram
        inner_sweep<true>(smem, wave, lane);
    }
    // ---- 4. Y_P <- Y_P Theta on the bf16 matrix cores: Theta split into
    //         three planes once (the wave's B fragments stay in registers),
    //         32-row chunks of Y_P split and staged as in the Gram, the A
    //         fragments (8 consecutive columns of one row) read with the
    //         transposing LDS read; six plane products per output, as in the
    //         Gram. Wave (tm, tn) writes rows 16 tm .. 16 tm + 15 of each chunk,
    //         columns 32 tn .. 32 tn + 31 (two 16 x 16 tiles), a lane four
    //         consecutive rows of one column per tile.
    {
        const int tm = wave >> 1, tn = wave & 1;
        const float (*Tf)[PD] = reinterpret_cast<const float (*)[PD]>(smem);   // Theta[w][c], fp32
        bf16x8 bq[2][2][3];   // [column tile][K step of 32][plane]
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int c = 32 * tn + 16 * ct + (lane & 15);
                const int w0 = 32 * ks + 8 * (lane >> 4);
                f32x4 t0, t1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    t0[v] = Tf[w0 + v][c];
                    t1[v] = Tf[w0 + 4 + v][c];
                }
                split8(t0, t1, bq[ct][ks][0], bq[ct][ks][1], bq[ct][ks][2]);
            }
        __syncthreads();                       // the Y_P planes overwrite Theta
        float* Y = Xtb + static_cast<int64_t>(b) * strideX;
        fetch(Y, 0);
        if (nch > 0) pair_stash(lds, 0, tid, pre);
        __syncthreads();
        const int cst[2] = {col[32 * tn + (lane & 15)], col[32 * tn + 16 + (lane & 15)]};
        for (int it = 0; it < nit; ++it) {
            const int s = it & 1;
            const int r0 = (ch0 + it) * PC;
            fetch(Y, it + 1);
            if (NG == 1 || it < nch) {
                f32x4 acc[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 af[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) af[p] = apply_frag(lds, s, p, tm, ks, lane);
#pragma unroll
                    for (int q = 0; q < 6; ++q)
#pragma unroll
                        for (int ct = 0; ct < 2; ++ct)
                            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[kPlanePairs[q][0]],
                                                                              bq[ct][ks][kPlanePairs[q][1]], acc[ct],
                                                                              0, 0, 0);
                }
                // rows r0 + 16 tm + 4 (lane >> 4) + v of column cst[ct]
                const int rr = r0 + 16 * tm + 4 * (lane >> 4);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    const int c = cst[ct];
                    if (c >= 0) {
                        float* dst = Y + static_cast<int64_t>(c) * k + rr;
                        if (vec4 && rr + 4 <= k) {
                            *reinterpret_cast<f32x4*>(dst) = acc[ct];
                        } else {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                if (rr + v < k) dst[v] = acc[ct][v];
                        }
                    }
                }
            }
            if (it + 1 < nch) pair_stash(lds, s ^ 1, tid, pre);
            __syncthreads();
        }
    }
}

// norms[b][c] = |y_c| in fp64, one wave per column (coalesced over the
// column's k contiguous entries); grid (ceil(k / 4), batch). Between sweeps
// (rotb != NULL) a matrix whose previous sweep rotated nothing is skipped.
__global__ __launch_bounds__(256) void jacobi_norms_kernel(const float* Ytb, int k, int64_t strideX,
                                                           double* normsb, const int* rotb, int max_sweeps,
                                                           int sweep) {
    const int b = blockIdx.y;
    if (rotb != nullptr && sweep > 0 && rotb[static_cast<int64_t>(b) * max_sweeps + sweep - 1] == 0) return;
    const int c = 4 * blockIdx.x + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (c >= k) return;
    const float* y = Ytb + static_cast<int64_t>(b) * strideX + static_cast<int64_t>(c) * k;
    double s = 0.0;
    for (int i = lane; i < k; i += 64) s += static_cast<double>(y[i]) * static_cast<double>(y[i]);
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) normsb[static_cast<int64_t>(b) * k + c] = sqrt(s);
}

// The order of the columns for the coming sweep: by decreasing norm (ties
// by index; a NaN norm counts as -1, last), jperm[b][rank] = column. Sweeping
// the blocks of a norm-ordered matrix pairs columns of like size first and
// cuts the rotations the later sweeps need (about 17% fewer pair rotations
// and one sweep fewer on the 4096 x 11008 workload in a CPU model of these
// sweeps). The rank of column c is the number of columns ahead of it, counted by
// eight threads a column, 32 columns a workgroup, each with the matrix's norms
// in LDS (k = 1056: 8 us; one thread a column took 36 us, one workgroup of
// 1024 threads per matrix 63-124 us a sweep); converged matrices are skipped.
__global__ __launch_bounds__(256) void jacobi_order_kernel(const double* normsb, int k, int* jpermb,
                                                           const int* rotb, int max_sweeps, int sweep) {
    const int b = blockIdx.y;
    if (sweep > 0 && rotb[static_cast<int64_t>(b) * max_sweeps + sweep - 1] == 0) return;
    extern __shared__ unsigned char smem[];
    double* nv = reinterpret_cast<double*>(smem);
    for (int c = threadIdx.x; c < k; c += blockDim.x) {
        const double v = normsb[static_cast<int64_t>(b) * k + c];
        nv[c] = (v == v) ? v : -1.0;
    }
    __syncthreads();
    const int c = 32 * blockIdx.x + (threadIdx.x >> 3);
    const double vc = nv[min(c, k - 1)];
    int rank = 0;
#pragma unroll 4
    for (int c2 = threadIdx.x & 7; c2 < k; c2 += 8) {
        const double v2 = nv[c2];
        rank += (v2 > vc) || (v2 == vc && c2 < c);
    }
    for (int o = 4; o > 0; o >>= 1) rank += __shfl_xor(rank, o);
    if ((threadIdx.x & 7) == 0 && c < k) jpermb[static_cast<int64_t>(b) * k + rank] = c;
}

// Xa[j][:] = y_perm(j) / sigma_perm(j) (row j of the result contiguous) for the
// matrices finalize marked refinable; one workgroup per row j; grid (k, batch)
__global__ __launch_bounds__(256) void jacobi_gather_kernel(const float* Ytb, int k, int64_t strideX,
                                                            const double* normsb, const int* permb,
                                                            const int* flags, float* Xab) {
    const int b = blockIdx.y;
    if (flags[b] == 0) return;
    const int j = blockIdx.x;
    const int c = permb[static_cast<int64_t>(b) * k + j];
    const double inv = 1.0 / normsb[static_cast<int64_t>(b) * k + c];
    const float* y = Ytb + static_cast<int64_t>(b) * strideX + static_cast<int64_t>(c) * k;
    float* x = Xab + static_cast<int64_t>(b) * strideX + static_cast<int64_t>(j) * k;
    for (int i = threadIdx.x; i < k; i += blockDim.x) x[i] = static_cast<float>(static_cast<double>(y[i]) * inv);
}

// sigma_j = |y_j| (fp64), order descending (ties by index, NaN last);
// Ur[:, j] = y_perm(j) / sigma_perm(j) for the r leading columns, zero columns
// completed orthonormally. scratch: 2 k + r doubles per matrix.
__global__ __launch_bounds__(256) void jacobi_finalize_kernel(const float* Ytb, int k, int64_t strideX,
                                                              int r, float* Urb, int64_t strideUr,
                                                              float* sigma, int64_t stride_sigma,
                                                              const int* rotb, int max_sweeps, int nsweeps, int* info,
                                                              double* scratchb, int64_t strideScratch,
                                                              const int* expb, const double* normsb, const int* permb,
                                                              int* flags) {
    extern __shared__ unsigned char smem[];
    double* sig = reinterpret_cast<double*>(smem);
    int* perm = reinterpret_cast<int*>(sig + k);
    __shared__ double red[4];
    __shared__ int nkeep_s;
    const int b = blockIdx.x;
    const float* Yt = Ytb + static_cast<int64_t>(b) * strideX;
    float* Ur = Urb + static_cast<int64_t>(b) * strideUr;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    // the descending order of the norms (ties by index, NaN last), ranked by
    // jacobi_order_kernel into permb before this kernel
    for (int c = tid; c < k; c += blockDim.x) {
        sig[c] = normsb[static_cast<int64_t>(b) * k + c];
        perm[c] = permb[static_cast<int64_t>(b) * k + c];
    }
    if (tid == 0) nkeep_s = r;
    __syncthreads();
    // kept columns: up to the first that is zero or NaN
    for (int j = tid; j < r; j += blockDim.x)
        if (!(sig[perm[j]] > 0.0)) {
            atomicMin(&nkeep_s, j);
            break;
        }
    if (sigma != nullptr) {
        for (int j = tid; j < r; j += blockDim.x) {
            const double v = ldexp(sig[perm[j]], -expb[b]);     // undo the sweeps' scaling
            sigma[static_cast<int64_t>(b) * stride_sigma + j] = (v > 0.0 || v != v) ? static_cast<float>(v) : 0.0f;
        }
    }
    __syncthreads();
    const int nkeep = nkeep_s;
    // refinable: every column norm finite and positive; those matrices get all
    // k ordered columns (jacobi_gather_kernel, from permb) and their Ur from the
    // fp64 refinement; the others (rank-deficient, non-finite) keep the vectors
    // written here
    const bool refinable = flags != nullptr && (nkeep == r) && sig[perm[k - 1]] > 0.0 && sig[perm[0]] <= DBL_MAX;
    if (flags != nullptr && tid == 0) flags[b] = refinable ? 1 : 0;
    if (!refinable) {
        const int64_t total = static_cast<int64_t>(k) * nkeep;
        for (int64_t pos = tid; pos < total; pos += blockDim.x) {
            const int i = static_cast<int>(pos / nkeep);
            const int j = static_cast<int>(pos - static_cast<int64_t>(i) * nkeep);
            const int c = perm[j];
            Ur[static_cast<int64_t>(i) * r + j] =
                static_cast<float>(static_cast<double>(Yt[static_cast<int64_t>(c) * k + i]) / sig[c]);
        }
    }
    if (info != nullptr) {
        // 0: converged; kInfoSweepLimit: none of the nsweeps sweeps run came
        // out rotation-free; kInfoNonFinite: a column norm is NaN or Inf
        // (non-finite input)
        const int* rot = rotb + static_cast<int64_t>(b) * max_sweeps;
        int bad = 0;
        for (int c = tid; c < k; c += blockDim.x) bad |= !(sig[c] <= DBL_MAX);
        const int free_sweep = __syncthreads_or(tid < nsweeps && rot[tid] == 0);
        bad = __syncthreads_or(bad);
        if (tid == 0) info[b] = bad ? kInfoNonFinite : (free_sweep ? 0 : kInfoSweepLimit);
    }
    if (nkeep >= r) return;
    // ---- orthonormal completion of columns nkeep .. r-1 (rank-deficient B) ----
    // Each new column starts from the unit vector e_i least covered by the
    // columns kept so far (smallest squared row norm rn2[i], so its residual
    // 1 - rn2[i] is the largest, at least (k - j) / k), is orthogonalised twice
    // against them (classical Gram-Schmidt) and normalised.
    __syncthreads();
    double* v = scratchb + static_cast<int64_t>(b) * strideScratch;   // k
    double* dots = v + k;                                              // r
    double* rn2 = dots + r;                                            // k
    __shared__ double bestv[4];
    __shared__ int besti[4];
    for (int i = tid; i < k; i += blockDim.x) {
        double a = 0.0;
        for (int m = 0; m < nkeep; ++m) {
            const double u = Ur[static_cast<int64_t>(i) * r + m];
            a += u * u;
        }
        rn2[i] = a;
    }
    __syncthreads();
    for (int j = nkeep; j < r; ++j) {
        // argmin of rn2 (lowest index on ties)
        double bv = 1e300;
        int bi = k;
        for (int i = tid; i < k; i += blockDim.x)
            if (rn2[i] < bv) { bv = rn2[i]; bi = i; }
        for (int o = 32; o > 0; o >>= 1) {
            const double ov = __shfl_xor(bv, o);
            const int oi = __shfl_xor(bi, o);
            if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { bestv[wave] = bv; besti[wave] = bi; }
        __syncthreads();
        int cand = besti[0];
        double cv = bestv[0];
        for (int w = 1; w < 4; ++w)
            if (bestv[w] < cv || (bestv[w] == cv && besti[w] < cand)) { cv = bestv[w]; cand = besti[w]; }
        for (int i = tid; i < k; i += blockDim.x) v[i] = (i == cand) ? 1.0 : 0.0;
        __syncthreads();
        for (int pass = 0; pass < 2; ++pass) {
            for (int m = tid; m < j; m += blockDim.x) {
                double d = 0.0;
                for (int i = 0; i < k; ++i) d += static_cast<double>(Ur[static_cast<int64_t>(i) * r + m]) * v[i];
                dots[m] = d;
            }
            __syncthreads();
            for (int i = tid; i < k; i += blockDim.x) {
                double x = v[i];
                for (int m = 0; m < j; ++m) x -= dots[m] * static_cast<double>(Ur[static_cast<int64_t>(i) * r + m]);
                v[i] = x;
            }
            __syncthreads();
        }
        double nn = 0.0;
        for (int i = tid; i < k; i += blockDim.x) nn += v[i] * v[i];
        for (int o = 32; o > 0; o >>= 1) nn += __shfl_xor(nn, o);
        if (lane == 0) red[wave] = nn;
        __syncthreads();
        const double norm = sqrt(red[0] + red[1] + red[2] + red[3]);
        const double inv = (norm > 0.0) ? 1.0 / norm : 0.0;
        for (int i = tid; i < k; i += blockDim.x) {
            const double u = v[i] * inv;
            Ur[static_cast<int64_t>(i) * r + j] = static_cast<float>(u);
            rn2[i] += u * u;
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_jacobi_prepare(const double* R, int k, int64_t strideR, float* Yt, int64_t strideX,
                                 int* rot, int max_sweeps, const double* diag, int* exps, int batch,
                                 hipStream_t stream) {
    hipLaunchKernelGGL(jacobi_scale_kernel, dim3(batch), dim3(256), 0, stream, diag, k, exps);
    int64_t blocks = (static_cast<int64_t>(k) * k + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(jacobi_prepare_kernel, dim3(static_cast<unsigned>(blocks), batch), dim3(256),
                       0, stream, R, k, strideR, Yt, strideX, rot, max_sweeps, exps);
    return hipGetLastError();
}

hipError_t launch_jacobi_order(const float* Yt, int k, int64_t strideX, double* norms, int* jperm, const int* rot,
                               int max_sweeps, int sweep, int batch, hipStream_t stream) {
    hipLaunchKernelGGL(jacobi_norms_kernel, dim3((k + 3) / 4, batch), dim3(256), 0, stream, Yt, k, strideX, norms, rot,
                       max_sweeps, sweep);
    hipLaunchKernelGGL(jacobi_order_kernel, dim3((k + 31) / 32, batch), dim3(256), static_cast<size_t>(k) * sizeof(double),
                       stream, norms, k, jperm, rot, max_sweeps, sweep);
    return hipGetLastError();
}

hipError_t launch_jacobi_step(float* Yt, int k, int64_t strideX, int nblocks, int step, int sweep, int* rot,
                              int max_sweeps, double tol, const int* jperm, int batch, int in_flight,
                              hipStream_t stream) {
    const int pairs = step_pairs(k, JB);
    const int skip_dummy = nblocks / 2 - pairs;   // the padding block's pair
    if (wide_pairs(k, pairs, batch, in_flight))
        hipLaunchKernelGGL(jacobi_pair_kernel<4>, dim3(pairs, batch), dim3(4 * JT), 0, stream, Yt, k, strideX, nblocks,
                           step, sweep, rot, max_sweeps, tol, skip_dummy, jperm);
    else
        hipLaunchKernelGGL(jacobi_pair_kernel<1>, dim3(pairs, batch), dim3(JT), 0, stream, Yt, k, strideX, nblocks,
                           step, sweep, rot, max_sweeps, tol, skip_dummy, jperm);
    return hipGetLastError();
}

hipError_t launch_jacobi_finalize(const float* Yt, int k, int64_t strideX, int r, float* Ur, int64_t strideUr,
                                  float* sigma, int64_t stride_sigma, const int* rot, int max_sweeps, int nsweeps,
                                  int* info,
                                  double* scratch, int64_t strideScratch, const int* exps, double* norms,
                                  int* perm, float* Xa, int* flags, int batch, hipStream_t stream) {
    hipLaunchKernelGGL(jacobi_norms_kernel, dim3((k + 3) / 4, batch), dim3(256), 0, stream, Yt, k, strideX, norms,
                       static_cast<const int*>(nullptr), 0, 0);
    // their descending order into perm (sweep 0: no convergence check)
    hipLaunchKernelGGL(jacobi_order_kernel, dim3((k + 31) / 32, batch), dim3(256), static_cast<size_t>(k) * sizeof(double),
                       stream, norms, k, perm, static_cast<const int*>(nullptr), 0, 0);
    const size_t shmem = static_cast<size_t>(k) * (sizeof(double) + sizeof(int));
    hipLaunchKernelGGL(jacobi_finalize_kernel, dim3(batch), dim3(256), shmem, stream, Yt, k, strideX, r, Ur,
                       strideUr, sigma, stride_sigma, rot, max_sweeps, nsweeps, info, scratch, strideScratch, exps,
                       norms,
                       perm, flags);
    if (Xa != nullptr)
        hipLaunchKernelGGL(jacobi_gather_kernel, dim3(k, batch), dim3(256), 0, stream, Yt, k, strideX, norms, perm,
                           flags, Xa);
    return hipGetLastError();
}

}  // namespace galore
