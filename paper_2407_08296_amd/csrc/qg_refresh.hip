// Subspace refresh (Sec. 3.2: the projection matrix is recomputed from the current gradient; the paper takes the
// first r left singular vectors from an SVD).  Here one pass of orthogonal iteration started from the stored INT4
// projection replaces the SVD:
//     R = dequant(P)^T G  (the projection kernel of the optimizer step)      bf16 MFMA
//     Z = bf16(R)
//     Y = G Z^T           (m x r)                                            bf16 MFMA, fp32 accumulation (qg_tile_gemm.h)
//     Q = Y T^-1          with Y = Q T, T upper triangular, diag(T) > 0      fp64 MFMA (Cholesky QR)
//     P <- quant_int4(Q)  (Sec. 3.3)
// followed by the cosine check of Sec. 3.2 between the old and the new P.
//
// The orthonormalisation works on the r x r Gram matrix S = Y^T Y in fp64: S = L L^T (blocked Cholesky, 64-wide
// blocks), X = L^-1, Q = Y X^T, and all of that a second time on the result (Cholesky QR twice): one round leaves
// |Q^T Q - I| ~ 1e-16 * cond(Y)^2, which for the low-rank-plus-noise gradients this is made for (cond(Y) up to 1e7)
// is far from orthonormal; the second round starts from a matrix with cond ~ 1 and lands within fp32 rounding of
// the Gram-Schmidt factor, because multiplying Y from the right by a triangular matrix with a positive diagonal
// does not change that factor.  Each Gram matrix gets a shift of 2^-46 of its trace on the diagonal, which keeps
// the first round's pivots positive for cond(Y) well beyond 1e8 at no cost in the result.  A column that is
// numerically dependent on its predecessors (a last-round pivot no larger than the shift) is reported through
// `info`; every kernel runs to completion whatever the data.
#include "qg_cossim.h"
#include "qg_tile_gemm.h"

namespace qg {

int launch_project_batch(const ProjBatch& batch, int count, float* R, int64_t strideR, int64_t m, int64_t n, int64_t ld,
                         int64_t r, hipStream_t stream);   // qg_gemm.hip
int launch_project(const uint8_t* Pq, const float* Ps, const uint16_t* G, float* R, int64_t m, int64_t n, int64_t ld,
                   int64_t r, hipStream_t stream);        // qg_gemm.hip

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int kNB = 64;               // block size of the fp64 kernels: one workgroup (4 waves) per 64 x 64 block
constexpr int kKC = 16;               // K extent staged in LDS per barrier pair: 20 KB of LDS per workgroup
constexpr int kPitchKF = kKC + 1;     // LDS pitch of a [64][k] chunk (k fastest): odd, so that the 16 rows a fragment
                                      // read touches at one k fall on 16 different bank pairs (36 gave 4-way conflicts)

// ROWS x COLS block at (row0, col0) of a row-major matrix (fp32 or fp64) -> registers -> LDS doubles.  Elements
// outside [0, rows) x [0, cols) read as zero.  col0 and cols are even, so an element pair never straddles the edge.
template <int ROWS, int COLS, int PITCH, typename T>
struct BlockStage {
    static constexpr int PER = ROWS * COLS / 2 / 256;
    static_assert(ROWS * COLS % 512 == 0, "256 threads, two elements each");
    T v[PER][2];   // (as fetched: converted when written to LDS, so that nothing waits for the load before)
    __device__ __forceinline__ void fetch(const T* __restrict__ src, int64_t ld, int row0, int col0, int rows, int cols) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int idx = threadIdx.x + 256 * q;
            const int gr = row0 + idx / (COLS / 2), gc = col0 + (idx % (COLS / 2)) * 2;
            v[q][0] = v[q][1] = T(0);
            if (gr < rows && gc < cols) {
                typedef T pair_t __attribute__((ext_vector_type(2)));
                const pair_t p = *reinterpret_cast<const pair_t*>(src + (int64_t)gr * ld + gc);
                v[q][0] = p[0];
                v[q][1] = p[1];
            }
        }
    }
    // place(row): the row of dst that row `row` of the block goes to
    template <typename Place>
    __device__ __forceinline__ void commit(double* dst, Place place) const {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int idx = threadIdx.x + 256 * q;
            double* d = dst + place(idx / (COLS / 2)) * PITCH + (idx % (COLS / 2)) * 2;
            d[0] = (double)v[q][0];
            d[1] = (double)v[q][1];
        }
    }
    __device__ __forceinline__ void commit(double* dst) const {
        commit(dst, [](int row) { return row; });
    }
};

// One K chunk (KC deep) of a 64 x 64 product of the factorization, a chain of a few chunks each.  Wave (wi, wj) owns a quadrant of W x W blocks
// of v_mfma_f64_16x16x4: lane l supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16]; register v of the
// result is element (i = 4 v + l / 16, j = l % 16).  Operand element (i, k) of A sits at At[i * a_pi + k * a_pk], element
// (k, j) of B at Bt[j * b_pj + k * b_pk].
template <int KC = kKC, int W>
__device__ __forceinline__ void mma_chunk(const double* At, int a_pi, int a_pk, const double* Bt, int b_pj, int b_pk,
                                          f64x4 (&acc)[W][W], int lane, int wi, int wj) {
    const double* ap = At + (wi * 16 * W + (lane & 15)) * a_pi + (lane >> 4) * a_pk;
    const double* bp = Bt + (wj * 16 * W + (lane & 15)) * b_pj + (lane >> 4) * b_pk;
#pragma unroll
    for (int k0 = 0; k0 < KC; k0 += 4) {
        double af[W], bf[W];
#pragma unroll
        for (int a = 0; a < W; ++a) af[a] = ap[a * 16 * a_pi + k0 * a_pk];
#pragma unroll
        for (int b = 0; b < W; ++b) bf[b] = bp[b * 16 * b_pj + k0 * b_pk];
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
            for (int b = 0; b < W; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
    }
}

template <int W>
__device__ __forceinline__ void zero_acc(f64x4 (&acc)[W][W]) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
}

// f(row, col, value) for every element of the wave's quadrant, row and col inside the workgroup's block.
template <int W, typename F>
__device__ __forceinline__ void for_each_acc(const f64x4 (&acc)[W][W], int lane, int wi, int wj, F f) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                f((wi * W + a) * 16 + 4 * v + (lane >> 4), (wj * W + b) * 16 + (lane & 15), acc[a][b][v]);
}

// The same product on v_mfma_f64_4x4x4, four independent 4 x 4 x 4 products: lane l supplies A[i = l % 4][k = l / 16] and
// B[k = l / 16][j = l % 4] of block l / 4 % 4 and gets D[i = l / 16][j = l % 4] of it.  Blocks 0, 1 and 2, 3 are given the same
// four rows, 0, 2 and 1, 3 the same four columns: 8 x 8 results of two fragments, a quadrant of 16 W x 16 W from 2 W + 2 W.
// On this chip it sustains 76 TFLOP/s on random operands, v_mfma_f64_16x16x4 36 to 50 (registers only, 8 waves per SIMD).
struct Lane4 {
    int a, b, i, j;   // row of A / column of B of the lane's fragment element, row / column of its result, in an 8 x 8 block
    __device__ __forceinline__ explicit Lane4(int lane)
        : a((lane >> 3 & 1) * 4 + (lane & 3)), b((lane >> 2 & 1) * 4 + (lane & 3)), i((lane >> 3 & 1) * 4 + (lane >> 4)), j(b) {}
};

// One K chunk, both operands [k][x]: a 16-byte read is two neighbouring x, so that fragment f of the 16 rows a pair of
// fragments covers holds rows 2 l.a + f (columns 2 l.b + f).
template <int KC, int PITCH, int W>
__device__ __forceinline__ void mma4_kslow(const double* At, const double* Bt, double (&acc)[2 * W][2 * W], int lane, int wi, int wj) {
    const Lane4 l(lane);
    const double* ap = At + (lane >> 4) * PITCH + wi * 16 * W + 2 * l.a;
    const double* bp = Bt + (lane >> 4) * PITCH + wj * 16 * W + 2 * l.b;
#pragma unroll
    for (int k0 = 0; k0 < KC; k0 += 4) {
        f64x2 af[W], bf[W];
#pragma unroll
        for (int a = 0; a < W; ++a) af[a] = *reinterpret_cast<const f64x2*>(ap + k0 * PITCH + 16 * a);
#pragma unroll
        for (int b = 0; b < W; ++b) bf[b] = *reinterpret_cast<const f64x2*>(bp + k0 * PITCH + 16 * b);
#pragma unroll
        for (int a = 0; a < 2 * W; ++a)
#pragma unroll
            for (int b = 0; b < 2 * W; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[a / 2][a % 2], bf[b / 2][b % 2], acc[a][b], 0, 0, 0);
    }
}

// Both operands [x][k]: a 16-byte read is two neighbouring k, of which an instruction takes four even or four odd ones.
// Fragment f of A holds rows 8 f + l.a of the quadrant, fragment f of B the rows of Bt (columns of the result) 8 f + l.b.
template <int KC, int PITCH, int W>
__device__ __forceinline__ void mma4_kfast(const double* At, const double* Bt, double (&acc)[2 * W][2 * W], int lane, int wi, int wj) {
    const Lane4 l(lane);
    const double* ap = At + (wi * 16 * W + l.a) * PITCH + 2 * (lane >> 4);
    const double* bp = Bt + (wj * 16 * W + l.b) * PITCH + 2 * (lane >> 4);
#pragma unroll
    for (int k0 = 0; k0 < KC; k0 += 8) {
        f64x2 af[2 * W], bf[2 * W];
#pragma unroll
        for (int a = 0; a < 2 * W; ++a) af[a] = *reinterpret_cast<const f64x2*>(ap + 8 * a * PITCH + k0);
#pragma unroll
        for (int b = 0; b < 2 * W; ++b) bf[b] = *reinterpret_cast<const f64x2*>(bp + 8 * b * PITCH + k0);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int a = 0; a < 2 * W; ++a)
#pragma unroll
                for (int b = 0; b < 2 * W; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[a][p], bf[b][p], acc[a][b], 0, 0, 0);
    }
}

// f(row, col, value) for every result of the wave's quadrant, row and col inside the workgroup's block.
template <bool KSLOW, int NF, typename F>
__device__ __forceinline__ void for_each_acc4(const double (&acc)[NF][NF], int lane, int wi, int wj, F f) {
    const Lane4 l(lane);
#pragma unroll
    for (int a = 0; a < NF; ++a)
#pragma unroll
        for (int b = 0; b < NF; ++b) {
            if constexpr (KSLOW) f(wi * 8 * NF + a / 2 * 16 + 2 * l.i + a % 2, wj * 8 * NF + b / 2 * 16 + 2 * l.j + b % 2, acc[a][b]);
            else f((wi * NF + a) * 8 + l.i, (wj * NF + b) * 8 + l.j, acc[a][b]);
        }
}

template <int W>
__device__ __forceinline__ void zero_acc4(double (&acc)[W][W]) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) acc[a][b] = 0.0;
}

// A batch of matrices with the same m and r runs through the fp64 kernels in one launch each (matrix b = blockIdx.z, or decoded
// from the tile number in k_gram and k_apply); its pieces sit at these element strides from matrix 0's (all zero for a single
// one).  The in and out matrices of a round share the stride Y/Q (both are m x r fp32 arrays of the same batch layout).
struct BatchStride {
    int64_t Y, Q, S, X, D, part, shift;
};

// 1 / sqrt(d) for d > 0 to fp64 accuracy: the hardware estimate and two Newton steps (the correctly rounded sqrt
// and divide of the library cost an order of magnitude more instructions, on the critical path of every column).
__device__ __forceinline__ double rsqrt_f64(double d) {
    double y = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = fma(-d * y, y, 1.0);      // 1 - d y^2
        y = fma(0.5 * y, e, y);
    }
    return y;
}

// 1 / d for d > 0: the hardware estimate and one step of third order.
__device__ __forceinline__ double rcp_f64(double d) {
    const double y = __builtin_amdgcn_rcp(d), e = fma(-d, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// (bi, bj) with bi >= bj of the idx-th block of a lower block triangle, rows first.
__device__ __forceinline__ void lower_pair(int idx, int& bi, int& bj) {
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= idx) ++i;
    bi = i;
    bj = idx - i * (i + 1) / 2;
}

// ---------------------------------------------------------------------------------------------------------------
// Z = bf16(R), round to nearest even
// ---------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_f32_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t quads) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < quads; i += (int64_t)gridDim.x * 256) {
        const f32x4 v = reinterpret_cast<const f32x4*>(x)[i];
        u32x2 o;
        o[0] = pack_bf16x2(v[0], v[1]);
        o[1] = pack_bf16x2(v[2], v[3]);
        reinterpret_cast<u32x2*>(y)[i] = o;
    }
}

// Energy that each column of a projection captures from the gradient: e[z][k] = sum_j R_z[k][j]^2 with
// R_z = P_z^T G_z (r rows of n elements, pitch ld, matrix z at R + z * strideR).  One workgroup per row; every thread
// adds its elements in index order, the 256 partial sums are added by a fixed tree: deterministic.
__global__ __launch_bounds__(256) void k_row_energy(const float* __restrict__ R, int64_t strideR, int n, int ld, int r,
                                                    float* __restrict__ e) {
    __shared__ float sh[256];
    const float* row = R + (int64_t)blockIdx.y * strideR + (int64_t)blockIdx.x * ld;
    float acc = 0.f;
    for (int j = threadIdx.x; j < n; j += 256) acc = __builtin_fmaf(row[j], row[j], acc);
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) e[(int64_t)blockIdx.y * r + blockIdx.x] = sh[0];
}

__global__ void k_set_i32(int32_t* p, int32_t v, int count) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = v;
}

// ---------------------------------------------------------------------------------------------------------------
// S = Y^T Y in fp64, lower block triangle only (Y fp32 m x r; S r x r row-major).  The m rows are cut into
// slices so that the launch fills the chip; slice s writes its partial sums to part + s * r * r and
// k_gram_reduce adds the slices in a fixed order (the result does not depend on scheduling).
// ---------------------------------------------------------------------------------------------------------------
constexpr int kGramMaxSlices = 8;

// The two products over m rows come with 64 x 64 blocks (TB) and 16- or 32-deep chunks for many workgroups, and with 32 x 32
// blocks and 64-deep chunks for few, where a workgroup's chain of chunks is what counts: a quarter of the MFMAs per chunk row,
// four times the workgroups, a quarter of the barriers.  The order of every sum is the same in both.
// Bound by the matrix pipe: sixteen 4096 x 4096, r = 1024 (73 GFLOP each launch) k_gram 1790 -> 1290 us (57 TFLOP/s), k_apply
// 1520 -> 1340 (54), against 16 x 16 x 4 instructions, tiles dealt over the XCDs one by one and, in both, a wait for the next
// chunk as soon as it was requested.  Measured beside it: k_gram with 32-deep chunks 1345, k_apply with 16-deep ones 1490; 128 x 128
// blocks in two LDS stages 1450 and, spilling, 1850; a higher wave priority in mma() no change.
template <int TB>
struct F64Tile {
    static constexpr int W = TB / 32;
    static constexpr int KC_GRAM = TB == kNB ? kKC : 64, KC_APPLY = TB == kNB ? 32 : 64;
    static constexpr int PITCH_KF = KC_APPLY + 2;            // [x][k] chunk, k fastest: 8 rows on 8 different groups of 4 banks
    static constexpr int PITCH_KS = TB + 16;                 // [k][x] chunk, k slowest
};

// The chunks of a workgroup from k_begin on: fetch(k) brings the operands of one into registers, commit() writes them to LDS,
// mma() multiplies.
template <int KC, typename FETCH, typename COMMIT, typename MMA>
__device__ __forceinline__ void f64_chunks(int k_begin, int k_end, FETCH fetch, COMMIT commit, MMA mma) {
    fetch(k_begin);
    for (int k = k_begin; k < k_end; k += KC) {
        commit();
        __syncthreads();
        if (k + KC < k_end) fetch(k + KC);
        mma();
        __syncthreads();
    }
}

template <int TB>
__global__ __launch_bounds__(256, TB == kNB ? 6 : 1) void k_gram(const float* __restrict__ Y, double* __restrict__ part, int m, int r,
                                              int slice_rows, uint32_t pairs, uint32_t slices, uint32_t tiles, BatchStride st) {
    using F = F64Tile<TB>;
    const uint32_t id = xcd_tile(blockIdx.x, gridDim.x);
    if (id >= tiles) return;
    const uint32_t slice = id / pairs % slices, z = id / pairs / slices;
    Y += z * st.Y;
    part += z * st.part;
    __shared__ __attribute__((aligned(16))) double At[F::KC_GRAM * F::PITCH_KS];
    __shared__ __attribute__((aligned(16))) double Bt[F::KC_GRAM * F::PITCH_KS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wi = wave >> 1, wj = wave & 1;
    int bi, bj;
    lower_pair(id % pairs, bi, bj);
    const bool diag = bi == bj;
    const int k_begin = slice * slice_rows, k_end = min(m, k_begin + slice_rows);
    double* S = part + (int64_t)slice * r * r;
    BlockStage<F::KC_GRAM, TB, F::PITCH_KS, float> sa, sb;
    double acc[2 * F::W][2 * F::W];
    zero_acc4(acc);
    f64_chunks<F::KC_GRAM>(k_begin, k_end,
        [&](int k) {
            sa.fetch(Y, r, k, bi * TB, k_end, r);
            if (!diag) sb.fetch(Y, r, k, bj * TB, k_end, r);
        },
        [&] {
            sa.commit(At);
            if (!diag) sb.commit(Bt);
        },
        [&] { mma4_kslow<F::KC_GRAM, F::PITCH_KS, F::W>(At, diag ? At : Bt, acc, lane, wi, wj); });
    const Lane4 l(lane);
#pragma unroll
    for (int a = 0; a < 2 * F::W; ++a)
#pragma unroll
        for (int b = 0; b < F::W; ++b) {
            const int gi = bi * TB + (wi * F::W + a / 2) * 16 + 2 * l.i + a % 2, gj = bj * TB + (wj * F::W + b) * 16 + 2 * l.j;
            if (gi < r && gj < r) *reinterpret_cast<f64x2*>(S + (int64_t)gi * r + gj) = f64x2{acc[a][2 * b], acc[a][2 * b + 1]};
        }
}

__global__ __launch_bounds__(256) void k_gram_reduce(const double* __restrict__ part, double* __restrict__ S, int r,
                                                     int slices, BatchStride st) {
    part += blockIdx.z * st.part;
    S += blockIdx.z * st.S;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)r * r) return;
    const int i = (int)(e / r), j = (int)(e % r);
    if (j / kNB > i / kNB) return;                 // above the lower block triangle: no sums (the factor is kept there, see below)
    double sum = 0.0;
    for (int s = 0; s < slices; ++s) sum += part[(int64_t)s * r * r + e];
    S[e] = sum;
}

// ---------------------------------------------------------------------------------------------------------------
// Blocked Cholesky S + sigma I = L L^T in place (lower triangle), right-looking, one block column per step kb:
//   chol_diag_block: L_kk from the diagonal block, and X_kk = L_kk^-1 (to Dinv[kb] and to the diagonal block of X)
//   k_chol_panel:    L_ik = S_ik X_kk^T for the blocks below, kept transposed as block (k, i) of S (whose upper triangle holds
//                    nothing else), so that S_ik stays what it is for all that read it in the same launch
//   k_chol_update:   S_ij -= L_ik L_jk^T for i >= j > kb, and in the same launch the next diagonal block (by the
//                    workgroup that has just updated it) and block row kb of X = L^-1
// Rows and columns at or past r (r not a multiple of 64) behave like an identity block.  A pivot that is not positive
// is replaced by 1 so that the factorization runs to completion whatever the data.
//
// sigma = 2^-46 trace(S) (at least 128 units of fp64 roundoff of the largest eigenvalue) keeps the pivots of a Gram
// matrix with cond(Y) beyond ~1e8 positive.  The shift changes L, not the factor Q in exact arithmetic (Y X^T for any
// triangular X with a positive diagonal has the same Gram-Schmidt factor); the second round, on a matrix with a far
// smaller condition number, removes what it costs in orthogonality.  Each diagonal block gets it when it is factored.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kSB = 16;               // sub-block of the diagonal block: one fp64 MFMA tile
constexpr int kPitchD = kNB + 1;      // LDS pitch of the diagonal block (odd: 16 rows of a fragment on 16 bank pairs)

constexpr int kPitchX = kSB + 1;      // ... of the inverses of its 16 x 16 diagonal blocks

// x of lane L of each row of 16 lanes, in all 16.
template <int L>
__device__ __forceinline__ double row_bcast_f64(double x) {
    long long b = __builtin_bit_cast(long long, x);
    b = __builtin_amdgcn_mov_dpp(b, 0x150 + L, 0xf, 0xf, true);   // row_newbcast:L
    return __builtin_bit_cast(double, b);
}

// f(0), ..., f(N - 1) with the index as a compile-time constant.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<N, I + 1>(f);
    }
}

// acc += A B for 16 x 16 blocks in LDS: element (i, k) of A at a[i * a_pi + k * a_pk], (k, j) of B at b[k * b_pk + j * b_pj].
__device__ __forceinline__ f64x4 mma16(const double* a, int a_pi, int a_pk, const double* b, int b_pk, int b_pj, f64x4 acc,
                                       int lane) {
    const double* ap = a + (lane & 15) * a_pi + (lane >> 4) * a_pk;
    const double* bp = b + (lane >> 4) * b_pk + (lane & 15) * b_pj;
#pragma unroll
    for (int k = 0; k < kSB; k += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k * a_pk], bp[k * b_pk], acc, 0, 0, 0);
    return acc;
}

// Sum of the diagonal of S (r x r), the same value in every thread; red: 4 doubles of LDS.
__device__ __forceinline__ double trace_of(const double* __restrict__ S, int r, double* red) {
    double acc = 0.0;
    for (int i0 = threadIdx.x; i0 < r; i0 += 1024) {
        double x[4];                                  // four loads in flight
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = i0 + 256 * q < r ? S[(int64_t)(i0 + 256 * q) * (r + 1)] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += x[q];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Factors the 64 x 64 block in T (pitch kPitchD, lower triangle, complete when called: no barrier needed before) and
// inverts the factor; writes X_kk to Dinv and X (nothing reads L_kk).  D: 4 * kSB * kPitchX doubles of LDS.  A serial chain
// of 64 pivots, so everything is arranged around its latency.  Per 16 columns: one wave eliminates the 16 x 16 diagonal block
// (lane % 16 = row) and, with the same multipliers, the identity beside it (lane % 16 = column of X_pp), which fills the
// chain's idle cycles; the pivot and the multipliers come from other lanes by DPP row broadcasts (all four rows of 16 lanes
// do the same, a broadcast does not leave its row).  Then L_ip = S_ip X_pp^T for the blocks below, and what is right of the 16
// columns together with block row p of X, from 16 x 16 fp64 MFMAs spread over the four waves.  k_chol_diag on one matrix, cycles:
// 34000, 3900 of them per 16 pivots (14 us); with all 64 rows in the chain and v_readlane, whose scalar registers spilled,
// 7000 per 16 pivots, the inverse afterwards 12500 and the load of T, one element at a time, 18000: 75000 (31 us).
__device__ __forceinline__ void chol_diag_block(double* T, double* D, int r, int kb, double* __restrict__ Dinv,
                                                double* __restrict__ X, int32_t* __restrict__ info, double sigma,
                                                double flag_factor) {
    constexpr int P = kPitchD, PX = kPitchX, NSB = kNB / kSB;
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, l4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int base = kb * kNB;
    // a pivot at or below flag_factor * sigma is reported: 0 in the first round (only pivots that are not positive),
    // 16 in the last, where a pivot that small is the shift alone, i.e. a column that is numerically dependent
    const double floor_d = flag_factor * sigma;
    if (t < kNB && base + t < r) T[t * P + t] += sigma;
    __syncthreads();
    for (int p = 0; p < NSB; ++p) {
        const int c0 = p * kSB;
        double* Dp = D + p * kSB * PX;
        if (wave == 0) {
            double b[kSB], x[kSB];
#pragma unroll
            for (int c = 0; c < kSB; ++c) {
                b[c] = T[(c0 + l16) * P + c0 + c];
                x[c] = c == l16 ? 1.0 : 0.0;
            }
            // U D U^T form: a reciprocal of the pivot is all that the chain from one pivot to the next needs; the square
            // roots are taken at the end, of all sixteen pivots at once (dv: lane % 16 = pivot)
            int bad = kSB;                              // first pivot that is too small, not positive, or NaN
            double dv = 1.0;
            double u = 0.0;                             // column j of U D over the pivot, of the pivot before
            static_for<kSB + 1>([&](auto jc) {          // per scheduling region: pivot j's chain, the rest of pivot j - 1
                constexpr int j = decltype(jc)::value;
                double u1 = 0.0;
                if constexpr (j > 0 && j + 1 < kSB) b[j + 1] = fma(-row_bcast_f64<j + 1>(u), b[j - 1], b[j + 1]);
                if constexpr (j < kSB) {
                    const double d = row_bcast_f64<j>(b[j]);
                    const bool positive = d > 0.0;
                    const double inv = positive ? rcp_f64(d) : 1.0;
                    if constexpr (j + 1 < kSB) b[j + 1] = fma(-(row_bcast_f64<j + 1>(b[j]) * b[j]), inv, b[j + 1]);
                    u1 = b[j] * inv;
                    bad = !(d > floor_d) && bad == kSB ? j : bad;
                    dv = l16 == j && positive ? d : dv;
                }
                if constexpr (j > 0)
                    static_for<kSB - j>([&](auto ic) {
                        constexpr int c = j + decltype(ic)::value;
                        const double l = row_bcast_f64<c>(u);
                        if constexpr (c > j + 1) b[c] = fma(-l, b[j - 1], b[c]);
                        x[c] = fma(-l, x[j - 1], x[c]);
                        asm volatile("" : "+v"(x[c]));   // (here, not where X_pp is stored, with every l kept until then)
                    });
                u = u1;
                __builtin_amdgcn_sched_barrier(0);
            });
            const double rs = rsqrt_f64(dv);
            static_for<kSB>([&](auto cc) { x[decltype(cc)::value] *= row_bcast_f64<decltype(cc)::value>(rs); });
            if (lane == 0 && bad < kSB && base + c0 + bad < r) atomicCAS(info, 0, base + c0 + bad + 1);
            if (lane < kSB) {
#pragma unroll
                for (int c = 0; c < kSB; ++c) Dp[c * PX + lane] = c >= lane ? x[c] : 0.0;
            }
        }
        __syncthreads();
        if (p + 1 + wave < NSB) {                       // L_ip = S_ip X_pp^T
            double* Tip = T + (p + 1 + wave) * kSB * P + c0;
            const f64x4 u = mma16(Tip, P, 1, Dp, 1, PX, f64x4{0.0, 0.0, 0.0, 0.0}, lane);
#pragma unroll
            for (int v = 0; v < 4; ++v) Tip[(4 * v + l4) * P + l16] = u[v];
        }
        __syncthreads();
        // X_pj = -X_pp sum_{k=j}^{p-1} L_pk X_kj for j < p, element (i, c) kept at T[column][row] of the strict upper
        // triangle, which holds nothing else; block (i, j) -= L_ip L_jp^T for p < j <= i.
        const int left = NSB - 1 - p, trailing = left * (left + 1) / 2;
        for (int task = wave; task < p + trailing; task += 4) {
            if (task < p) {
                const int j = task;
                const double* Lp = T + c0 * P;
                f64x4 w = mma16(Lp + j * kSB, P, 1, D + j * kSB * PX, PX, 1, f64x4{0.0, 0.0, 0.0, 0.0}, lane);
                for (int k = j + 1; k < p; ++k) w = mma16(Lp + k * kSB, P, 1, T + j * kSB * P + k * kSB, 1, P, w, lane);
                // W's accumulator layout (row 4 v + l / 16, column l % 16) is the B operand layout of k = 4 v + l / 16
                f64x4 u{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    u = __builtin_amdgcn_mfma_f64_16x16x4f64(Dp[l16 * PX + 4 * v + l4], w[v], u, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) T[(j * kSB + l16) * P + c0 + 4 * v + l4] = -u[v];
            } else {
                int bi, bj;
                lower_pair(task - p, bi, bj);
                const int ri = (p + 1 + bi) * kSB, rj = (p + 1 + bj) * kSB;
                const f64x4 u = mma16(T + ri * P + c0, P, 1, T + rj * P + c0, 1, P, f64x4{0.0, 0.0, 0.0, 0.0}, lane);
#pragma unroll
                for (int v = 0; v < 4; ++v) T[(ri + 4 * v + l4) * P + rj + l16] -= u[v];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kNB * kNB / 256; ++q) {         // (row i of X: lane = column)
        const int i = 4 * q + wave, c = lane, ib = i / kSB, cb = c / kSB;
        const double y = *(cb == ib ? D + i * PX + c % kSB : T + c * P + i), x = cb <= ib ? y : 0.0;
        Dinv[(int64_t)kb * kNB * kNB + i * kNB + c] = x;
        if (base + i < r && base + c < r) X[(int64_t)(base + i) * r + base + c] = x;
    }
}

// Diagonal block kb; the first one (FIRST: kb is 0) also forms sigma, kept for the later ones.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_chol_diag(double* __restrict__ S, int r, int kb, double* __restrict__ Dinv,
                                                   double* __restrict__ X, int32_t* __restrict__ info,
                                                   double* __restrict__ shift, double flag_factor, BatchStride st) {
    S += blockIdx.z * st.S;
    __shared__ double T[kNB * kPitchD];
    __shared__ double D[kNB * kPitchX];
    __shared__ double red[4];
    const int base = FIRST ? 0 : kb * kNB;
    double v[kNB * kNB / 256];                               // all loads in flight at once
#pragma unroll
    for (int q = 0; q < kNB * kNB / 256; ++q) {
        const int i = 4 * q + (threadIdx.x >> 6), c = threadIdx.x & 63;
        v[q] = (base + i < r && base + c < r) ? S[(int64_t)(base + i) * r + base + c] : (i == c ? 1.0 : 0.0);
    }
    double sigma;
    if constexpr (FIRST) {
        const double tr = trace_of(S, r, red);
        sigma = tr > 0.0 ? 0x1p-46 * tr : 0.0;
        if (threadIdx.x == 0) shift[blockIdx.z * st.shift] = sigma;
    } else {
        sigma = shift[blockIdx.z * st.shift];
    }
#pragma unroll
    for (int q = 0; q < kNB * kNB / 256; ++q) T[(4 * q + (threadIdx.x >> 6)) * kPitchD + (threadIdx.x & 63)] = v[q];
    __syncthreads();
    chol_diag_block(T, D, r, FIRST ? 0 : kb, Dinv + blockIdx.z * st.D, X + blockIdx.z * st.X, info + blockIdx.z, sigma, flag_factor);
}

__global__ __launch_bounds__(256) void k_chol_panel(double* __restrict__ S, int r, int kb, const double* __restrict__ Dinv,
                                                    BatchStride st) {
    constexpr int P = kKC + 2;
    S += blockIdx.z * st.S;
    Dinv += blockIdx.z * st.D;
    __shared__ __attribute__((aligned(16))) double At[kNB * P];
    __shared__ __attribute__((aligned(16))) double Bt[kNB * P];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wi = wave >> 1, wj = wave & 1;
    const int ib = kb + 1 + blockIdx.x;
    const double* D = Dinv + (int64_t)kb * kNB * kNB;
    BlockStage<kNB, kKC, P, double> sa, sb;
    double acc[4][4];
    zero_acc4(acc);
    f64_chunks<kKC>(0, kNB,
        [&](int k) {
            sa.fetch(S, r, ib * kNB, kb * kNB + k, r, r);
            sb.fetch(D, kNB, 0, k, kNB, kNB);
        },
        [&] {
            sa.commit(At);
            sb.commit(Bt);
        },
        [&] { mma4_kfast<kKC, P, 2>(At, Bt, acc, lane, wi, wj); });
    for_each_acc4<false>(acc, lane, wi, wj, [&](int row, int col, double x) {
        if (ib * kNB + row < r) S[(int64_t)(kb * kNB + col) * r + ib * kNB + row] = x;
    });
}

// ---------------------------------------------------------------------------------------------------------------
// X = L^-1, block (ib, kb) with kb < ib (all block rows above are complete):  X_ik = -X_ii (sum_{j=k}^{i-1} L_ij X_jk).  A
// workgroup takes 16 columns of the block (strip 0 .. 3), a wave 16 rows of them, and whole 64-deep blocks of the sum, the
// next one in registers meanwhile: with 64 columns and 16-deep chunks a workgroup was a chain of up to 60 chunks of 16 MFMAs,
// two barriers and a load each (last block row at r = 1024: 60 us, now 24).
// At, Bt: kNB * kPitchD and kNB * kPitchX doubles of LDS.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kStrips = kNB / kSB;    // strips of a block of X

__device__ __forceinline__ void trinv_strip(const double* __restrict__ S, double* __restrict__ X,
                                            const double* __restrict__ Dinv, int r, int ib, int kb, int strip, double* At,
                                            double* Bt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
    const int c0 = kb * kNB + strip * kSB;
    if (c0 >= r) return;
    BlockStage<kNB, kNB, kPitchD, double> sa;
    BlockStage<kNB, kSB, kPitchX, double> sb;
    auto product = [&](int a_pi, int a_pk) {   // element (i, k) of A at At[i * a_pi + k * a_pk]
        f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
        const double *ap = At + (wave * kSB + l16) * a_pi + l4 * a_pk, *bp = Bt + l4 * kPitchX + l16;
#pragma unroll
        for (int k = 0; k < kNB; k += 4)
            acc[(k / 4) & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k * a_pk], bp[k * kPitchX], acc[(k / 4) & 1], 0, 0, 0);
        return acc[0] + acc[1];
    };
    f64x4 sum{0.0, 0.0, 0.0, 0.0};
    sa.fetch(S, r, kb * kNB, ib * kNB, r, r);
    sb.fetch(X, r, kb * kNB, c0, r, r);
    for (int j = kb; j < ib; ++j) {
        sa.commit(At);
        sb.commit(Bt);
        __syncthreads();
        if (j + 1 < ib) {
            sa.fetch(S, r, (j + 1) * kNB, ib * kNB, r, r);
            sb.fetch(X, r, (j + 1) * kNB, c0, r, r);
        } else {
            sa.fetch(Dinv + (int64_t)ib * kNB * kNB, kNB, 0, 0, kNB, kNB);
        }
        sum += product(1, kPitchD);
        __syncthreads();
    }
    sa.commit(At);
#pragma unroll
    for (int v = 0; v < 4; ++v) Bt[(wave * kSB + 4 * v + l4) * kPitchX + l16] = sum[v];
    __syncthreads();
    const f64x4 x = product(kPitchD, 1);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = ib * kNB + wave * kSB + 4 * v + l4, c = c0 + l16;
        if (i < r && c < r) X[(int64_t)i * r + c] = -x[v];
    }
}

// The whole block by one workgroup, a quarter of the staging per MFMA, for launches that fill the chip (see kBlocksFrom).  The
// order of every sum is the strips': per 64 deep, even and odd quadruples of the contraction index apart.
// At: kTrinvA, Bt: kNB * kPitchT doubles of LDS.
constexpr int kPitchT = kNB + 2;      // LDS pitch of a 64 x 64 intermediate
constexpr int kTrinvA = kKC * F64Tile<kNB>::PITCH_KS;   // a chunk of L, then one of X_ii
static_assert(kTrinvA >= kNB * kPitchKF, "either fits");

__device__ __forceinline__ void trinv_block(const double* __restrict__ S, double* __restrict__ X,
                                            const double* __restrict__ Dinv, int r, int ib, int kb, double* At, double* Bt) {
    constexpr int PITCH = F64Tile<kNB>::PITCH_KS;
    static_assert(kNB * kPitchT >= kKC * PITCH, "the intermediate reuses the X chunk's buffer");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wi = wave >> 1, wj = wave & 1;
    f64x4 sum[2][2], acc[2][2][2];
    zero_acc(sum);
    zero_acc(acc[0]);
    zero_acc(acc[1]);
    auto product = [&](int a_pi, int a_pk, const double* B, int pitch) {   // element (i, k) of A at At[i * a_pi + k * a_pk]
#pragma unroll
        for (int k0 = 0; k0 < kKC; k0 += 4)
            mma_chunk<4>(At + k0 * a_pk, a_pi, a_pk, B + k0 * pitch, 1, pitch, acc[(k0 / 4) & 1], lane, wi, wj);
    };
    BlockStage<kKC, kNB, PITCH, double> sa, sb;
    BlockStage<kNB, kKC, kPitchKF, double> sd;
    const double* D = Dinv + (int64_t)ib * kNB * kNB;
    const int k_end = ib * kNB;
    sa.fetch(S, r, kb * kNB, ib * kNB, r, r);
    sb.fetch(X, r, kb * kNB, kb * kNB, r, r);
    for (int kc = kb * kNB; kc < k_end; kc += kKC) {
        sa.commit(At);
        sb.commit(Bt);
        __syncthreads();
        if (kc + kKC < k_end) {
            sa.fetch(S, r, kc + kKC, ib * kNB, r, r);
            sb.fetch(X, r, kc + kKC, kb * kNB, r, r);
        } else {
            sd.fetch(D, kNB, 0, 0, kNB, kNB);     // first chunk of the second product
        }
        product(1, PITCH, Bt, PITCH);
        if ((kc + kKC) % kNB == 0) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) sum[a][b] += acc[0][a][b] + acc[1][a][b];
            zero_acc(acc[0]);
            zero_acc(acc[1]);
        }
        __syncthreads();
    }
    double* Tm = Bt;
    for_each_acc(sum, lane, wi, wj, [&](int row, int col, double x) { Tm[row * kPitchT + col] = x; });
    for (int kc = 0; kc < kNB; kc += kKC) {
        sd.commit(At);
        __syncthreads();       // also publishes Tm on the first pass
        if (kc + kKC < kNB) sd.fetch(D, kNB, 0, kc + kKC, kNB, kNB);
        product(kPitchKF, 1, Tm + kc * kPitchT, kPitchT);
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) sum[a][b] = acc[0][a][b] + acc[1][a][b];
    for_each_acc(sum, lane, wi, wj, [&](int row, int col, double x) {
        const int gi = ib * kNB + row, gj = kb * kNB + col;
        if (gi < r && gj < r) X[(int64_t)gi * r + gj] = -x;
    });
}

template <bool BLOCKS>
__global__ __launch_bounds__(256) void k_trinv_row(const double* __restrict__ S, double* __restrict__ X,
                                                   const double* __restrict__ Dinv, int r, int ib, BatchStride st) {
    __shared__ double buf[BLOCKS ? kTrinvA + kNB * kPitchT : kNB * (kPitchD + kPitchX)];
    S += blockIdx.z * st.S;
    X += blockIdx.z * st.X;
    Dinv += blockIdx.z * st.D;
    if constexpr (BLOCKS) trinv_block(S, X, Dinv, r, ib, blockIdx.x, buf, buf + kTrinvA);
    else trinv_strip(S, X, Dinv, r, ib, blockIdx.x / kStrips, blockIdx.x % kStrips, buf, buf + kNB * kPitchD);
}

// Workgroups 0 .. pairs-1: the trailing blocks of step kb.  kUpdateFused: block (kb+1, kb+1) goes on to be factored, and
// workgroups the kStrips * kb after them take block row kb of X (L's row kb and X_kk are final, X's rows above too): in one launch
// the three fill the chip together, and a block column costs two launches where it takes four.  But every workgroup then holds
// the diagonal block's registers and 42 KB of LDS, three on a CU; on its own the trailing update fits more.
// kUpdatePanel: the panel too.  A workgroup forms the two blocks of L that it needs itself, 64 x 64 x 64 products of 1.7 us that
// a launch of their own takes 5 us for; only where every workgroup has a CU, since there are three products instead of one and
// 101 KB of LDS, one workgroup on a CU.
// (us per refresh, never / up to 128 / 256 / 512 workgroups: 768 x 768, r = 256 285 / 263 / 265 / 264, 2048 x 2048, r = 512 585 / 533 / 533 /
// 533, sixteen of them 1676 / 1678 / 1675 / 1703, 4096 x 4096, r = 1024 1448 / 1334 / 1334 / 1336.)
enum : int { kUpdateAlone = 0, kUpdateFused = 1, kUpdatePanel = 2 };

template <int MODE>
__global__ __launch_bounds__(256, MODE == kUpdateFused ? 3 : 1) void k_chol_update(double* __restrict__ S, int r, int kb, int pairs,
                                                     double* __restrict__ Dinv, double* __restrict__ X,
                                                     int32_t* __restrict__ info, const double* __restrict__ shift,
                                                     double flag_factor, BatchStride st) {
    S += blockIdx.z * st.S;
    X += blockIdx.z * st.X;
    Dinv += blockIdx.z * st.D;
    constexpr int P = F64Tile<kNB>::PITCH_KS, PW = kNB + 2;   // pitch of a chunk of L, of a whole 64 x 64 block
    constexpr int UPDATE = MODE == kUpdatePanel ? 3 * kNB * PW : 2 * kKC * P, BLOCK = kNB * (kPitchD + kPitchX);
    __shared__ __attribute__((aligned(16))) double buf[MODE != kUpdateAlone && BLOCK > UPDATE ? BLOCK : UPDATE];
    if constexpr (MODE != kUpdateAlone) {
        const int strip = (int)blockIdx.x - pairs;
        if (strip >= 0) {
            trinv_strip(S, X, Dinv, r, kb, strip / kStrips, strip % kStrips, buf, buf + kNB * kPitchD);
            return;
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wi = wave >> 1, wj = wave & 1;
    int pi, pj;
    lower_pair(blockIdx.x, pi, pj);
    const int ib = kb + 1 + pi, jb = kb + 1 + pj;
    double acc[4][4];
    zero_acc4(acc);
    if constexpr (MODE == kUpdatePanel) {
        BlockStage<kNB, kNB, PW, double> si, sj, sd;
        double *Li = buf, *Lj = ib == jb ? Li : buf + kNB * PW, *D = buf + 2 * kNB * PW;
        si.fetch(S, r, ib * kNB, kb * kNB, r, r);
        sd.fetch(Dinv + (int64_t)kb * kNB * kNB, kNB, 0, 0, kNB, kNB);
        if (ib != jb) sj.fetch(S, r, jb * kNB, kb * kNB, r, r);
        si.commit(Li);
        sd.commit(D);
        if (ib != jb) sj.commit(Lj);
        __syncthreads();
        auto panel = [&](double* L) {   // L <- (L X_kk^T)^T
            double x[4][4];
            zero_acc4(x);
            mma4_kfast<kNB, PW, 2>(L, D, x, lane, wi, wj);
            __syncthreads();
            for_each_acc4<false>(x, lane, wi, wj, [&](int row, int col, double v) { L[col * PW + row] = v; });
        };
        panel(Li);
        if (ib != jb) panel(Lj);
        __syncthreads();
        if (ib == jb)   // kept for X
            for (int e = threadIdx.x; e < kNB * kNB; e += 256) {
                const int k = e / kNB, row = e % kNB;
                if (ib * kNB + row < r) S[(int64_t)(kb * kNB + k) * r + ib * kNB + row] = Li[k * PW + row];
            }
        mma4_kslow<kNB, PW, 2>(Li, Lj, acc, lane, wi, wj);
        __syncthreads();
    } else {
        double *At = buf, *Bt = ib == jb ? At : buf + kKC * P;
        BlockStage<kKC, kNB, P, double> sa, sb;
        f64_chunks<kKC>(0, kNB,
            [&](int k) {
                sa.fetch(S, r, kb * kNB + k, ib * kNB, r, r);
                if (ib != jb) sb.fetch(S, r, kb * kNB + k, jb * kNB, r, r);
            },
            [&] {
                sa.commit(At);
                if (ib != jb) sb.commit(Bt);
            },
            [&] { mma4_kslow<kKC, P, 2>(At, Bt, acc, lane, wi, wj); });
    }
    if (MODE == kUpdateAlone || blockIdx.x != 0) {
        for_each_acc4<true>(acc, lane, wi, wj, [&](int row, int col, double x) {
            const int gi = ib * kNB + row, gj = jb * kNB + col;
            if (gi < r && gj < r) S[(int64_t)gi * r + gj] -= x;
        });
        return;
    }
    if constexpr (MODE != kUpdateAlone) {
        for_each_acc4<true>(acc, lane, wi, wj, [&](int row, int col, double x) {
            const int gi = ib * kNB + row, gj = ib * kNB + col;
            buf[row * kPitchD + col] = (gi < r && gj < r) ? S[(int64_t)gi * r + gj] - x : (row == col ? 1.0 : 0.0);
        });
        __syncthreads();
        chol_diag_block(buf, buf + kNB * kPitchD, r, kb + 1, Dinv, X, info + blockIdx.z, shift[blockIdx.z * st.shift], flag_factor);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Q = Y X^T (X lower triangular: column block jb needs the contraction index up to the end of that block only)
// ---------------------------------------------------------------------------------------------------------------
constexpr int kApplyStrip = 8;        // row tiles per strip of the tile numbering

template <int TB>
__global__ __launch_bounds__(256) void k_apply(const float* __restrict__ Y, const double* __restrict__ X,
                                               float* __restrict__ Q, int m, int r, int tiles_m, int tiles_r, uint32_t tiles,
                                               BatchStride st) {
    using F = F64Tile<TB>;
    const uint32_t id = xcd_tile(blockIdx.x, gridDim.x);
    if (id >= tiles) return;
    const uint32_t z = id / (uint32_t)(tiles_m * tiles_r);
    const int tile = (int)(id % (uint32_t)(tiles_m * tiles_r));
    Y += z * st.Y;
    X += z * st.X;
    Q += z * st.Q;
    constexpr int NF = 2 * F::W;
    __shared__ __attribute__((aligned(16))) double At[TB * F::PITCH_KF];
    __shared__ __attribute__((aligned(16))) double Bt[TB * F::PITCH_KF];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wi = wave >> 1, wj = wave & 1;
    // strips of eight row tiles, column tile by column tile, the longest contraction first
    const int strip = tile / (kApplyStrip * tiles_r), in_strip = tile % (kApplyStrip * tiles_r);
    const int strip_rows = min(kApplyStrip, tiles_m - strip * kApplyStrip);
    const int a0 = (strip * kApplyStrip + in_strip % strip_rows) * TB, b0 = (tiles_r - 1 - in_strip / strip_rows) * TB;
    const int kend = min(r, (b0 / kNB + 1) * kNB);           // X is zero above its diagonal blocks
    BlockStage<TB, F::KC_APPLY, F::PITCH_KF, float> sa;
    BlockStage<TB, F::KC_APPLY, F::PITCH_KF, double> sb;
    double acc[NF][NF];
    zero_acc4(acc);
    // The 16 W columns of a quadrant are dealt out to its 2 W fragments, so that a lane ends up with 2 W neighbouring ones.
    auto place = [](int c) { return c / (8 * NF) * (8 * NF) + c % NF * 8 + c % (8 * NF) / NF; };
    f64_chunks<F::KC_APPLY>(0, kend,
        [&](int k) {
            sa.fetch(Y, r, a0, k, m, r);
            sb.fetch(X, r, b0, k, r, r);
        },
        [&] {
            sa.commit(At);
            sb.commit(Bt, place);
        },
        [&] { mma4_kfast<F::KC_APPLY, F::PITCH_KF, F::W>(At, Bt, acc, lane, wi, wj); });
    const Lane4 l(lane);
    typedef float run_t __attribute__((ext_vector_type(NF)));
#pragma unroll
    for (int a = 0; a < NF; ++a) {
        const int gi = a0 + (wi * NF + a) * 8 + l.i, gj = b0 + (wj * 8 + l.j) * NF;
        run_t x;
#pragma unroll
        for (int b = 0; b < NF; ++b) x[b] = (float)acc[a][b];
        if (gi < m && gj < r) *reinterpret_cast<run_t*>(Q + (int64_t)gi * r + gj) = x;
    }
}

static size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Number of row slices of the Gram kernel: a function of the shape only (never of the batch size), so that a
// matrix gets bit-identical results alone and inside a batch.  About two workgroups per CU for a single matrix,
// at least 256 rows per slice.
static int gram_slices(int64_t m, int64_t r, int* slice_rows) {
    const int nt = (int)((r + kNB - 1) / kNB);
    const int pairs = nt * (nt + 1) / 2;
    int slices = (512 + pairs - 1) / pairs;
    const int by_rows = (int)((m + 255) / 256);
    slices = slices < by_rows ? slices : by_rows;
    slices = slices < kGramMaxSlices ? slices : kGramMaxSlices;
    *slice_rows = (int)(((m + slices - 1) / slices + kKC - 1) / kKC) * kKC;
    return (int)((m + *slice_rows - 1) / *slice_rows);
}

// Workspace of the orthonormalisation of `batch` matrices of one shape: per matrix S and X (r x r fp64), the
// inverted diagonal blocks, the result of the first round T (fp32 m x r) and the Gram slices.
struct OrthLayout {
    size_t S, X, Dinv, T, part, shift, total;
    BatchStride st;   // element strides between consecutive matrices; st.Y = st.Q = stride of T
};
static OrthLayout orth_layout(int64_t m, int64_t r, int64_t batch) {
    const int64_t nt = (r + kNB - 1) / kNB;
    int slice_rows;
    const int slices = gram_slices(m, r, &slice_rows);
    const size_t bS = align256((size_t)r * r * 8), bD = align256((size_t)nt * kNB * kNB * 8),
                 bT = align256((size_t)m * r * 4), bP = align256((size_t)slices * r * r * 8);
    OrthLayout L;
    L.S = 0;
    L.X = L.S + bS * batch;
    L.Dinv = L.X + bS * batch;
    L.T = L.Dinv + bD * batch;
    L.part = L.T + bT * batch;
    L.shift = L.part + bP * batch;
    L.total = L.shift + 256 * (size_t)batch;     // one double per matrix, 256 bytes apart
    L.st = BatchStride{(int64_t)(bT / 4), (int64_t)(bT / 4), (int64_t)(bS / 8), (int64_t)(bS / 8), (int64_t)(bD / 8),
                       (int64_t)(bP / 8), 256 / 8};
    return L;
}

// Workspace of the refresh of `batch` matrices of one shape: R and Z of the matrix in flight (shared: the
// per-matrix launches are ordered on the stream), per matrix Y (which also receives Q), then the orthonormalisation's
// and the cosine check's.
// The two GEMMs that precede the orthonormalisation (R = P^T G, Y = G Z^T) run over groups of up to kRefreshGroup
// matrices per launch, so R and Z are held for that many matrices; Y, Q and the Cholesky QR for the whole batch.
constexpr int kRefreshGroup = 16;
static_assert(kRefreshGroup <= kProjBatchMax && kRefreshGroup <= kLinBatchMax && kRefreshGroup <= kCosBatchMax, "group size");
struct RefreshLayout {
    size_t R, Z, Y, orth, cos, wts, total;
    size_t y_bytes;   // per matrix
    size_t r_bytes, z_bytes;
    int group;        // matrices per GEMM launch
};
// n: elements per row of R and Z as stored, i.e. the row pitch of the gradients.
static RefreshLayout refresh_layout(int64_t m, int64_t n, int64_t r, int64_t batch) {
    RefreshLayout L;
    L.group = (int)(batch < kRefreshGroup ? batch : kRefreshGroup);
    L.y_bytes = align256((size_t)m * r * 4);
    const size_t slice = ((size_t)r * n + 127) / 128 * 128;   // elements per matrix of R and of Z: the same count, so
    L.r_bytes = slice * 4;                                     // that one conversion launch maps R onto Z slice by slice
    L.z_bytes = slice * 2;
    L.R = 0;
    L.Z = L.R + L.r_bytes * L.group;
    L.Y = L.Z + L.z_bytes * L.group;
    L.orth = L.Y + 2 * L.y_bytes * batch;        // Y and Q of every matrix
    L.cos = L.orth + orth_layout(m, r, batch).total;
    L.wts = L.cos + align256(cossim_batch_workspace_bytes(m, r, L.group));
    L.total = L.wts + align256((size_t)L.group * r * 4);   // the columns' captured energies, one group at a time
    return L;
}

static int check_mr(int64_t m, int64_t r) {
    if (m <= 0 || r <= 0 || (r & 7) || r > m || m >= (int64_t(1) << 31) / r) return QG_ERR_SHAPE;
    return QG_OK;
}

// Y = G Z^T: G m x n and Z r x n, both bf16 with the contraction index n as their fast index; Y fp32 m x r.
// ldg, ldz: row pitches of G and Z in elements.
static int launch_range(const uint16_t* G, const uint16_t* Z, float* Y, int64_t m, int64_t n, int64_t ldg, int64_t ldz,
                        int64_t r, hipStream_t st) {
    const LinOperand A = {G, nullptr, ldg, 0}, B = {Z, nullptr, ldz, 0};
    return launch_tile_gemm<kBf16KFast, kBf16KFast, float>(A, B, nullptr, Y, m, r, n, st);
}

// k_gram and k_apply number the 64 x 64 tiles of a whole batch in one grid dimension, whose threads a launch counts in 32 bits.
constexpr int64_t kMaxTiles = (int64_t(1) << 32) / 256 - 8;   // (a multiple of 8, as the grid is)
static int64_t cholqr_tiles(int64_t m, int64_t r) {           // the larger of the two, per matrix
    const int64_t nt = (r + kNB - 1) / kNB;
    int slice_rows;
    const int64_t gram = nt * (nt + 1) / 2 * gram_slices(m, r, &slice_rows), apply = (m + kNB - 1) / kNB * nt;
    return gram > apply ? gram : apply;
}

// One round on `batch` matrices (matrix b at Y + b * sYin, result at Q + b * sQout): Q = Y L^-T with L the Cholesky
// factor of Y^T Y.
static void launch_cholqr(const float* Y, int64_t sYin, float* Q, int64_t sQout, int64_t m, int64_t r, int batch,
                          int32_t* info, double flag_factor, char* ws, const OrthLayout& L, hipStream_t stream) {
    double* S = reinterpret_cast<double*>(ws + L.S);
    double* X = reinterpret_cast<double*>(ws + L.X);
    double* Dinv = reinterpret_cast<double*>(ws + L.Dinv);
    double* part = reinterpret_cast<double*>(ws + L.part);
    double* shift = reinterpret_cast<double*>(ws + L.shift);
    BatchStride st = L.st;
    st.Y = sYin;
    st.Q = sQout;
    const int nt = (int)((r + kNB - 1) / kNB);
    const int pairs = nt * (nt + 1) / 2;
    int slice_rows;
    const int slices = gram_slices(m, r, &slice_rows);
    const dim3 blk(256);
    const unsigned B = (unsigned)batch;
    auto blocks = [](int64_t n, int size) { return (unsigned)((n + size - 1) / size); };
    auto gram = [&](auto kernel, int tb) {
        const unsigned n = blocks(r, tb), np = n * (n + 1) / 2, tiles = np * slices * B;
        hipLaunchKernelGGL(kernel, dim3((tiles + 7) / 8 * 8), blk, 0, stream, Y, part, (int)m, (int)r, slice_rows, np, (unsigned)slices, tiles, st);
    };
    auto apply = [&](auto kernel, int tb) {
        const unsigned tm = blocks(m, tb), tr = blocks(r, tb), tiles = tm * tr * B;
        hipLaunchKernelGGL(kernel, dim3((tiles + 7) / 8 * 8), blk, 0, stream, Y, X, Q, (int)m, (int)r, (int)tm, (int)tr, tiles, st);
    };
    // 32 x 32 blocks while 64 x 64 ones are about a workgroup per CU or fewer (us per refresh, always 64 / this line / up to
    // 1000 / 9000 workgroups: 768 x 768, r = 256 318 / 284 / 285 / 284, 2048 x 2048, r = 512 626 / 595 / 597 / 596, four of them
    // 802 / 803 / 803 / 820, sixteen 1724 / 1723 / 1723 / 1893, 3000 x 700, r = 128, eight of them 351 / 339 / 341 / 341)
    constexpr int64_t kFewBlocks = 300;
    const int64_t gram_blocks = (int64_t)pairs * slices * batch, apply_blocks = (int64_t)blocks(m, kNB) * nt * batch;
    if (gram_blocks < kFewBlocks) gram(k_gram<32>, 32);
    else gram(k_gram<kNB>, kNB);
    hipLaunchKernelGGL(k_gram_reduce, dim3((unsigned)((r * r + 255) / 256), 1, B), blk, 0, stream, part, S, (int)r, slices, st);
    // One launch per block column up to 1024 block rows of 64 (ms per refresh, fused / separate: 4096 x 4096, r = 1024, one 1.33 /
    // 1.90, 32 of them 16.6 / 17.2, 48 24.6 / 25.0, 64 32.2 / 32.7; 2048 x 2048, r = 512: 32 3.02 / 3.20, 128 11.01 / 11.04; 1024 x
    // 1024, r = 256, 256 matrices 4.49 / 4.48).  The arithmetic is the same, and with it every bit.
    const bool fused = batch * nt <= 1024;
    // Strips while whole blocks are fewer than the CUs or so (us, 16 matrices, 192 blocks strips 41 / blocks 48, 240 63 / 60; 40
    // matrices: 120 13 / 16, 200 24.0 / 23.9, 400 77 / 56, 600 138 / 100; 128 matrices: 128 9 / 11, 256 23 / 15, 1920 388 / 238)
    constexpr int kBlocksFrom = 200;
    auto launch_trinv_row = [&](int ib) {
        if ((int64_t)ib * batch >= kBlocksFrom)
            hipLaunchKernelGGL(k_trinv_row<true>, dim3(ib, 1, B), blk, 0, stream, S, X, Dinv, (int)r, ib, st);
        else
            hipLaunchKernelGGL(k_trinv_row<false>, dim3(kStrips * ib, 1, B), blk, 0, stream, S, X, Dinv, (int)r, ib, st);
    };
    hipLaunchKernelGGL(k_chol_diag<true>, dim3(1, 1, B), blk, 0, stream, S, (int)r, 0, Dinv, X, info, shift, flag_factor, st);
    for (int kb = 0; kb + 1 < nt; ++kb) {
        const int below = nt - kb - 1, left = below * (below + 1) / 2;
        const bool panel = fused && (int64_t)(left + kStrips * kb) * batch <= 256;
        if (!panel) hipLaunchKernelGGL(k_chol_panel, dim3(below, 1, B), blk, 0, stream, S, (int)r, kb, Dinv, st);
        if (fused) {
            hipLaunchKernelGGL(panel ? k_chol_update<kUpdatePanel> : k_chol_update<kUpdateFused>, dim3(left + kStrips * kb, 1, B), blk, 0,
                               stream, S, (int)r, kb, left, Dinv, X, info, shift, flag_factor, st);
        } else {
            hipLaunchKernelGGL(k_chol_update<kUpdateAlone>, dim3(left, 1, B), blk, 0, stream, S, (int)r, kb, left, Dinv, X, info, shift,
                               flag_factor, st);
            hipLaunchKernelGGL(k_chol_diag<false>, dim3(1, 1, B), blk, 0, stream, S, (int)r, kb + 1, Dinv, X, info, shift,
                               flag_factor, st);
        }
    }
    for (int ib = fused ? nt - 1 : 1; ib < nt; ++ib)   // (none if nt is 1)
        if (ib > 0) launch_trinv_row(ib);
    if (apply_blocks < kFewBlocks) apply(k_apply<32>, 32);
    else apply(k_apply<kNB>, kNB);
}

// Cholesky QR twice: Y -> T -> Q.  info: `batch` consecutive device ints.
static int launch_orth(const float* Y, int64_t sY, float* Q, int64_t sQ, int64_t m, int64_t r, int batch, int32_t* info,
                       bool reset_info, char* ws, hipStream_t stream) {
    const OrthLayout L = orth_layout(m, r, batch);
    float* T = reinterpret_cast<float*>(ws + L.T);
    if (reset_info)
        hipLaunchKernelGGL(k_set_i32, dim3((batch + 255) / 256), dim3(256), 0, stream, info, 0, batch);
    launch_cholqr(Y, sY, T, L.st.Y, m, r, batch, info, 0.0, ws, L, stream);
    launch_cholqr(T, L.st.Y, Q, sQ, m, r, batch, info, 16.0, ws, L, stream);
    return check_launch();
}

static int launch_to_bf16(const float* R, uint16_t* Z, int64_t count, hipStream_t st) {
    const int64_t quads = count / 4, blocks = (quads + 255) / 256;
    hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, R, Z, quads);
    return check_launch();
}

}  // namespace qg

using namespace qg;

extern "C" int qg_range_apply(const uint16_t* G_bf16, const uint16_t* Z_bf16, int64_t m, int64_t n, int64_t r, float* Y,
                              void* stream) {
    if (!G_bf16 || !Z_bf16 || !Y) return QG_ERR_NULL;
    if (int e = check_mr(m, r)) return e;
    if (n <= 0 || m * n >= (int64_t(1) << 32) || r * n >= (int64_t(1) << 32)) return QG_ERR_SHAPE;
    if (!aligned16(G_bf16) || !aligned16(Z_bf16) || !aligned16(Y)) return QG_ERR_ALIGN;
    return launch_range(G_bf16, Z_bf16, Y, m, n, n, n, r, (hipStream_t)stream);
}

extern "C" size_t qg_orthonormalize_workspace_bytes(int64_t m, int64_t r) {
    if (check_mr(m, r) != QG_OK) return 0;
    return orth_layout(m, r, 1).total;
}

extern "C" int qg_orthonormalize(const float* Y, int64_t m, int64_t r, float* Q, int32_t* info, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    if (!Y || !Q || !info) return QG_ERR_NULL;
    if (int e = check_mr(m, r)) return e;
    if (!aligned16(Y) || !aligned16(Q) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(info) & 3)) return QG_ERR_ALIGN;
    if (Y == Q) return QG_ERR_SHAPE;
    if (!workspace || workspace_bytes < orth_layout(m, r, 1).total) return QG_ERR_WORKSPACE;
    return launch_orth(Y, 0, Q, 0, m, r, 1, info, true, static_cast<char*>(workspace), (hipStream_t)stream);
}

static int check_ld(int64_t m, int64_t n, int64_t r, int64_t ld) {
    if (n <= 0 || ld < n || (ld != n && (ld & 15))) return QG_ERR_SHAPE;
    if (m * ld >= (int64_t(1) << 32) || r * ld >= (int64_t(1) << 32)) return QG_ERR_SHAPE;
    return QG_OK;
}

extern "C" size_t qg_refresh_workspace_bytes(int count, int64_t m, int64_t n, int64_t r) {
    if (count < 1 || check_mr(m, r) != QG_OK || check_ld(m, n, r, n) != QG_OK) return 0;
    return refresh_layout(m, n, r, count).total;
}

extern "C" int qg_subspace_refresh_many_ld(int count, const qg_refresh_desc* descs, int64_t m, int64_t n, int64_t ld,
                                           int64_t r, int group, int passes, float* cos_out, int32_t* info,
                                           void* workspace, size_t workspace_bytes, void* stream) {
    if (!descs || !cos_out || !info) return QG_ERR_NULL;
    if (count < 1 || passes < 1 || passes > 64) return QG_ERR_SHAPE;
    if (int e = check_mr(m, r)) return e;
    if (ld == 0) ld = n;
    if (int e = check_ld(m, n, r, ld)) return e;
    if (group != kGroup) return QG_ERR_GROUP;
    if (!aligned16(workspace) || (reinterpret_cast<uintptr_t>(cos_out) & 3) || (reinterpret_cast<uintptr_t>(info) & 3))
        return QG_ERR_ALIGN;
    for (int i = 0; i < count; ++i) {
        const qg_refresh_desc& d = descs[i];
        if (!d.Pq || !d.Ps || !d.G || !d.Pq_new || !d.Ps_new) return QG_ERR_NULL;
        if (!aligned16(d.Pq) || !aligned16(d.Ps) || !aligned16(d.G) || !aligned16(d.Pq_new) || !aligned16(d.Ps_new))
            return QG_ERR_ALIGN;
        if (d.Pq == d.Pq_new || d.Ps == d.Ps_new) return QG_ERR_SHAPE;   // the cosine check needs the old P intact
    }
    if (!workspace) return QG_ERR_WORKSPACE;
    // as many matrices per batch as the workspace holds; R and Z are stored with the gradients' row pitch
    int batch = count < 32768 ? count : 32768;   // the batch index is a grid dimension
    while (batch > 1 && (refresh_layout(m, ld, r, batch).total > workspace_bytes || cholqr_tiles(m, r) * batch > kMaxTiles))
        batch = (batch + 1) / 2;
    const RefreshLayout L = refresh_layout(m, ld, r, batch);
    if (L.total > workspace_bytes) return QG_ERR_WORKSPACE;
    char* ws = static_cast<char*>(workspace);
    float* R = reinterpret_cast<float*>(ws + L.R);
    uint16_t* Z = reinterpret_cast<uint16_t*>(ws + L.Z);
    float* Y = reinterpret_cast<float*>(ws + L.Y);
    float* Q = reinterpret_cast<float*>(ws + L.Y + L.y_bytes * batch);
    float* wts = reinterpret_cast<float*>(ws + L.wts);
    const int64_t sY = (int64_t)(L.y_bytes / 4);
    hipStream_t st = (hipStream_t)stream;
    const int64_t sR = (int64_t)(L.r_bytes / 4);
    // R_b = dequant(P_b)^T G_b for the `ng` matrices from descriptor `d0` on, into the R slices
    auto project_group = [&](const qg_refresh_desc* d0, int ng, bool new_p) -> int {
        if (ng == 1) {   // one matrix: the single-matrix launch (smaller tiles, lower latency)
            return launch_project(new_p ? d0->Pq_new : d0->Pq, new_p ? d0->Ps_new : d0->Ps, d0->G, R, m, n, ld, r, st);
        }
        ProjBatch pb;
        for (int b = 0; b < kRefreshGroup; ++b) {   // unused slots: valid pointers, never dereferenced
            const qg_refresh_desc& d = d0[b < ng ? b : 0];
            pb.Pq[b] = new_p ? d.Pq_new : d.Pq;
            pb.Ps[b] = new_p ? d.Ps_new : d.Ps;
            pb.G[b] = d.G;
        }
        return launch_project_batch(pb, ng, R, sR, m, n, ld, r, st);
    };
    for (int first = 0; first < count; first += batch) {
        const int nb = count - first < batch ? count - first : batch;
        for (int pass = 0; pass < passes; ++pass) {
            for (int g0 = 0; g0 < nb; g0 += L.group) {
                const int ng = nb - g0 < L.group ? nb - g0 : L.group;
                const qg_refresh_desc* d0 = descs + first + g0;
                if (int e = project_group(d0, ng, pass > 0)) return e;
                // the slices of R and of Z hold the same number of elements
                if (int e = launch_to_bf16(R, Z, sR * (ng - 1) + r * ld, st)) return e;
                if (ng == 1) {
                    if (int e = launch_range(d0->G, Z, Y + g0 * sY, m, n, ld, ld, r, st)) return e;
                    continue;
                }
                LinBatch lb;
                for (int b = 0; b < kRefreshGroup; ++b) lb.a[b] = d0[b < ng ? b : 0].G;
                lb.strideB_bytes = (int64_t)L.z_bytes;
                lb.strideC = sY;
                const LinOperand A = {d0->G, nullptr, ld, 0}, B = {Z, nullptr, ld, 0};
                if (int e = launch_tile_gemm<kBf16KFast, kBf16KFast, float>(A, B, nullptr, Y + g0 * sY, m, r, n, st, &lb, ng))
                    return e;
            }
            if (int e = launch_orth(Y, sY, Q, sY, m, r, nb, info + first, pass == 0, ws + L.orth, st)) return e;
            for (int b = 0; b < nb; ++b) {
                const qg_refresh_desc& d = descs[first + b];
                if (int e = qg_quant_int4(Q + b * sY, m, r, group, d.Pq_new, d.Ps_new, stream)) return e;
            }
        }
        // the convergence check: column cosines of the old and the new projection, each weighted with the energy of
        // the gradient that the new column captures (squared row norms of R_new = dequant(P_new)^T G)
        for (int g0 = 0; g0 < nb; g0 += L.group) {
            const int ng = nb - g0 < L.group ? nb - g0 : L.group;
            const qg_refresh_desc* d0 = descs + first + g0;
            if (int e = project_group(d0, ng, true)) return e;
            hipLaunchKernelGGL(k_row_energy, dim3((unsigned)r, (unsigned)ng), dim3(256), 0, st, (const float*)R, sR, (int)n,
                               (int)ld, (int)r, wts);
            if (int e = check_launch()) return e;
            CosBatch cb;
            for (int b = 0; b < kCosBatchMax; ++b) {   // unused slots repeat the first pair
                const qg_refresh_desc& d = d0[b < ng ? b : 0];
                cb.PqA[b] = d.Pq; cb.PsA[b] = d.Ps; cb.PqB[b] = d.Pq_new; cb.PsB[b] = d.Ps_new;
            }
            if (int e = launch_cossim_batch(cb, ng, m, r, cos_out + first + g0, reinterpret_cast<float*>(ws + L.cos), st,
                                            wts, r))
                return e;
        }
    }
    return QG_OK;
}

extern "C" int qg_subspace_refresh_many(int count, const qg_refresh_desc* descs, int64_t m, int64_t n, int64_t r, int group,
                                        int passes, float* cos_out, int32_t* info, void* workspace,
                                        size_t workspace_bytes, void* stream) {
    return qg_subspace_refresh_many_ld(count, descs, m, n, n, r, group, passes, cos_out, info, workspace, workspace_bytes,
                                       stream);
}

extern "C" int qg_subspace_refresh(const uint8_t* Pq, const float* Ps, const uint16_t* G_bf16, int64_t m, int64_t n,
                                   int64_t r, int group, int passes, uint8_t* Pq_new, float* Ps_new, float* cos_out,
                                   int32_t* info, void* workspace, size_t workspace_bytes, void* stream) {
    const qg_refresh_desc d = {Pq, Ps, G_bf16, Pq_new, Ps_new};
    return qg_subspace_refresh_many(1, &d, m, n, r, group, passes, cos_out, info, workspace, workspace_bytes, stream);
}
