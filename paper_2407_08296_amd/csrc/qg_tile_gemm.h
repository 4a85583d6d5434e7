// bf16 MFMA GEMM on row-major operands in any of the four orientations, with an INT8 operand dequantized while
// its tile is staged: the kernel of the INT8 linear layer (Appendix A) and of the refresh's Y = G Z^T (Sec. 3.2).
//
// The contraction index of an operand is either its fast (contiguous) index - the operand is then staged as an
// [x][k] tile and read with 16-byte LDS reads - or its slow index - staged as a [k][x] tile and read with the
// transposing LDS reads of the optimizer step's kernels.  Rows may start at any element offset (n = 5461 in the
// LLaMA-1B shapes): chunks are fetched with under-aligned wide loads; past the edge of a matrix the last row or chunk is
// fetched again, or the last whole chunk is shifted, and element by element goes only what straddles the end of the
// contraction, or an operand of less than a chunk.
#pragma once
#include "qg_common.h"
#include "qg_gemm_kernels.h"

#include <type_traits>

namespace qg {

// (the Z layouts: INT8 with a zero point per block, dequantized as (code - zero) * scale)
enum : int { kBf16KFast = 0, kBf16KSlow = 1, kInt8KFast = 2, kInt8KSlow = 3, kInt8ZKFast = 4, kInt8ZKSlow = 5 };

constexpr int kLinTM = 128;                // output tile: 128 (A's index) x TN (B's index, 256 or 128), 4 waves of 64 x TN/2;
                                           // BK (32 or 64) = contraction depth per step
constexpr int kLinStrip = 8;               // row tiles per strip of the tile numbering

// 16 consecutive INT8 codes starting at `src`, of which the first `valid` lie inside the matrix.
__device__ __forceinline__ u32x4 load16_i8_guarded(const int8_t* src, int valid) {
    if (valid >= 16) return *reinterpret_cast<const u32x4_align1*>(src);
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (j < valid) w[j >> 2] |= (uint32_t)(uint8_t)src[j] << (8 * (j & 3));
    const u32x4 o = {w[0], w[1], w[2], w[3]};
    return o;
}

// bf16(fl32(code * s)) of the 8 codes in two words; ZP: bf16(fl32((code - z) * s)), the difference being exact
template <bool ZP = false>
__device__ __forceinline__ u32x4 dequant8_i8_bf16(uint32_t c0, uint32_t c1, float s, float z = 0.f) {
    float e[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = (float)(int)(int8_t)(c0 >> (8 * j)), b = (float)(int)(int8_t)(c1 >> (8 * j));
        e[j] = ZP ? (a - z) * s : a * s;
        e[4 + j] = ZP ? (b - z) * s : b * s;
    }
    const u32x4 o = {pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]), pack_bf16x2(e[4], e[5]), pack_bf16x2(e[6], e[7])};
    return o;
}

// One GEMM operand: a row-major matrix (bf16, or INT8 codes with one fp32 scale per block of 256 elements of a
// row) of which a workgroup needs XT "x" indices starting at x0 (X of them exist) against the contraction index k
// (K of them).  LAYOUT says which of the two is the column (fast) index of the matrix in memory.
struct LinOperand {
    const void* base;
    const float* scales;   // INT8 only: [rows][sgroups]
    int64_t ld;            // row length in elements
    int sgroups;
    const float* zeros = nullptr;   // INT8 with zero points only: [rows][sgroups]
};

// Several GEMMs of one shape in one launch (gridDim.y of them): GEMM z takes its A operand from a[z], its B operand
// strideB_bytes * z past B's base and writes C + strideC * z.  One GEMM: a[0] = A's base, strides 0.
constexpr int kLinBatchMax = 16;
struct LinBatch {
    const void* a[kLinBatchMax];
    int64_t strideB_bytes;
    int64_t strideC;
    int64_t ldc = 0;   // row pitch of C in elements (0: N, dense rows)
};

// What a fetch may take for granted: the chunk lies inside the matrix and is 16-byte aligned; the step lies inside the
// contraction and no chunk straddles the end of the x indices (those past it read the last row or chunk again, for results
// that are never stored); the same, but the chunk that straddles the end is the last whole one shifted; nothing.
enum : int { kFetchAligned = 0, kFetchClamped = 1, kFetchShifted = 2, kFetchGuarded = 3 };

// Staging of one operand tile: global -> registers (fetch) -> LDS (commit; INT8 is dequantized here).
template <int LAYOUT, int XT, int BK, int NT = 256, int PADK = kPadK>
struct LinStage {
    static constexpr bool kFast = LAYOUT == kBf16KFast || LAYOUT == kInt8KFast || LAYOUT == kInt8ZKFast;
    static constexpr bool kZero = LAYOUT == kInt8ZKFast || LAYOUT == kInt8ZKSlow;
    static constexpr bool kInt8 = LAYOUT == kInt8KFast || LAYOUT == kInt8KSlow || kZero;
    static constexpr int CH = kInt8 ? 16 : 8;                   // elements per 16-byte chunk (one block scale each)
    static constexpr int CPR = (kFast ? BK : XT) / CH;          // chunks per tile row
    static constexpr int PITCH = kFast ? BK + kPadX : XT + PADK;   // LDS pitch: [x][k] or [k][x]
    static constexpr int ELEMS = (kFast ? XT : BK) * PITCH;
    static constexpr int PER = XT * BK / CH / NT;               // chunks per thread (NT threads in the workgroup)
    static_assert(XT * BK % (CH * NT) == 0, "tile must divide evenly over the threads");
    u32x4 v[PER];
    float s[kInt8 ? PER : 1];
    float z[kZero ? PER : 1];
    // (a workgroup of more than NT threads: every NT of them stage tiles of their own)
    __device__ static __forceinline__ int thread() { return threadIdx.x & (NT - 1); }

    // KI: int or int64_t.  Over a 64-bit k0 the compiler turns the addresses of a loop into running pointers; over a 32-bit
    // one it recomputes a 64-bit product per chunk and step (grad_W with 128 x 128 x 32 tiles, 2048 tokens, 2560 x 2048:
    // 36.2 against 38.6 us), which takes fewer registers.
    template <int FETCH, typename KI>
    __device__ __forceinline__ void fetch(const LinOperand& op, int x0, int X, KI k0, int K) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int idx = thread() + NT * q;
            const int tr = idx / CPR, tc = (idx % CPR) * CH;         // row and first column inside the tile
            int x = x0 + (kFast ? tr : tc);                          // ... and inside the matrix
            const int xs = min(x, X - 1);                            // for the block scale: the chunk's own block
            const int past = FETCH == kFetchShifted && !kFast ? min(max(x - (X - CH), 0), CH - 1) : 0;
            if constexpr (FETCH == kFetchClamped || FETCH == kFetchShifted) x = min(x, kFast ? X - 1 : X - CH);
            const KI k = k0 + (kFast ? tc : tr);
            const auto row = kFast ? x : k;
            const auto col = kFast ? k : x;
            int valid = CH;
            if constexpr (FETCH == kFetchGuarded) {
                valid = kFast ? (x < X ? K - (int)k : 0) : ((int)k < K ? X - x : 0);
            }
            const int64_t off = (int64_t)row * op.ld + col;
            if constexpr (kInt8) {
                const int8_t* src = static_cast<const int8_t*>(op.base) + off;
                if constexpr (FETCH == kFetchAligned) v[q] = *reinterpret_cast<const u32x4*>(src);
                else v[q] = load16_i8_guarded(src, valid);
                const auto block = (!kFast && FETCH == kFetchShifted ? xs : col) >> 8;
                s[q] = valid > 0 ? op.scales[(int64_t)row * op.sgroups + block] : 0.f;
                if constexpr (kZero) z[q] = valid > 0 ? op.zeros[(int64_t)row * op.sgroups + block] : 0.f;
            } else {
                const uint16_t* src = static_cast<const uint16_t*>(op.base) + off;
                if constexpr (FETCH == kFetchAligned) v[q] = *reinterpret_cast<const u32x4*>(src);
                else v[q] = load8_bf16_guarded(src, valid);
            }
            if constexpr (FETCH == kFetchShifted && !kFast) v[q] = shift_right_128(v[q], past * (128 / CH));
        }
    }
    __device__ __forceinline__ void commit(uint16_t* tile) const {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int idx = thread() + NT * q;
            uint16_t* dst = tile + (idx / CPR) * PITCH + (idx % CPR) * CH;
            if constexpr (kInt8) {
                *reinterpret_cast<u32x4*>(dst) = dequant8_i8_bf16<kZero>(v[q][0], v[q][1], s[q], kZero ? z[q] : 0.f);
                *reinterpret_cast<u32x4*>(dst + 8) = dequant8_i8_bf16<kZero>(v[q][2], v[q][3], s[q], kZero ? z[q] : 0.f);
            } else {
                *reinterpret_cast<u32x4*>(dst) = v[q];
            }
        }
    }
    // Whether the tile of the XT x indices from x0 on can be fetched clamped (chunks along x: whole ones, or all inside).
    __device__ static __forceinline__ bool clampable(int x0, int X) { return kFast || X % CH == 0 || x0 + XT <= X; }
    // ... shifted (at least one whole chunk along x).
    __device__ static __forceinline__ bool shiftable(int X) { return kFast || X >= CH; }
    // MFMA operand fragment of the 32 x indices starting at xb for the 16-deep sub-step kk
    __device__ static __forceinline__ bf16x8 frag(const uint16_t* tile, int xb, int kk, int lane) {
        if constexpr (kFast)
            return *reinterpret_cast<const bf16x8*>(tile + (xb + (lane & 31)) * PITCH + kk * 16 + 8 * (lane >> 5));
        else
            return read_kmajor_frag(tile + kk * 16 * PITCH + xb + kmajor_lane_offset(PITCH, lane), PITCH);
    }
};

// A wave's 32 x 32 block of C, rows from row0 and columns from col0 on: through LDS (tp: kTransposeFloats floats of the
// wave's own), so that C is written in 16-byte runs of a row.  A lane of the accumulator holds single elements of 16
// rows, and the memory pipe's address unit takes 16 cycles per wave-wide access whatever its width: as 2-byte stores a
// 256 x 256 bf16 tile spent 7 us there.  Rows of C may start at any element; EXACT: the block lies inside C.
// bj: added to the lane's column (lane % 32).
template <bool EXACT, typename OUT>
__device__ __forceinline__ void store_block(const f32x16& acc, float bj, float* tp, OUT* __restrict__ C, int64_t ldc, int row0,
                                            int col0, int M, int N, int lane) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
        tp[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kTransposePitch + (lane & 31)] = acc[v] + bj;
    constexpr int RUN = 16 / sizeof(OUT), LPR = 32 / RUN, RPI = 64 / LPR;   // elements per run, lanes per row, rows per access
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int row = RPI * i + lane / LPR, col = RUN * (lane % LPR);
        const float* src = tp + row * kTransposePitch + col;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(src);
        u32x4 o;
        if constexpr (sizeof(OUT) == 4) {
            o = __builtin_bit_cast(u32x4, lo);
        } else {
            const f32x4 hi = *reinterpret_cast<const f32x4*>(src + 4);
            o = u32x4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
        }
        OUT* dst = C + (int64_t)(row0 + row) * ldc + col0 + col;
        const int left = EXACT ? RUN : (row0 + row < M ? N - (col0 + col) : 0);
        if (left >= RUN) {
            if constexpr (sizeof(OUT) == 4) *reinterpret_cast<u32x4_align4*>(dst) = o;
            else *reinterpret_cast<u32x4_align2*>(dst) = o;
        } else {
#pragma unroll
            for (int e = 0; e < RUN - 1; ++e)
                if (e < left) {
                    if constexpr (sizeof(OUT) == 4) dst[e] = __builtin_bit_cast(float, (uint32_t)o[e & 3]);
                    else dst[e] = (OUT)(o[e >> 1] >> (16 * (e & 1)));
                }
        }
    }
}

// C[M][N] (bf16 or fp32) = sum_k A(i, k) B(k, j) (+ bias[j]); A's x index runs over the rows of C, B's over its
// columns.  Tile TM = 32 MB WM rows x TN columns, a wave computes 32 MB x TN / 2.
// Two LDS stages, one barrier per step.  DEEP: two register sets - while the MFMAs of step kt read stage kt & 1, the
// operands of step kt + 1 are written to the other stage and those of step kt + 2 are fetched, all of it between the
// MFMAs: for workgroups that have a CU to themselves.  Otherwise one set - the operands of step kt + 1 are fetched before
// the MFMAs of step kt and written to the other stage after them: fewer registers, and workgroups that share a CU cover for
// each other.
// WM: wave rows of the workgroup (2: 256 threads, several workgroups per CU; 4: 512 threads, one workgroup per CU - the
// B tile, and with it the dequantization of an INT8 B operand, is then shared by twice as many MFMAs).
// KG: groups of waves of the workgroup that take the steps in turn (group g the steps g, g + KG, ...), each with LDS stages of
// its own; their sums are added in the order of the groups.  For a workgroup that has its CU to itself: the chain of steps is KG
// times shorter, and a SIMD has a wave to issue while another waits.
// EXACT: every tile lies inside the matrices, K is a whole number of steps, rows are 16-byte aligned.  Otherwise a workgroup
// runs unchecked too, but for the last, partial step, with its x indices clamped to the operand's last row or chunk: the
// checks cost a wave three branches per chunk, and the workgroups at the edge, which took them, were the last to end (1000
// tokens, 2048 -> 2048: forward 28.5 -> 20.9 us, grad_input 29.4 -> 21.7; 1024 tokens 20.4 and 22.0).  Where the last chunk of
// an operand with k slow is not whole, the tile at its edge takes the last whole chunk and shifts it (1000 tokens, 2048 ->
// 5461: grad_input 98.6 -> 50.9, grad_W 80.1 -> 48.1; with every element of that chunk checked and loaded alone, the few
// workgroups of that edge took longer than all others together).  Checked are operands of less than a chunk.
template <int AL, int BL, int MB, int TN, int BK, int WM, int KG = 1>
struct TileGemm {
    static constexpr int TM = 32 * MB * WM, NT = 128 * WM;
    static constexpr int PADK = KG > 1 ? 16 : kPadK;
    using SA = LinStage<AL, TM, BK, NT, PADK>;
    using SB = LinStage<BL, TN, BK, NT, PADK>;
    static constexpr int STAGING = 2 * (SA::ELEMS + SB::ELEMS), TRANSPOSE = 2 * WM * kTransposeFloats * 2;
    static constexpr int SMEM = STAGING > TRANSPOSE ? STAGING : TRANSPOSE;   // uint16 elements
};

template <int AL, int BL, bool EXACT, typename OUT, int MB, int TN, int BK, int WM, bool DEEP, int KG = 1>
__device__ __forceinline__ void tile_gemm(const LinOperand& A, const LinOperand& B, const uint16_t* __restrict__ bias,
                                          OUT* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m, int tiles_n,
                                          uint32_t tile, uint16_t* smem) {
    using T = TileGemm<AL, BL, MB, TN, BK, WM, KG>;
    using SA = typename T::SA;
    using SB = typename T::SB;
    constexpr int TM = T::TM;
    static_assert(KG == 1 || DEEP, "groups: two register sets");
    const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / T::NT);
    smem += group * T::SMEM;
    auto At = [&](int stage) { return smem + stage * SA::ELEMS; };
    auto Bt = [&](int stage) { return smem + 2 * SA::ELEMS + stage * SB::ELEMS; };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x & (T::NT - 1)) >> 6), wm = wave >> 1, wn = wave & 1;
    // Tiles are numbered in strips eight row tiles tall, column tile by column tile: the tiles in flight on an XCD share
    // eight A panels and a few B panels.
    const int strip = (int)(tile / (uint32_t)(kLinStrip * tiles_n)), in_strip = (int)(tile % (uint32_t)(kLinStrip * tiles_n));
    const int strip_rows = min(kLinStrip, tiles_m - strip * kLinStrip);
    const int i0 = (strip * kLinStrip + in_strip % strip_rows) * TM, j0 = (in_strip / strip_rows) * TN;
    SA sa[DEEP ? 2 : 1];
    SB sb[DEEP ? 2 : 1];
    constexpr int NB = TN / 64;                // 32 x 32 blocks of a wave: MB x NB
    f32x16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    auto mfma_step = [&](int stage) {
        if constexpr (!DEEP) __builtin_amdgcn_s_setprio(kMfmaPrio);   // the wave in its MFMA phase goes first
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 af[MB], bf[NB];
#pragma unroll
            for (int a = 0; a < MB; ++a) af[a] = SA::frag(At(stage), wm * 32 * MB + a * 32, kk, lane);
#pragma unroll
            for (int b = 0; b < NB; ++b) bf[b] = SB::frag(Bt(stage), wn * (TN / 2) + b * 32, kk, lane);
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bf[b], acc[a][b], 0, 0, 0);
            if constexpr (!DEEP) __builtin_amdgcn_sched_barrier(0);   // fragments of one sub-step at a time
        }
        if constexpr (!DEEP) __builtin_amdgcn_s_setprio(0);
    };
    // The KT steps from k = 0 on, every chunk of them fetched under FETCH's terms.
    // (64-deep steps with two register sets have no registers left for running pointers.)
    using KI = std::conditional_t<DEEP && BK == 64, int, int64_t>;
    auto steps = [&](auto fetch_mode, int KT) {
        constexpr int FETCH = decltype(fetch_mode)::value;
        auto fetch = [&](KI k0, int set) {
            sa[set].template fetch<FETCH>(A, i0, M, k0, K);
            sb[set].template fetch<FETCH>(B, j0, N, k0, K);
        };
        auto commit = [&](int set, int stage) {
            sa[set].commit(At(stage));
            sb[set].commit(Bt(stage));
        };
        if constexpr (!DEEP) {
            KI k0 = 0;
            fetch(k0, 0);
            commit(0, 0);
            __syncthreads();   // (lds_barrier, across which nothing is scheduled: grad_input of the 7B layer 143 against 134 us)
            for (int kt = 0; kt < KT; ++kt) {
                const int cur = kt & 1;
                const bool more = kt + 1 < KT;
                k0 += BK;
                if (more) fetch(k0, 0);
                mfma_step(cur);
                if (more) commit(0, cur ^ 1);
                __syncthreads();
            }
            return;
        }
        // this group's i-th step; past the end: the last slab again, never consumed
        auto slab = [&](int i) { return (KI)min(KG * i + group, KT - 1) * BK; };
        const int n = (KT + KG - 1) / KG, all = KT % KG == 0 ? n : n - 1;   // steps of the longest group, of every group
        fetch(slab(0), 0);
        fetch(slab(1), DEEP);
        commit(0, 0);
        lds_barrier();
        int i = 0;
        for (; i + 1 < all; i += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // one scheduling region: fragment reads, the fetches of step i + u + 2 and the commit of step i + u + 1
                // between the MFMAs
                mfma_step(u);
                fetch(slab(i + u + 2), DEEP ? u : 0);
                commit(DEEP ? u ^ 1 : 0, u ^ 1);
                constexpr int READS = MB * (SA::kFast ? 1 : 2) + NB * (SB::kFast ? 1 : 2), MFMAS = MB * NB;
                __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
#pragma unroll
                for (int j = 0; j < BK / 16 * MFMAS; ++j) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, (READS + MFMAS - 1) / MFMAS, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                }
                lds_barrier();
            }
        }
#pragma unroll
        for (int u = 0; u < (KG == 1 ? 1 : 2); ++u) {   // at most one step is left, or two if only some groups have the last
            if (i + u >= n) break;
            if (KG == 1 || KG * (i + u) + group < KT) mfma_step(u);
            if (KG > 1 && u == 0 && i + 1 < n) commit(1, 1);
            lds_barrier();
        }
    };
    bool inside = true;
    if constexpr (EXACT) {
        steps(std::integral_constant<int, kFetchAligned>(), K / BK);
    } else {
        inside = i0 + TM <= M && j0 + TN <= N;
        const int whole = K / BK;
        const bool shiftable = SA::shiftable(M) && SB::shiftable(N);
        if (!shiftable) {
            steps(std::integral_constant<int, kFetchGuarded>(), (K + BK - 1) / BK);
        } else {
            if (whole > 0) {
                if (SA::clampable(i0, M) && SB::clampable(j0, N)) steps(std::integral_constant<int, kFetchClamped>(), whole);
                else steps(std::integral_constant<int, kFetchShifted>(), whole);
            }
            if (whole * BK < K) {
                const bool mine = KG == 1 || group == whole % KG;   // (wave-uniform)
                if (mine) {
                    sa[0].template fetch<kFetchGuarded>(A, i0, M, whole * BK, K);
                    sb[0].template fetch<kFetchGuarded>(B, j0, N, whole * BK, K);
                    sa[0].commit(At(0));
                    sb[0].commit(Bt(0));
                }
                lds_barrier();
                if (mine) mfma_step(0);
                lds_barrier();
            }
        }
    }
    if constexpr (KG > 1) {   // the groups' sums through LDS, group 0 adds them in order
        static_assert(MB * NB * T::NT * 16 * 4 <= T::SMEM * 2, "they fit in a group's staging buffers");
        const int t = threadIdx.x & (T::NT - 1);
        if (group != 0) {
#pragma unroll
            for (int q = 0; q < MB * NB * 4; ++q) {
                const f32x16& c = acc[q / 4 / NB][q / 4 % NB];
                reinterpret_cast<f32x4*>(smem)[q * T::NT + t] = f32x4{c[q % 4 * 4], c[q % 4 * 4 + 1], c[q % 4 * 4 + 2], c[q % 4 * 4 + 3]};
            }
        }
        __syncthreads();
        if (group != 0) return;
#pragma unroll
        for (int g = 1; g < KG; ++g)
#pragma unroll
            for (int q = 0; q < MB * NB * 4; ++q) {
                const f32x4 x = reinterpret_cast<const f32x4*>(smem + g * T::SMEM)[q * T::NT + t];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[q / 4 / NB][q / 4 % NB][q % 4 * 4 + e] += x[e];
            }
    }
    float* tp = reinterpret_cast<float*>(smem) + wave * kTransposeFloats;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int row0 = i0 + wm * 32 * MB + a * 32, col0 = j0 + wn * (TN / 2) + b * 32, col = col0 + (lane & 31);
            const float bj = (bias != nullptr && (EXACT || col < N)) ? __builtin_bit_cast(float, (uint32_t)bias[col] << 16) : 0.f;
            if (EXACT || inside) store_block<true>(acc[a][b], bj, tp, C, ldc, row0, col0, M, N, lane);
            else store_block<false>(acc[a][b], bj, tp, C, ldc, row0, col0, M, N, lane);
        }
}

template <int AL, int BL, bool EXACT, typename OUT, int MB, int TN, int BK, int WM, bool DEEP, int KG = 1>
__global__ __launch_bounds__(WM * 128 * KG, KG > 1 ? (MB == 1 ? 4 : 2) : WM == 2 ? 2 : 1) void k_tile_gemm(LinOperand A, LinOperand B,
                                                      const uint16_t* __restrict__ bias,
                                                      OUT* __restrict__ C, int M, int N, int K, int tiles_m, int tiles_n,
                                                      LinBatch batch) {
    __shared__ __attribute__((aligned(16))) uint16_t smem[KG * TileGemm<AL, BL, MB, TN, BK, WM, KG>::SMEM];
    A.base = batch.a[blockIdx.y];
    B.base = static_cast<const char*>(B.base) + batch.strideB_bytes * blockIdx.y;
    // each XCD (own L2) takes a contiguous range of tiles
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    if (tile >= (uint32_t)(tiles_m * tiles_n)) return;
    tile_gemm<AL, BL, EXACT, OUT, MB, TN, BK, WM, DEEP, KG>(A, B, bias, C + batch.strideC * blockIdx.y, batch.ldc ? batch.ldc : N, M, N, K,
                                                  tiles_m, tiles_n, tile, smem);
}

// A product as a kernel argument.
struct LinProduct {
    LinOperand A, B;
    uint16_t* C;
    int64_t ldc;
    int M, N, K, tiles_m, tiles_n;
};

// The contraction split over the KW waves of a workgroup: 32 x 32 tiles, wave w takes the 64-deep steps w, w + KW, ... of
// the whole tile, and the KW partial tiles are added through LDS in a fixed order.  For products of few tiles, where what
// counts is the length of a workgroup's serial chain (fetch, commit, fragments, MFMAs per step): it is KW times shorter than
// with the tile split over the waves, there are four times as many workgroups as with 64 x 64 tiles, and since a wave stages
// its own operands (its LDS accesses complete in order) there is no barrier before the final sum.
template <int AL, int BL, int KW>
struct KSplit {
    static constexpr int BK = 64, NT = 64 * KW;
    using SA = LinStage<AL, 32, BK, 64>;
    using SB = LinStage<BL, 32, BK, 64>;
    static constexpr int WAVE = SA::ELEMS + SB::ELEMS;   // uint16 elements of a wave's operands, then of its partial tile
    static_assert(2 * kTransposeFloats <= WAVE, "the partial tile fits where the operands were");
    static constexpr int SMEM = KW * WAVE;
};

template <int AL, int BL, bool EXACT, int KW>
__device__ __forceinline__ void ksplit_gemm(const LinOperand& A, const LinOperand& B, const uint16_t* __restrict__ bias,
                                            uint16_t* __restrict__ C, int64_t ldc, int M, int N, int K, int tiles_m, int tiles_n,
                                            uint32_t tile, uint16_t* smem) {
    using T = KSplit<AL, BL, KW>;
    using SA = typename T::SA;
    using SB = typename T::SB;
    constexpr int BK = T::BK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint16_t *At = smem + wave * T::WAVE, *Bt = At + SA::ELEMS;
    const int strip = (int)(tile / (uint32_t)(kLinStrip * tiles_n)), in_strip = (int)(tile % (uint32_t)(kLinStrip * tiles_n));
    const int strip_rows = min(kLinStrip, tiles_m - strip * kLinStrip);
    const int i0 = (strip * kLinStrip + in_strip % strip_rows) * 32, j0 = (in_strip / strip_rows) * 32;
    auto steps_below = [&](int n) { return n > wave ? (n - wave + KW - 1) / KW : 0; };   // of this wave, below step n
    SA sa[2];
    SB sb[2];
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    // between a wave's writes of its tiles and its reads, and back: its LDS instructions complete in order, so what has to
    // be kept is the order in which they are issued (the scheduler does not see the transposing reads as accesses)
    auto in_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&](int set, auto fetch_next) {
        sa[set].commit(At);
        sb[set].commit(Bt);
        in_order();
        bf16x8 af[BK / 16], bf[BK / 16];
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            af[kk] = SA::frag(At, 0, kk, lane);
            bf[kk] = SB::frag(Bt, 0, kk, lane);
        }
        in_order();
        fetch_next();
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk], bf[kk], acc, 0, 0, 0);
    };
    // this wave's steps first, first + KW, ... (`count` of them), fetched two ahead under FETCH's terms
    auto run = [&](auto fetch_mode, int first, int count) {
        constexpr int FETCH = decltype(fetch_mode)::value;
        auto fetch = [&](int i, int set) {
            if (i >= count) return;
            const int k0 = (first + KW * i) * BK;
            sa[set].template fetch<FETCH>(A, i0, M, k0, K);
            sb[set].template fetch<FETCH>(B, j0, N, k0, K);
        };
        fetch(0, 0);
        fetch(1, 1);
        for (int i = 0; i < count; i += 2) {
            compute(0, [&] { fetch(i + 2, 0); });
            if (i + 1 < count) compute(1, [&] { fetch(i + 3, 1); });
        }
    };
    using Guarded = std::integral_constant<int, kFetchGuarded>;
    const int total = (K + BK - 1) / BK, whole = K / BK;
    if constexpr (EXACT) {
        run(std::integral_constant<int, kFetchAligned>(), wave, steps_below(total));
    } else if (SA::shiftable(M) && SB::shiftable(N)) {
        const int n = steps_below(whole);
        if (SA::clampable(i0, M) && SB::clampable(j0, N)) run(std::integral_constant<int, kFetchClamped>(), wave, n);
        else run(std::integral_constant<int, kFetchShifted>(), wave, n);
        if (steps_below(total) > n) run(Guarded(), wave + KW * n, 1);   // the last, partial step
    } else {
        run(Guarded(), wave, steps_below(total));
    }
    float* tp = reinterpret_cast<float*>(At);
#pragma unroll
    for (int v = 0; v < 16; ++v) tp[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * kTransposePitch + (lane & 31)] = acc[v];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const int row = threadIdx.x / 8, col = (threadIdx.x % 8) * 4;        // four columns of a row per thread
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(smem + w * T::WAVE) +
                                                        row * kTransposePitch + col);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += x[e];
    }
    const int left = EXACT ? 4 : (i0 + row < M ? N - (j0 + col) : 0);
    if (bias != nullptr) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < left) sum[e] += __builtin_bit_cast(float, (uint32_t)bias[j0 + col + e] << 16);
    }
    const u32x2 o = {pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3])};
    uint16_t* dst = C + (int64_t)(i0 + row) * ldc + j0 + col;
    if (left >= 4) {
        *reinterpret_cast<u32x2_align2*>(dst) = o;
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < left) dst[e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
    }
}

template <int BL, bool EXACT, int KW>
__global__ __launch_bounds__(64 * KW) void k_ksplit_gemm(LinProduct p, const uint16_t* __restrict__ bias) {
    __shared__ __attribute__((aligned(16))) uint16_t smem[KSplit<kBf16KFast, BL, KW>::SMEM];
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    if (tile >= (uint32_t)(p.tiles_m * p.tiles_n)) return;
    ksplit_gemm<kBf16KFast, BL, EXACT, KW>(p.A, p.B, bias, p.C, p.ldc, p.M, p.N, p.K, p.tiles_m, p.tiles_n, tile, smem);
}

// The two products of a backward pass in one launch: they do not depend on each other, and each alone leaves most of the chip
// idle (one after the other their times add up).  The first grid0 workgroups run the first (A bf16 with k fast, B the
// weight), the others the second (both bf16 with k slow).  SPLIT: 32 x 32 tiles with the contraction split over the waves,
// otherwise 64 x 64 tiles.
template <int AL, int BL, bool SPLIT>
constexpr int kPairSmem = SPLIT ? KSplit<AL, BL, 4>::SMEM : TileGemm<AL, BL, 1, 64, 64, 2>::SMEM;
template <int AL, int BL, bool EXACT, bool SPLIT>
__device__ __forceinline__ void pair_product(const LinProduct& p, uint32_t block, uint32_t blocks, uint16_t* smem) {
    const uint32_t tile = xcd_tile(block, blocks);
    if (tile >= (uint32_t)(p.tiles_m * p.tiles_n)) return;
    if constexpr (SPLIT)
        ksplit_gemm<AL, BL, EXACT, 4>(p.A, p.B, nullptr, p.C, p.ldc, p.M, p.N, p.K, p.tiles_m, p.tiles_n, tile, smem);
    else
        tile_gemm<AL, BL, EXACT, uint16_t, 1, 64, 64, 2, true>(p.A, p.B, nullptr, p.C, p.ldc, p.M, p.N, p.K, p.tiles_m, p.tiles_n,
                                                               tile, smem);
}
template <int BL, bool EXACT, bool SPLIT0, bool SPLIT1>
__global__ __launch_bounds__(256, 2) void k_gemm_pair(LinProduct p0, LinProduct p1, uint32_t grid0) {
    constexpr int S0 = kPairSmem<kBf16KFast, BL, SPLIT0>, S1 = kPairSmem<kBf16KSlow, kBf16KSlow, SPLIT1>;
    __shared__ __attribute__((aligned(16))) uint16_t smem[S0 > S1 ? S0 : S1];
    if (blockIdx.x < grid0) pair_product<kBf16KFast, BL, EXACT, SPLIT0>(p0, blockIdx.x, grid0, smem);
    else pair_product<kBf16KSlow, kBf16KSlow, EXACT, SPLIT1>(p1, blockIdx.x - grid0, gridDim.x - grid0, smem);
}

// Both operands bf16 with the contraction index as their slow index, whole tiles and aligned rows (grad_W at the
// LLaMA shapes): the staging of the optimizer step's projection kernel for its gradient operand, applied to both -
// direct global -> LDS loads into unpadded swizzled [k][x] tiles (no staging registers, no LDS write instructions),
// two stages, the loads of step k+1 issued ahead of the MFMAs of step k, three workgroups per CU.
template <typename OUT>
__global__ __launch_bounds__(256, 3) void k_gemm_kslow_direct(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                              OUT* __restrict__ C, int M, int N, int K, int tiles_m,
                                                              int tiles_n) {
    constexpr int TN = 256, BK = 32;
    const int64_t ldc = N;   // dense operands and output only
    using AD = KMajorSwizzled<kLinTM, BK, 256>;
    using BD = KMajorSwizzled<TN, BK, 256>;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][AD::STAGE];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BD::STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    if (tile >= (uint32_t)(tiles_m * tiles_n)) return;
    const int strip = (int)(tile / (uint32_t)(kLinStrip * tiles_n)), in_strip = (int)(tile % (uint32_t)(kLinStrip * tiles_n));
    const int strip_rows = min(kLinStrip, tiles_m - strip * kLinStrip);
    const int i0 = (strip * kLinStrip + in_strip % strip_rows) * kLinTM, j0 = (in_strip / strip_rows) * TN;
    static_assert(AD::VARIANTS == 1 && BD::VARIANTS == 2, "per-lane source offsets below");
    const uint32_t a_byte = AD::lane_src_bytes(lane, M, 0);
    const uint32_t b_byte[2] = {BD::lane_src_bytes(lane, N, 0), BD::lane_src_bytes(lane, N, 1)};
    auto gload = [&](int kt, int stage) {
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(A + (int64_t)kt * BK * M + i0);
        const __amdgpu_buffer_rsrc_t rb = make_rsrc(B + (int64_t)kt * BK * N + j0);
#pragma unroll
        for (int p = 0; p < AD::PER; ++p)
            buffer_load_lds16(ra, As[stage] + AD::load_row0(wave, p) * kLinTM, a_byte, 2u * (uint32_t)(AD::load_row0(wave, p) * M));
#pragma unroll
        for (int p = 0; p < BD::PER; ++p)
            buffer_load_lds16(rb, Bs[stage] + BD::load_row0(wave, p) * TN, b_byte[p % 2], 2u * (uint32_t)(BD::load_row0(wave, p) * N));
    };
    constexpr int MB = 2, NB = 4;
    f32x16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    int a_lane[MB], b_lane[NB];
#pragma unroll
    for (int a = 0; a < MB; ++a) a_lane[a] = AD::lane_offset(lane) + ((wm * 64 + a * 32) ^ AD::lane_swizzle(lane));
#pragma unroll
    for (int b = 0; b < NB; ++b) b_lane[b] = BD::lane_offset(lane) + ((wn * 128 + b * 32) ^ BD::lane_swizzle(lane));
    auto mfma_step = [&](int stage) {
        __builtin_amdgcn_s_setprio(kMfmaPrio);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 af[MB], bf[NB];
#pragma unroll
            for (int a = 0; a < MB; ++a) af[a] = read_kmajor_frag(As[stage] + kk * 16 * kLinTM + a_lane[a], kLinTM);
#pragma unroll
            for (int b = 0; b < NB; ++b) bf[b] = read_kmajor_frag(Bs[stage] + kk * 16 * TN + b_lane[b], TN);
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bf[b], acc[a][b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    auto landed = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };   // direct loads count like any other load
    const int KT = K / BK;
    // unrolled by two: constant LDS stages; loads past the end re-read the last K slab (in bounds, never consumed)
    gload(0, 0);
    landed();
    __syncthreads();
    for (int kt = 0; kt < KT; kt += 2) {
        gload(min(kt + 1, KT - 1), 1);
        mfma_step(0);
        landed();
        __syncthreads();
        gload(min(kt + 2, KT - 1), 0);
        if (kt + 1 < KT) mfma_step(1);
        landed();
        __syncthreads();
    }
    // Straight from the accumulators: three workgroups per CU cover for each other's stores here (64 tokens, 4096 x 11008:
    // 20.8 us, as 16-byte runs through LDS 23.0; 4096 tokens 329 and 331).
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int col = j0 + wn * 128 + b * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = i0 + wm * 64 + a * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                const float x = acc[a][b][v];
                if constexpr (sizeof(OUT) == 4) C[(int64_t)row * ldc + col] = x;
                else C[(int64_t)row * ldc + col] = to_bf16(x);
            }
        }
}

// bf16 [X][64] operand tile (rows along the contraction index, 128 bytes each) filled by direct global -> LDS loads:
// one wave-wide 16-byte-per-lane load deposits 1 KB = 8 rows, lane l at row l / 8, chunk position l % 8.  Rows are
// not padded; bank spreading comes from a swizzle on the source side: position p of row x holds the row's chunk
// p ^ (x & 7), so the 8 rows that 8 consecutive lanes of a fragment read touch (same chunk) sit at 8 different
// positions.  X rows over NW waves.
template <int XT, int NW>
struct KFastDirect {
    static constexpr int BK = 64, ROW = BK;                 // elements per tile row
    static constexpr int ELEMS = XT * BK;
    static constexpr int PER = XT / 8 / NW;                 // wave-wide loads per wave
    static_assert(XT % (8 * NW) == 0, "tile rows must divide evenly over the waves");
    // byte offset, from the tile's first element (row pitch ld elements), of the chunk lane `lane` fetches in the
    // load that covers rows [8 q, 8 q + 8): the same for every q
    __device__ static __forceinline__ uint32_t lane_src_bytes(int lane, int64_t ld) {
        const int row = lane >> 3, chunk = (lane & 7) ^ row;
        return (uint32_t)(2 * (row * ld + chunk * 8));
    }
    // element offset of the fragment of lane `lane` for the 32 rows starting at xb (a multiple of 32), sub-step kk
    __device__ static __forceinline__ int frag_offset(int xb, int kk, int lane) {
        const int row = xb + (lane & 31), chunk = (2 * kk + (lane >> 5)) ^ (lane & 7);
        return row * ROW + chunk * 8;
    }
};

// C = A B^T-style product for operands whose contraction index is fast in both: A bf16 through direct loads, B INT8
// dequantized through registers.  256 x 256 tile, 64-deep steps, eight waves (64 x 128 each), whole tiles only:
// M % 256 = N % 256 = K % 64 = 0, rows of A and B 16-byte aligned.  (With a bf16 B through direct loads as well the
// refresh's G Z^T ran 0.5 % slower than through k_tile_gemm: a wave's fragment reads queue behind its own pending
// direct loads, and with both operands direct nothing else is left to overlap them with.  With an INT8 B the direct
// A loads pay: about 4 % on the forward pass of a 7B layer and on grad_input on transposed storage.  With an INT8 B
// whose contraction index is slow, grad_input, they made it 1.5 % slower: that case stays in k_tile_gemm.)
template <int BL, typename OUT>
__global__ __launch_bounds__(512, 1) void k_gemm_kfast_direct(LinOperand A, LinOperand B, const uint16_t* __restrict__ bias,
                                                              OUT* __restrict__ C, int M, int N, int K, int tiles_m,
                                                              int tiles_n, LinBatch batch) {
    constexpr int TM = 256, TN = 256, BK = 64, NW = 8;
    static_assert(BL == kInt8KFast || BL == kInt8ZKFast, "B: INT8 with the contraction index fast");
    using AD = KFastDirect<TM, NW>;
    using SB = LinStage<BL, TN, BK, 512>;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][AD::ELEMS];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][SB::ELEMS];
    A.base = batch.a[blockIdx.y];
    B.base = static_cast<const char*>(B.base) + batch.strideB_bytes * blockIdx.y;
    C += batch.strideC * blockIdx.y;
    const int64_t ldc = batch.ldc ? batch.ldc : N;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
    const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
    if (tile >= (uint32_t)(tiles_m * tiles_n)) return;
    const int strip = (int)(tile / (uint32_t)(kLinStrip * tiles_n)), in_strip = (int)(tile % (uint32_t)(kLinStrip * tiles_n));
    const int strip_rows = min(kLinStrip, tiles_m - strip * kLinStrip);
    const int i0 = (strip * kLinStrip + in_strip % strip_rows) * TM, j0 = (in_strip / strip_rows) * TN;
    const uint16_t* Ag = static_cast<const uint16_t*>(A.base) + (int64_t)i0 * A.ld;
    const uint32_t a_byte = AD::lane_src_bytes(lane, A.ld);
    SB sb;
    auto gload = [&](int kt, int stage) {
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(Ag + kt * BK);
#pragma unroll
        for (int p = 0; p < AD::PER; ++p) {
            const int row0 = (wave * AD::PER + p) * 8;
            buffer_load_lds16(ra, As[stage] + row0 * AD::ROW, a_byte, 2u * (uint32_t)(row0 * A.ld));
        }
        sb.template fetch<kFetchAligned>(B, j0, N, kt * BK, K);
    };
    constexpr int MB = 2, NB = 4;
    f32x16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    auto mfma_step = [&](int stage) {
        __builtin_amdgcn_s_setprio(kMfmaPrio);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 af[MB], bf[NB];
#pragma unroll
            for (int a = 0; a < MB; ++a)
                af[a] = *reinterpret_cast<const bf16x8*>(As[stage] + AD::frag_offset(wm * 64 + a * 32, kk, lane));
#pragma unroll
            for (int b = 0; b < NB; ++b) bf[b] = SB::frag(Bs[stage], wn * 128 + b * 32, kk, lane);
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bf[b], acc[a][b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    auto landed = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };   // direct loads count like any other load
    const int KT = K / BK;
    // two LDS stages; the loads of step kt + 1 are issued before the MFMAs of step kt and land in the other stage
    gload(0, 0);
    sb.commit(Bs[0]);
    landed();
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        const bool more = kt + 1 < KT;
        if (more) gload(kt + 1, cur ^ 1);
        mfma_step(cur);
        if (more) sb.commit(Bs[cur ^ 1]);
        landed();
        __syncthreads();
    }
    float* tp = reinterpret_cast<float*>(As[0]) + wave * kTransposeFloats;
    static_assert(2 * AD::ELEMS >= NW * kTransposeFloats * 2, "the transpose buffers fit in the A stages");
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int col0 = j0 + wn * 128 + b * 32;
            const float bj = bias != nullptr ? __builtin_bit_cast(float, (uint32_t)bias[col0 + (lane & 31)] << 16) : 0.f;
            store_block<true>(acc[a][b], bj, tp, C, ldc, i0 + wm * 64 + a * 32, col0, M, N, lane);
        }
}

// DEEP_EXACT, DEEP_RAGGED: two register sets where every tile and step is whole, and where not.
template <int AL, int BL, typename OUT, int MB, int TN, int BK, int WM, bool DEEP_EXACT, bool DEEP_RAGGED, int KG = 1>
static void launch_tile_gemm_shape(const LinOperand& A, const LinOperand& B, const uint16_t* bias, OUT* C, int64_t M,
                                   int64_t N, int64_t K, hipStream_t st, const LinBatch* many, int count, int64_t ldc) {
    constexpr int TM = 32 * MB * WM;
    const int64_t tiles_m = (M + TM - 1) / TM, tiles_n = (N + TN - 1) / TN;
    const dim3 grid((unsigned)((tiles_m * tiles_n + 7) / 8 * 8), (unsigned)count);   // x: a multiple of the 8 XCDs
    LinBatch batch;
    if (many != nullptr) {
        batch = *many;
    } else {
        batch.a[0] = A.base;
        batch.strideB_bytes = 0;
        batch.strideC = 0;
    }
    batch.ldc = ldc;
    // no checks at all when every tile and every step is whole and rows start 16-byte aligned
    const bool exact = M % TM == 0 && N % TN == 0 && K % BK == 0 && A.ld % 8 == 0 && B.ld % 16 == 0;
    if (exact)
        hipLaunchKernelGGL((k_tile_gemm<AL, BL, true, OUT, MB, TN, BK, WM, DEEP_EXACT, KG>), grid, dim3(128 * WM * KG), 0, st, A, B, bias,
                           C, (int)M, (int)N, (int)K, (int)tiles_m, (int)tiles_n, batch);
    else
        hipLaunchKernelGGL((k_tile_gemm<AL, BL, false, OUT, MB, TN, BK, WM, DEEP_RAGGED, KG>), grid, dim3(128 * WM * KG), 0, st, A, B, bias,
                           C, (int)M, (int)N, (int)K, (int)tiles_m, (int)tiles_n, batch);
}

// Whether a product runs 64 x 64 tiles (see launch_tile_gemm).
template <int AL, int BL>
static bool lin_small(int64_t M, int64_t N, int count) {
    constexpr bool slow_weight = BL == kInt8KSlow || BL == kInt8ZKSlow, grad_w = AL == kBf16KSlow && BL == kBf16KSlow;
    return ((M + 127) / 128) * ((N + 127) / 128) * count < (slow_weight ? 160 : grad_w ? 200 : 256);
}

// Whether a product of the linear layer splits its contraction over the waves of a workgroup (T: its 32 x 32 tiles).  Against
// the tiles of launch_tile_gemm, us, split / not: forward, 256 tokens, 768 -> 768 (T = 192) 4.0 / 6.6, 2048 -> 2048 (512) 9.2 /
// 13.4, 500 tokens, 1024 -> 1024 (512) 6.5 / 7.4.  From 513 to 768 of them two groups of waves (64 x 64 tiles, at most a workgroup
// per CU) take 0.93 of the split's time on average over 22 shapes and ten lengths of the contraction from 512 to 11008: 0.78 to 0.91
// where rows start unaligned, 256 tokens, 2048 -> 3072 (768) 12.0 / 11.2, 4096 -> 3072 22.5 / 20.5, 2000 tokens, 11008 -> 384 (756)
// 62.7 / 52.4, 1000 tokens, 768 -> 768 the same; they lose up to 8 % at K = 2048 with some hundred ragged rows (500 tokens, 1280
// columns (640) 11.3 / 12.2, 1000 tokens, 768 columns 11.7 / 12.2) and 2 to 4 % on ragged tiles at K = 512.  Where they do not have
// a CU each, 32 tokens, 2048 -> 17408 (544) 12.9 / 19.9, 4096 -> 24576 (768) 24.7 / 37.0.  A weight with k
// slow (grad_input) needs twice the LDS per wave, and a chain that is long for the number of tiles: 256 tokens, 2048 -> 2048
// (512) 11.7 / 13.9, 500 tokens, K = 3001, 1007 columns (512) 55 / 95, but with grad_W in the same launch 256 tokens, K = 768,
// 2048 columns (512) 9.4 / 8.0, K = 1024, 2736 columns (688) 14.3 / 11.0.  grad_W: 512 x 512 (256), 1024 tokens 4.8 / 7.1, 4096
// tokens 10.9 / 30, but 256 tokens with grad_input in the same launch 4.2 / 3.7, and 768 x 768 (576), 1024 tokens 9.5 / 7.4.
// beside: the contraction of grad_W where a backward pass would run both products in one launch (whether it is asked for both or
// not), 0 otherwise.  There are no two groups there, and 64 x 64 tiles, which are fewer, leave grad_W more of the chip.  From 513
// to 768 tiles, a weight with k fast (stored transposed), both products / grad_input alone, split and 64 x 64 tiles: 1000 tokens,
// 768 columns (768), K = 768 14.0 and 11.1 / 6.4 and 6.9, K = 2048 21.6 and 20.0 / 12.0 and 17.8, 500 tokens, 1280 columns (640), K
// = 2048 17.9 and 19.4 / 11.3 and 17.8, 1000 tokens, 640 columns, K = 4096 32.5 and 35.7 / 20.6 and 31.9, but 2000 tokens, 320 columns
// (630), K = 2048 25.5 and 19.7 / 12.3 and 17.6, and on unaligned rows 602 tokens, 1207 columns, K = 2416 30.0 and 26.0, 536 tokens, 1143 columns,
// K = 3315 44.5 and 37.8.
template <int AL, int BL>
static bool lin_ksplit(int64_t M, int64_t N, int64_t K, int64_t beside) {
    const int64_t T = ((M + 31) / 32) * ((N + 31) / 32);
    if (AL == kBf16KSlow && BL == kBf16KSlow) return T <= 320 && K >= 512;
    if (BL == kInt8KSlow || BL == kInt8ZKSlow) return T <= 512 && K >= 3 * T;
    if (T <= 512 || K < 512) return T <= 768;
    if (beside != 0) return T <= 768 && K >= 2048 && K >= 2 * beside && K % 8 == 0 && N % 8 == 0;
    return T <= 768 && ((M + 63) / 64) * ((N + 63) / 64) > 256;   // (else two groups of waves, see launch_tile_gemm)
}

static LinProduct lin_product(const LinOperand& A, const LinOperand& B, uint16_t* C, int64_t M, int64_t N, int64_t K, int64_t ldc,
                              int tile) {
    return LinProduct{A, B, C, ldc, (int)M, (int)N, (int)K, (int)((M + tile - 1) / tile), (int)((N + tile - 1) / tile)};
}
// Whether every tile and every 64-deep step is whole and every row of the operands starts 16-byte aligned.
static bool lin_whole(const LinProduct& p, int tile) {
    return p.M % tile == 0 && p.N % tile == 0 && p.K % 64 == 0 && p.A.ld % 8 == 0 && p.B.ld % 16 == 0;
}
static unsigned lin_grid(const LinProduct& p) { return (unsigned)((p.tiles_m * p.tiles_n + 7) / 8 * 8); }   // the 8 XCDs

// Tile shape, from measurements on the linear layer (us unless said otherwise; T: 128 x 128 tiles of the product):
//  * large outputs with an INT8 B operand, or with the contraction index fast in both operands: 256 x 256 tiles with
//    64-deep steps, eight waves, one workgroup per CU (144 KB of LDS).  The B tile - and the dequantization of an
//    INT8 B - is shared by twice as many MFMAs as in a 128-row tile, global traffic per MFMA halves, and 64-deep
//    steps fetch whole cache lines of operands whose rows run along k.  7B shapes, ms per decoder layer at 4096 tokens:
//    forward 2.24 -> 1.87, grad_input 1.82 -> 1.66 (256 x 256 x 32 with eight waves: 1.72; 256 x 128 x 64: forward
//    unchanged at 2.24).  Two register sets where all tiles are whole (grad_input, 4096 tokens, 4096 -> 4096: 134 against
//    137 with one; 8192 tokens 253 / 260); with ragged edges only where the last round of tiles leaves most CUs idle and the
//    columns are whole (forward, 3000 tokens, 4096 -> 11008, 516 tiles: 333 / 377).  That line is from edges with checks on every
//    chunk; with clamped ones two sets are ahead elsewhere too (5000 tokens, 2048 -> 5461, 440 tiles: 122 / 135; 3000 tokens,
//    2048 -> 5461, 264 tiles: 115 / 130; grad_input, 3000 tokens, 5461 columns: 134 / 138).
//  * otherwise four waves: 128 x 128 x 64 when an operand is INT8 or both have k fast, with one register set where the
//    tiles make one round of two workgroups per CU (256 < T <= 512) and two sets below and above: forward, 2048 tokens,
//    2048 -> 2048 (T = 256) 26.7 with two against 31.3, 4096 tokens, 2048 -> 1280 (320) 40.0 / 36.0, 512 tokens, 4096 ->
//    11008 (344) 75 / 67, 6000 tokens, 2048 -> 1920 (705) 74 / 77, 1024 tokens, 4096 -> 11008 (688) 124 / 135.  An INT8 B
//    with k slow: two sets up to T = 256 only where rows and columns are whole (grad_input, 1024 tokens, 4096 -> 4096 46 /
//    57; ragged, with clamped edges, 1000 tokens 50 / 59 and 4100 tokens, 768 -> 768 13.3 / 14.4, but 1000 tokens, 5461 columns 54 /
//    48), and beyond T = 512 128 x 128 x 32 with four workgroups per CU (4096 tokens, 2048 -> 2048 (512): 64-deep 42.5, 32-deep
//    44; 4100 tokens (528) 62 / 55; 3000 tokens, 4096 -> 4096 (768) 132 / 125).
//    grad_W: 128 x 256 x 32 when that fills the chip twice, 128 x 128 x 32 below, with two register sets up to T = 256
//    (1000 tokens, 2048 x 2048: 17.1 against 18.1, 2000 x 2000 17.1 / 20.7) and where everything is whole (2048 tokens, 3072 x
//    2048, T = 384: 37.1 / 38.7; ragged, 2000 tokens, 3000 x 3000, T = 576: 55.3 / 54.7, 3001 x 2048, T = 384: 100 / 69).
//  * 64 x 64 x 64, four waves of one 32 x 32 block each, where 128 x 128 tiles would leave CUs idle: a K step of a lone
//    workgroup is a serial chain (fragments, MFMAs, commit, barrier), 1.2 us for 128 x 128 x 64 before the commit and the
//    fetches went between the MFMAs.  64 / 128: forward, 1000 tokens, 768 -> 2048 (T = 128) 9.7 / 12.8, 256 x 4096 -> 11008
//    (172) 47 / 48, 2048 tokens, 2048 -> 1664 (208) 31 / 27, ragged, 3000 tokens, 2048 -> 1280 (240) 33 / 29, but 1000 tokens,
//    1024 -> 2736 (176) 14.5 / 15.9 and 300 tokens, 4096 -> 11008 (258) 60 / 64; grad_input, 1000 x 2048 -> 2048 (128) 20 / 31,
//    256 x 4096 -> 11008 (172) 53 / 43; grad_W, 2048 tokens, 1024 x 1024 (64) 13 / 29, 1024 tokens, 1536 x 2048 (192) 15.7 / 15.9, 1664 x 2048 (208)
//    20.8 / 15.9.
//  * two groups of waves (INT8 B, K >= 512) where these tiles would be at most a workgroup per CU, us, one group / two:
//    64 x 64, forward, 256 tokens, 4096 -> 4096 31.0 / 20.5, 500 tokens, 2048 -> 2048 13.6 / 11.2, 512 -> 2048 6.3 / 5.9, 1000 tokens,
//    1024 -> 1024 9.0 / 7.9, grad_input 256 x 11008 -> 4096 80 / 50; shorter contractions go either way (500 tokens, 2048 columns, K =
//    256 4.4 / 4.5, 320 4.6 / 4.8, 384 5.2 / 4.8, 448 5.3 / 5.3).
//    128 x 64 where 64 x 64 ones are more than 256 and these are not: forward, 1000 tokens, 2048 -> 2048 21.7 / 18.9, grad_input 23.2 /
//    19.8 (two groups of 64 x 64 tiles 20.1 and 22.4; 288 tiles of 128 x 64, 1500 tokens, 1536 -> 1536, 19.8 / 24.2).  Two groups' time
//    over one's in 340 random products on aligned rows, forward and k slow alike: a whole number of steps, K = 512 to 576 1.02, 577 to 768 0.97,
//    up to 1600 0.92, beyond 0.85; with a partial last step, which one group takes while the other waits, K = 512 to 640 1.09, 641 to 896
//    1.03, 897 to 1024 0.99, up to 1600 0.96, beyond 0.88: from 640 and 960 on.  Where
//    rows start unaligned two groups lose on short contractions and gain on long ones; forward, 1000 tokens, 2048 columns, K = 2047
//    27.2 / 30.0, 2501 31.4 / 31.2, 3001 36.3 / 34.3, 4001 47.4 / 43.6 and eleven other shapes alike (K = 2047 0.85 to 1.02 of two
//    groups' time, 3001 0.96 to 1.10, 4101, 5000, 5461 and 7001 0.96 to 1.23, 1.08 on average), so from 4096 on.  A weight with k slow,
//    56 shapes of 100 to 2000 tokens, one group's time over two groups': odd rows, K = 1024 0.95 on average, 2048 1.00, 3008 1.01
//    (transposed forward, 1000 tokens, 2047 columns, K = 1024 13.2 / 14.6, 2048 23.3 / 24.4, 5461 63.2 / 61.0); rows of a multiple of 4,
//    up to 1024 tokens, K = 768 1.00, 1024 1.03, 2048 1.03, more tokens 0.93 and 0.97 (even ones are like these, 363 tokens, 4162
//    columns, K = 1472 17.1 / 16.0): from 2048 on, and from 1024 on even rows up to 1024 tokens.
//    128 x 128 x 64, forward, 1024 tokens, 4096 -> 4096 51 / 46, grad_input, 2000 tokens, 2000 -> 2000 37.5 / 27.7, 256 tokens, 4096 -> 11008
//    43 / 38, but not on a short contraction (2048 tokens, 2048 columns, forward, K = 512 10.7 / 11.0, 520 14.3 / 15.1, 768 14.5 / 14.6,
//    1024 18.0 / 17.9; grad_input on whole tiles, 1024 tokens, 4096 columns, 512 10.4 / 11.0, 1024 17.3 / 17.7, 2048 29.6 / 29.6;
//    ragged, 1000 tokens, 3000 columns, 512 12.5 / 11.5, 513 16.0 / 16.4, 768 18.4 / 15.4,
//    1733 tokens, 1456 columns, 595 17.4 / 16.2, 2165 tokens, 1296 columns, 571 16.9 / 15.8).
//    grad_W gains nothing (1000 tokens, 2048 x 2048, 17.9 / 18.8).
// ldc: row pitch of C in elements (0: N).  beside: see lin_ksplit; two groups only where it is 0.
template <int AL, int BL, typename OUT>
static int launch_tile_gemm(const LinOperand& A, const LinOperand& B, const uint16_t* bias, OUT* C, int64_t M, int64_t N,
                            int64_t K, hipStream_t st, const LinBatch* many = nullptr, int count = 1, int64_t ldc = 0,
                            int64_t beside = 0) {
    if constexpr (AL == kBf16KFast && BL != kBf16KFast && BL != kBf16KSlow && std::is_same_v<OUT, uint16_t>) {
        if (many == nullptr && lin_ksplit<AL, BL>(M, N, K, beside)) {
            const LinProduct p = lin_product(A, B, C, M, N, K, ldc ? ldc : N, 32);
            auto launch = [&](auto exact, auto waves) {
                hipLaunchKernelGGL((k_ksplit_gemm<BL, exact.value, waves.value>), dim3(lin_grid(p)), dim3(64 * waves.value), 0, st,
                                   p, bias);
            };
            using Four = std::integral_constant<int, 4>;
            using Eight = std::integral_constant<int, 8>;
            // eight waves up to one workgroup per CU (256 tokens, 2736 -> 1024 (T = 256) 7.5 us, with four 9.3; 64 tokens, 2048 ->
            // 5461 (342) 10.3 / 9.2)
            const bool eight = p.tiles_m * p.tiles_n <= 256;
            if (lin_whole(p, 32)) eight ? launch(std::true_type(), Eight()) : launch(std::true_type(), Four());
            else eight ? launch(std::false_type(), Eight()) : launch(std::false_type(), Four());
            return check_launch();
        }
        // Two groups of waves per tile (see tile_gemm) while tiles are about a workgroup per CU or fewer
        if (many == nullptr && beside == 0 && K >= 512) {
            const int64_t tiles_m = (M + 127) / 128, tiles_n = (N + 63) / 64;
            constexpr bool slow = BL == kInt8KSlow || BL == kInt8ZKSlow;
            auto launch = [&](auto mb, auto tn) {
                launch_tile_gemm_shape<AL, BL, OUT, mb.value, tn.value, 64, 2, true, true, 2>(A, B, bias, C, M, N, K, st, nullptr, 1,
                                                                                             ldc);
                return check_launch();
            };
            using N64 = std::integral_constant<int, 64>;
            using N128 = std::integral_constant<int, 128>;
            if (!lin_small<AL, BL>(M, N, 1)) {
                const bool whole = M % 128 == 0 && N % 128 == 0;
                const int64_t least = !slow ? 768 : whole ? 1536 : K % 8 == 0 ? 512 : 544;
                if (K >= least && tiles_m * ((N + 127) / 128) <= 256) return launch(std::integral_constant<int, 2>(), N128());
            } else if ((M + 63) / 64 * tiles_n <= 256) {
                return launch(std::integral_constant<int, 1>(), N64());
            } else if (tiles_m * tiles_n <= 256) {
                // dense rows start 16-byte aligned; k slow: or those of A do and the contraction is long enough for the weight's
                // (sizes, not the pitches: the order of the sums does not depend on them)
                const bool wide = slow ? K % 8 == 0 && (N % 16 == 0 || K >= (N % 2 == 0 && M <= 1024 ? 1024 : 2048)) : K % 16 == 0;
                if (wide ? K >= (K % 64 == 0 ? 640 : 960) : K >= 4096) return launch(std::integral_constant<int, 2>(), N64());
            }
        }
    }
    constexpr bool both_fast = (AL == kBf16KFast || AL == kInt8KFast || AL == kInt8ZKFast) &&
                               (BL == kBf16KFast || BL == kInt8KFast || BL == kInt8ZKFast);
    if constexpr (AL == kBf16KSlow && BL == kBf16KSlow) {
        const int64_t tiles_m = M / kLinTM, tiles_n = N / 256;
        if (many == nullptr && M % kLinTM == 0 && N % 256 == 0 && K % 32 == 0 && bias == nullptr &&
            tiles_m * tiles_n >= 512 && K >= 32 && A.ld == M && B.ld == N && (ldc == 0 || ldc == N)) {
            const unsigned grid = (unsigned)((tiles_m * tiles_n + 7) / 8 * 8);
            hipLaunchKernelGGL((k_gemm_kslow_direct<OUT>), dim3(grid), dim3(256), 0, st, static_cast<const uint16_t*>(A.base),
                               static_cast<const uint16_t*>(B.base), C, (int)M, (int)N, (int)K, (int)tiles_m, (int)tiles_n);
            return check_launch();
        }
    }
    constexpr bool int8_b = BL == kInt8KFast || BL == kInt8KSlow || BL == kInt8ZKFast || BL == kInt8ZKSlow;
    if constexpr (int8_b || both_fast) {
        if (M >= 1024 && ((M + 255) / 256) * ((N + 255) / 256) * count >= 256) {   // at least one workgroup per CU
            if constexpr (AL == kBf16KFast && (BL == kInt8KFast || BL == kInt8ZKFast)) {
                // whole tiles and aligned rows: the bf16 operand goes straight into LDS
                if (M % 256 == 0 && N % 256 == 0 && K % 64 == 0 && A.ld % 8 == 0 && B.ld % 16 == 0) {
                    const int64_t tiles_m = M / 256, tiles_n = N / 256;
                    const dim3 grid((unsigned)((tiles_m * tiles_n + 7) / 8 * 8), (unsigned)count);
                    LinBatch batch;
                    if (many != nullptr) {
                        batch = *many;
                    } else {
                        batch.a[0] = A.base;
                        batch.strideB_bytes = 0;
                        batch.strideC = 0;
                    }
                    batch.ldc = ldc;
                    hipLaunchKernelGGL((k_gemm_kfast_direct<BL, OUT>), grid, dim3(512), 0, st, A, B, bias, C, (int)M, (int)N,
                                       (int)K, (int)tiles_m, (int)tiles_n, batch);
                    return check_launch();
                }
            }
            const int64_t last = (((M + 255) / 256) * ((N + 255) / 256) * count - 1) % 256 + 1;   // tiles of the last round
            if (last <= 64 && N % 256 == 0)
                launch_tile_gemm_shape<AL, BL, OUT, 2, 256, 64, 4, true, true>(A, B, bias, C, M, N, K, st, many, count, ldc);
            else
                launch_tile_gemm_shape<AL, BL, OUT, 2, 256, 64, 4, true, false>(A, B, bias, C, M, N, K, st, many, count, ldc);
            return check_launch();
        }
    }
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128) * count;
    if (lin_small<AL, BL>(M, N, count)) {
        launch_tile_gemm_shape<AL, BL, OUT, 1, 64, 64, 2, true, true>(A, B, bias, C, M, N, K, st, many, count, ldc);
    } else if constexpr (both_fast || int8_b) {
        if constexpr (!both_fast) {
            if (tiles128 > 512) {
                launch_tile_gemm_shape<AL, BL, OUT, 2, 128, 32, 2, true, false>(A, B, bias, C, M, N, K, st, many, count, ldc);
                return check_launch();
            }
        }
        const bool two = tiles128 > 256 ? tiles128 > 512 : both_fast || (M % 128 == 0 && N % 128 == 0);
        if (two)
            launch_tile_gemm_shape<AL, BL, OUT, 2, 128, 64, 2, true, true>(A, B, bias, C, M, N, K, st, many, count, ldc);
        else
            launch_tile_gemm_shape<AL, BL, OUT, 2, 128, 64, 2, false, false>(A, B, bias, C, M, N, K, st, many, count, ldc);
    } else if (((M + kLinTM - 1) / kLinTM) * ((N + 255) / 256) * count >= 512) {
        launch_tile_gemm_shape<AL, BL, OUT, 2, 256, 32, 2, true, true>(A, B, bias, C, M, N, K, st, many, count, ldc);
    } else if (tiles128 <= 256) {
        launch_tile_gemm_shape<AL, BL, OUT, 2, 128, 32, 2, true, true>(A, B, bias, C, M, N, K, st, many, count, ldc);
    } else {
        launch_tile_gemm_shape<AL, BL, OUT, 2, 128, 32, 2, true, false>(A, B, bias, C, M, N, K, st, many, count, ldc);
    }
    return check_launch();
}

// dx (tokens x n_in = dy W, W with layout BL) and grad_W (rows x cols = A1^T B1 over the tokens): one launch where both
// products fit 64 x 64 tiles or are split over waves, otherwise one after the other.  Either output may be missing.  One 130M
// decoder layer on 256 tokens, forward and backward: 181 us with two launches per backward call, 151 with one; its backward
// calls alone, with the chain of grad_input split, 768 -> 768 7.0 -> 5.9, 2048 -> 768 14.7 -> 9.5.  grad_W comes along up to
// the chip's 256 tiles of 128 x 128, further than it runs 64 x 64 tiles alone: 256 tokens, 2048 -> 1664 (208) 13.8 us, two
// launches 18.8; 1024 tokens, 2048 -> 1920 (240) 33.1 / 36.4.
template <int BL>
static int launch_linear_backward(const LinOperand& A0, const LinOperand& B0, uint16_t* dx, int64_t M0, int64_t N0, int64_t K0,
                                  int64_t ldc0, const LinOperand& A1, const LinOperand& B1, uint16_t* G, int64_t M1, int64_t N1,
                                  int64_t K1, int64_t ldc1, hipStream_t st) {
    const bool split1 = lin_ksplit<kBf16KSlow, kBf16KSlow>(M1, N1, K1, 0);
    const bool pair1 = split1 || ((M1 + 127) / 128) * ((N1 + 127) / 128) < 256;
    const int64_t fits = lin_small<kBf16KFast, BL>(M0, N0, 1) && pair1 ? K1 : 0;
    const bool split0 = lin_ksplit<kBf16KFast, BL>(M0, N0, K0, fits);
    const bool pair0 = split0 || lin_small<kBf16KFast, BL>(M0, N0, 1);
    const int tile0 = split0 ? 32 : 64, tile1 = split1 ? 32 : 64;
    const LinProduct p0 = lin_product(A0, B0, dx, M0, N0, K0, ldc0, tile0), p1 = lin_product(A1, B1, G, M1, N1, K1, ldc1, tile1);
    // `with0` of the first product's workgroups, `with1` of the second's
    auto launch_pair = [&](bool with0, bool with1) {
        const unsigned grid0 = with0 ? lin_grid(p0) : 0, grid = grid0 + (with1 ? lin_grid(p1) : 0);
        const bool exact = (!with0 || lin_whole(p0, tile0)) && (!with1 || lin_whole(p1, tile1));
        auto launch = [&](auto e, auto s0, auto s1) {
            hipLaunchKernelGGL((k_gemm_pair<BL, e.value, s0.value, s1.value>), dim3(grid), dim3(256), 0, st, p0, p1, grid0);
        };
        auto pick = [&](auto e) {
            if (split0) split1 ? launch(e, std::true_type(), std::true_type()) : launch(e, std::true_type(), std::false_type());
            else split1 ? launch(e, std::false_type(), std::true_type()) : launch(e, std::false_type(), std::false_type());
        };
        exact ? pick(std::true_type()) : pick(std::false_type());
        return check_launch();
    };
    if (dx && G && pair0 && pair1) return launch_pair(true, true);
    // (a product whose contraction is split runs in this kernel alone too: the same bits whether the other is asked for or not)
    if (dx) {
        if (split0) {
            if (int e = launch_pair(true, false)) return e;
        } else if (int e = launch_tile_gemm<kBf16KFast, BL, uint16_t>(A0, B0, nullptr, dx, M0, N0, K0, st, nullptr, 1, ldc0,
                                                                                      fits)) {
            return e;
        }
    }
    if (!G) return QG_OK;
    if (split1) return launch_pair(false, true);
    return launch_tile_gemm<kBf16KSlow, kBf16KSlow, uint16_t>(A1, B1, nullptr, G, M1, N1, K1, st, nullptr, 1, ldc1);
}

}  // namespace qg
