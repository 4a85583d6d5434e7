// Host dispatch of the projection and back-projection kernels (see qg_gemm_kernels.h).
#include "qg_gemm_kernels.h"

#include <type_traits>

namespace qg {

// ---------------------------------------------------------------------------
// Host dispatch
// ---------------------------------------------------------------------------
static inline unsigned grid8(uint32_t tiles) { return ((tiles + 7u) / 8u) * 8u; }

// Edge mode of a matrix for tiles of TM (along r for the projection, along m for the back-projection) x TN and K
// steps of BK over `kdim`; ld is the row pitch of the n-wide arrays.  The direct loads need 16-byte aligned rows
// (ld % 8, and r % 16 for the 8-byte P fetches) and 32-bit per-lane offsets.
static inline bool unaligned(int64_t ld, int64_t r) { return ld > (int64_t(1) << 24) || (ld % 8) != 0 || (r % 16) != 0; }
static inline int edge_mode(int64_t tiled, int TM, int64_t n, int64_t ld, int TN, int64_t kdim, int BK, int64_t r) {
    if (unaligned(ld, r)) return kUnaligned;
    if ((tiled % TM) == 0 && (n % TN) == 0 && (kdim % BK) == 0) return kExact;
    return kMasked;
}
int project_mode(int64_t m, int64_t n, int64_t ld, int64_t r) { return edge_mode(r, kManyProjBM, n, ld, kManyProjBN, m, 32, r); }
int backproject_mode(int64_t m, int64_t n, int64_t ld, int64_t r) {
    return edge_mode(m, kManyBpBM, n, ld, kManyBpBN, r, 32, r);
}

// Tile configurations: tile, K step, wave grid, pipeline depth (LDS stages of the direct loads), workgroups per CU the
// instance is compiled for in the three edge modes.
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int NS_, int W0, int W1, int W2>
struct ProjCfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_, NS = NS_, NT = WGM_ * WGN_ * 64;
    static constexpr int kWg[3] = {W0, W1, W2};
};
template <int BM_, int BK_, int WGn_, int WGm_, int NS_, int W0, int W1, int W2>
struct BpCfg {
    static constexpr int BM = BM_, BN = kGroup, BK = BK_, WGn = WGn_, WGm = WGm_, NS = NS_, NT = WGn_ * WGm_ * 64;
    static constexpr int kWg[3] = {W0, W1, W2};
};
template <typename F>
static auto with_mode(int mode, F f) {
    if (mode == kExact) return f(std::integral_constant<int, kExact>());
    if (mode == kMasked) return f(std::integral_constant<int, kMasked>());
    return f(std::integral_constant<int, kUnaligned>());
}
// Projection tiles (rows of R x columns), and the rule that picks one for a launch.  A K step of one workgroup alone on
// its CU is bound by its own serial chain (fragment reads, MFMAs, dequantization, barrier): 0.31 us for 128 x 128, 0.23 us
// for 64 x 128, against 0.11 and 0.05 us of MFMA time, so a launch with few tiles takes the smaller ones, with four tiles
// in flight and the dequantization between the MFMAs; a launch with 128 x 256 workgroups enough (three fit a CU) lets
// the workgroups cover for each other and takes the tile with the least staging per MFMA.  Measured with Adam (us, tiles
// 64 x 128 / 128 x 128, at the number T of 128 x 128 tiles): 1024 x 1024, r = 256: T = 256 26 / 31, 320 32 / 41, 384 35 / 41,
// 448 46 / 45; 2048 x 2048, r = 512: 320 45 / 53, 384 51 / 57, 512 66 / 66; 4096 rows, r = 1024: 320 73 / 83, 376 86 / 87,
// 448 102 / 92: they cross between 384 and 448.  128 x 128 / 128 x 256, at the number of the latter: r = 256: 512 90 / 96,
// 1024 175 / 188, 1536 278 / 280; r = 512: 768 170 / 172, 1152 261 / 264, 1536 348 / 338; r = 1024: 768 269 / 250, 896
// 307 / 317, 1024 367 / 356, 1536 541 / 502.  Unaligned rows are staged through registers, which leaves the 128 x 256 instance two
// workgroups per CU (us, 128 x 128 / 128 x 256: 24 of 2048 x 5461, r = 512, 655 / 715, eight of 4096 x 11007, r = 1024, 1262 /
// 1310, 48 of 1024 x 1021, r = 256, 102 / 102); 64 x 128 / 128 x 128: 1024 x 1021, r = 256: T = 256 29 / 38, 384 34 / 40, 512 41 /
// 42, 768 55 / 50; 2048 x 5461, r = 512: 344 70 / 72, 516 108 / 93, so their line could lie between 400 and 500.  A matrix of
// 64 rows of R or fewer would leave half of every 128-row tile empty (64 x 100000, r = 64: 26 us; 128 x 128 34, 128 x 256 30).
template <typename F>
static auto with_proj(int cfg, F f) {
    if (cfg == kProj64) return f(ProjCfg<64, 128, 32, 2, 2, 4, 2, 2, 2>());
    if (cfg == kProj128) return f(ProjCfg<128, 128, 32, 2, 2, 4, 3, 3, 3>());
    return f(ProjCfg<kManyProjBM, kManyProjBN, 32, 2, 2, 2, 3, 3, 2>());
}
// r: the largest of the launch; tiles128: its 128 x 128 tiles, tiles256: its 128 x 256 tiles
int proj_config(int mode, int64_t r, int64_t tiles128, int64_t tiles256) {
    if (r <= 64 || tiles128 <= 320) return kProj64;
    return mode == kUnaligned || tiles256 < 1024 ? kProj128 : kProj256;
}
int64_t proj_tiles(int cfg, int64_t n, int64_t r) {
    return with_proj(cfg, [&](auto c) { return ((r + c.BM - 1) / c.BM) * ((n + c.BN - 1) / c.BN); });
}
int64_t proj_tiles_r(int cfg, int64_t r) { return with_proj(cfg, [&](auto c) { return (r + c.BM - 1) / c.BM; }); }
static int proj_config_of(int64_t n, int64_t ld, int64_t r, int64_t count) {
    return proj_config(unaligned(ld, r) ? kUnaligned : kExact, r, proj_tiles(kProj128, n, r) * count,
                       proj_tiles(kProj256, n, r) * count);
}

// Back-projection: 128 rows x one block of 256 columns, three workgroups per CU, once that gives every CU a workgroup and
// a half; below that 64 rows with four tiles in flight (us, 64 / 128 rows, at the number of the latter: 1024 x 1024, r = 256:
// 128 9.1 / 13.4, 256 13.1 / 14.5, 320 18.9 / 19.8, 384 19.3 / 20.1, 448 22.1 / 20.5; 2048 x 2048, r = 512: 128 11.8 / 17.6,
// 256 16.9 / 18.8, 384 25.1 / 25.7, 512 30.6 / 26.5; the weight tile shares the staging LDS, the VALU-heavy update epilogue of
// one workgroup overlaps the main loops of the others).  Unaligned rows: up to 300, where the loops with checks on
// every chunk crossed.  The present ones cross later, about where 64-row tiles make one round of three workgroups per CU (1024 x
// 1021, r = 256: 256 22 / 31, 288 29 / 43, 384 29 / 41, 448 37 / 44; 20000 x 300, r = 64, 314: 25 / 37; 2048 x 5461, r = 512, 352:
// 35 / 42; 2560 x 5461, 440: 47 / 42; 4096 x 4093, r = 1024, 512: 81 / 69).
template <typename F>
static auto with_bp(int cfg, F f) {
    if (cfg == kBp64) return f(BpCfg<64, 32, 2, 2, 4, 2, 2, 2>());
    return f(BpCfg<kManyBpBM, 32, 2, 2, 2, 3, 3, 2>());   // unaligned operands pass through registers
}
int bp_config(int mode, int64_t tiles128) { return tiles128 < (mode == kUnaligned ? 300 : 384) ? kBp64 : kBp128; }
int64_t bp_tiles_m(int cfg, int64_t m) { return with_bp(cfg, [&](auto c) { return (m + c.BM - 1) / c.BM; }); }

// The projection with Adam: a masked launch whose rows share cache lines has instances of its own (see kAuxStream).
template <typename F>
static auto with_adam_mode(int mode, bool lines, F f) {
    if (mode == kMasked && !lines) return f(std::integral_constant<int, kMaskedShared>());
    return with_mode(mode, f);
}
constexpr int wg_index(int mode) { return mode == kMaskedShared ? kMasked : mode; }

// Tiles in flight: two in the unaligned kernels.  Their operands pass through registers, and those of four tiles spilled (with
// the checks that kept the compiler from it, and from one K step to the next a load at a time at the edge, 2048 x 5461, r =
// 512, with Adam took 139 us instead of 50, the back-projection 76 instead of 46; 24 of them 812 / 688 and 808 / 676).
constexpr int stages(int mode, int ns) { return mode == kUnaligned ? 2 : ns; }
#define QG_PROJ(KERNEL, C, M, ...) (KERNEL<C::BM, C::BN, C::BK, C::WGM, C::WGN, stages(M, C::NS), M, C::kWg[wg_index(M)]>)
// ld: row pitch in elements of G, R, M, V, N (n for dense rows).
int launch_project_adam(const uint8_t* Pq, const float* Ps, const uint16_t* G, float* R, float* M, float* V,
                        uint16_t* N, int64_t m, int64_t n, int64_t ld, int64_t r, int64_t step, const qg_hparams* hp,
                        hipStream_t stream) {
    const AdamCoef coef = make_adam_coef(hp, step);
    return with_proj(proj_config_of(n, ld, r, 1), [&](auto c) {
        using C = decltype(c);
        return with_adam_mode(edge_mode(r, C::BM, n, ld, C::BN, m, C::BK, r), whole_lines(ld), [&](auto mode) {
            const uint32_t tr = (uint32_t)((r + C::BM - 1) / C::BM), tiles = tr * (uint32_t)((n + C::BN - 1) / C::BN);
            constexpr int WG = C::NS == 2 ? 2 : C::kWg[wg_index(mode())];   // (for three the 128 x 256 instance spills)
            hipLaunchKernelGGL((k_project_adam<C::BM, C::BN, C::BK, C::WGM, C::WGN, stages(mode(), C::NS), mode(), WG>),
                               dim3(grid8(tiles)), dim3(C::NT), 0, stream, Pq, Ps, G, R, M, V, N, (int)m, (int)n, (int)ld, (int)r,
                               tr, tiles, coef);
            return check_launch();
        });
    });
}

// Grouped launches: the plan stores the matrices class by class (kExact, kMasked, kUnaligned); each class that is
// not empty gets a launch of its own kernel instance.
static inline int class_first(const PlanHeader* h, int cls) {
    int first = 0;
    for (int c = 0; c < cls; ++c) first += h->class_count[c];
    return first;
}
static inline int class_count(const PlanHeader* h, int cls) { return h->class_count[cls]; }

int launch_project_adam_many(const PlanHeader* plan_host, const PlanHeader* plan_dev, int write_R, int64_t step,
                             const qg_hparams* hp, hipStream_t stream) {
    const AdamCoef coef = make_adam_coef(hp, step);
    for (int cls = 0; cls < kPlanClasses; ++cls) {
        const int cnt = class_count(plan_host, cls), first = class_first(plan_host, cls);
        const uint32_t tiles = plan_host->proj_tiles[cls];
        if (cnt == 0 || tiles == 0) continue;
        // (one matrix that shares lines decides for its class; us, 24 of 2048 x 5472, r = 512, one of them with n = 5464: 494 / 499,
        // two 516 / 513, three 537 / 528, all 795 / 561)
        bool lines = true;
        for (int i = first; i < first + cnt; ++i) lines = lines && whole_lines(plan_matrices(plan_host)[i].ld);
        const int e = with_proj((int)plan_host->proj_cfg[cls], [&](auto c) {
            using C = decltype(c);
            return with_adam_mode(cls, lines, [&](auto mode) {
                // (unaligned 128 x 128 tiles: four workgroups per CU; us, three / four: 24 of 2048 x 5461, r = 512, 695 /
                // 655, twelve 362 / 363, six of 4096 x 11007, r = 1024, 1000 / 958, 96 of 1024 x 1021, r = 256, 211 / 215)
                constexpr int WG = mode() == kUnaligned && C::BM == 128 && C::BN == 128 ? 4 : C::kWg[wg_index(mode())];
                hipLaunchKernelGGL((k_project_adam_many<C::BM, C::BN, C::BK, C::WGM, C::WGN, stages(mode(), C::NS), mode(), WG>),
                                   dim3(grid8(tiles)), dim3(C::NT), 0, stream, plan_dev, first, cnt, tiles, write_R, coef);
                return check_launch();
            });
        });
        if (e) return e;
    }
    return QG_OK;
}

int launch_project(const uint8_t* Pq, const float* Ps, const uint16_t* G, float* R, int64_t m, int64_t n, int64_t ld,
                   int64_t r, hipStream_t stream) {
    return with_proj(proj_config_of(n, ld, r, 1), [&](auto c) {
        using C = decltype(c);
        return with_mode(edge_mode(r, C::BM, n, ld, C::BN, m, C::BK, r), [&](auto mode) {
            const uint32_t tr = (uint32_t)((r + C::BM - 1) / C::BM), tiles = tr * (uint32_t)((n + C::BN - 1) / C::BN);
            hipLaunchKernelGGL(QG_PROJ(k_project, C, mode()), dim3(grid8(tiles)), dim3(C::NT), 0, stream, Pq, Ps, G, R, (int)m,
                               (int)n, (int)ld, (int)r, tr, tiles);
            return check_launch();
        });
    });
}

// R_z = dequant(P_z)^T G_z for `count` (<= kProjBatchMax) matrices of one shape in one launch (same arithmetic per element
// as launch_project: the order of the sum over m does not depend on the tile shape).
int launch_project_batch(const ProjBatch& batch, int count, float* R, int64_t strideR, int64_t m, int64_t n, int64_t ld,
                         int64_t r, hipStream_t stream) {
    return with_proj(proj_config_of(n, ld, r, count), [&](auto c) {
        using C = decltype(c);
        return with_mode(edge_mode(r, C::BM, n, ld, C::BN, m, C::BK, r), [&](auto mode) {
            const uint32_t tr = (uint32_t)((r + C::BM - 1) / C::BM), tiles_per = tr * (uint32_t)((n + C::BN - 1) / C::BN);
            const uint32_t tiles = tiles_per * (uint32_t)count;
            hipLaunchKernelGGL(QG_PROJ(k_project_batch, C, mode()), dim3(grid8(tiles)), dim3(C::NT), 0, stream, batch, R,
                               strideR, (int)m, (int)n, (int)ld, (int)r, tr, tiles_per, tiles);
            return check_launch();
        });
    });
}

// ld: row pitch in elements of N and Wq (n for dense rows); the U dump, if asked for, is dense.
int launch_backproject(const uint8_t* Pq, const float* Ps, const uint16_t* N, int8_t* Wq, float* Ws, float* Wz,
                       float* Udbg, int64_t m, int64_t n, int64_t ld, int64_t r, float alpha, float lr, uint64_t seed,
                       int64_t step, hipStream_t stream) {
    const uint32_t key = sr_key(seed, (uint64_t)step, 0u);
    const int cfg = bp_config(unaligned(ld, r) ? kUnaligned : kExact, bp_tiles_m(kBp128, m) * ((n + kGroup - 1) / kGroup));
    return with_bp(cfg, [&](auto c) {
        using C = decltype(c);
        return with_mode(edge_mode(m, C::BM, n, ld, kGroup, r, C::BK, r), [&](auto mode) {
            constexpr int MODE = mode();
            const uint32_t tm = (uint32_t)((m + C::BM - 1) / C::BM), tiles = tm * (uint32_t)((n + kGroup - 1) / kGroup);
            const dim3 grid(grid8(tiles)), block(C::NT);
            if (Wz != nullptr)   // zero-point weights (no U dump)
                hipLaunchKernelGGL((k_backproject<C::BM, C::BK, C::WGn, C::WGm, stages(MODE, C::NS), MODE, false, C::kWg[MODE], true>),
                                   grid, block, 0, stream, Pq, Ps, N, Wq, Ws, Wz, nullptr, (int)m, (int)n, (int)ld, (int)r,
                                   alpha, lr, key, tm, tiles);
            else if (Udbg != nullptr)
                hipLaunchKernelGGL((k_backproject<C::BM, C::BK, C::WGn, C::WGm, stages(MODE, C::NS), MODE, true, C::kWg[MODE]>), grid,
                                   block, 0, stream, Pq, Ps, N, Wq, Ws, nullptr, Udbg, (int)m, (int)n, (int)ld, (int)r, alpha,
                                   lr, key, tm, tiles);
            else
                hipLaunchKernelGGL((k_backproject<C::BM, C::BK, C::WGn, C::WGm, stages(MODE, C::NS), MODE, false, C::kWg[MODE]>), grid,
                                   block, 0, stream, Pq, Ps, N, Wq, Ws, nullptr, nullptr, (int)m, (int)n, (int)ld, (int)r,
                                   alpha, lr, key, tm, tiles);
            return check_launch();
        });
    });
}

int launch_project_many(const PlanHeader* plan_host, const PlanHeader* plan_dev, hipStream_t stream) {
    for (int cls = 0; cls < kPlanClasses; ++cls) {
        const int cnt = class_count(plan_host, cls), first = class_first(plan_host, cls);
        const uint32_t tiles = plan_host->proj_tiles[cls];
        if (cnt == 0 || tiles == 0) continue;
        const int e = with_proj((int)plan_host->proj_cfg[cls], [&](auto c) {
            using C = decltype(c);
            return with_mode(cls, [&](auto mode) {
                hipLaunchKernelGGL(QG_PROJ(k_project_many, C, mode()), dim3(grid8(tiles)), dim3(C::NT), 0, stream, plan_dev,
                                   first, cnt, tiles);
                return check_launch();
            });
        });
        if (e) return e;
    }
    return QG_OK;
}

int launch_backproject_many(const PlanHeader* plan_host, const PlanHeader* plan_dev, float alpha, float lr,
                            uint64_t seed, int64_t step, hipStream_t stream) {
    for (int cls = 0; cls < kPlanClasses; ++cls) {
        const int cnt = class_count(plan_host, cls), first = class_first(plan_host, cls);
        const uint32_t tiles = plan_host->bp_tiles[cls];
        if (cnt == 0 || tiles == 0) continue;
        const int e = with_bp((int)plan_host->bp_cfg[cls], [&](auto c) {
            using C = decltype(c);
            return with_mode(cls, [&](auto mode) {
                constexpr int MODE = mode();
                const dim3 grid(grid8(tiles)), block(C::NT);
                if (plan_host->zero_points)
                    hipLaunchKernelGGL((k_backproject_many<C::BM, C::BK, C::WGn, C::WGm, stages(MODE, C::NS), MODE, C::kWg[MODE], true>),
                                       grid, block, 0, stream, plan_dev, first, cnt, tiles, alpha, lr, seed, (uint64_t)step);
                else
                    hipLaunchKernelGGL((k_backproject_many<C::BM, C::BK, C::WGn, C::WGm, stages(MODE, C::NS), MODE, C::kWg[MODE]>),
                                       grid, block, 0, stream, plan_dev, first, cnt, tiles, alpha, lr, seed, (uint64_t)step);
                return check_launch();
            });
        });
        if (e) return e;
    }
    return QG_OK;
}

}  // namespace qg
