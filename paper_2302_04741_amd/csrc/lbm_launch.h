// Launcher templates: included by the per-lattice translation units, which
// instantiate them explicitly.
#pragma once

#include <algorithm>

#include "lbm_kernels.h"

namespace lbm {

// Launch shapes of the kernels off the step path, over the row wavefronts; lds limits
// the blocks of a CU as in step_shape.
struct FieldShape {
    dim3 grid, block;
    unsigned lds;
};
inline FieldShape field_shape(const GridDims &gd, unsigned threads, unsigned lds)
{
    const int64_t waves = ((int64_t(gd.nx) + 63) / 64) * gd.ny * gd.nz, wpb = threads / 64;
    return FieldShape{dim3(unsigned((waves + wpb - 1) / wpb)), dim3(threads), lds};
}
// The LDS a block asks for so that `blocks` of them share a CU: a third of the LDS does
// not fit three times once it is rounded up, so the request is rounded down (to 4 KiB).
inline unsigned lds_for_blocks(unsigned blocks) { return STEP_LDS_PER_CU / blocks / 4096u * 4096u; }
// Reading kernels: 256 threads; the FP32 moments of large grids 8 wavefronts a CU (us,
// against 12 and unlimited: D3Q39 160^3 152 / 152 / 155, 200^3 317 / 323 / 332, 256^3 611 /
// 601 / 620, D2Q37 3001x2999 309 / 315 / 320; FP64 and F16 within 2% either way).
template <int LAT, class S> inline FieldShape moments_shape(const GridDims &gd)
{
    const bool large = sizeof(S) == 4 && buffer_lines_bytes<LAT, S>(gd) >= STEP_LARGE_BYTES;
    return field_shape(gd, 256, large ? lds_for_blocks(2) : 0u);
}
// Scattering kernels (their shifted rows' lines are completed by neighbouring
// wavefronts, in the L2 of one XCD if one block holds the whole row): whole rows
// while 8 wavefronts do (4 on small grids), and on large grids few enough blocks
// that the lines are complete before they leave the L2: as many whole blocks as 12
// wavefronts a CU allow, 16 in F16 (rows of 5 wavefronts run 10 and 15, of 7, 7 and 14,
// of 8 and more, 8 and 16).  us, against 256 threads: D3Q39 FP32 160^3 159 / 211, 256^3
// 589 / 675; FP64 129x95x110 150 / 156, D2Q37 1537x1021 129 / 137; F16 256^3 375 / 416.
// F16 rows of 5 wavefronts, 15 a CU against 10: 320x256x200 385 / 402, the rebuild 538 /
// 605, 300x256x256 620 / 618, 821 / 849.
template <int LAT, class S> inline FieldShape scatter_shape(const GridDims &gd)
{
    const unsigned k = unsigned((gd.nx + 63) / 64);  // wavefronts a row
    const unsigned most = int64_t(k) * gd.ny * gd.nz <= 4096 ? 4u : 8u;
    const unsigned w = k <= most ? k * (most / k) : most;
    const bool large = buffer_lines_bytes<LAT, S>(gd) >= STEP_LARGE_BYTES;
    const unsigned per_cu = (sizeof(S) == 2 ? 16u : 12u) / w;
    return field_shape(gd, 64 * w, large ? lds_for_blocks(per_cu) : 0u);
}

template <int LAT, class F> hipError_t with_eq_fo(int eq, int fo, F &&f)
{
    hipError_t r = hipErrorInvalidValue;
    static_for<2, Lattice<LAT>::MAXEQ + 1>([&](auto E) {
        static_for<1, 5>([&](auto O) {
            if (eq == decltype(E)::value && fo == decltype(O)::value) r = f(E, O);
        });
    });
    return r;
}

// f(policy constant) for a runtime policy (STREAM_NT serves D3Q39 FP64 only)
template <int LAT, class S, class F> hipError_t with_policy(Policy p, F &&f)
{
    if (p == Policy::RESIDENT) return f(std::integral_constant<Policy, Policy::RESIDENT>{});
    if constexpr (LAT == 1 && sizeof(S) == 8) {
        if (p == Policy::STREAM_NT) return f(std::integral_constant<Policy, Policy::STREAM_NT>{});
    }
    return f(std::integral_constant<Policy, Policy::STREAM>{});
}
// The same for the kernels with plates, whose larger grids stream every store: K1c in one
// direction (channels are small), the plated batch kernel in both, as the periodic one.
template <class F> hipError_t with_wall_policy(Policy p, F &&f)
{
    if (p == Policy::RESIDENT) return f(std::integral_constant<Policy, Policy::RESIDENT>{});
    return f(std::integral_constant<Policy, Policy::STREAM>{});
}

// f(std::bool_constant) for a handle with plates or without
template <class F> hipError_t with_walls(const WallDesc &wd, F &&f)
{
    return wd.on ? f(std::true_type{}) : f(std::false_type{});
}

template <int LAT, class S>
hipError_t launch_step_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                          const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc)
{
    // blocks of bx/64 wavefronts, one wavefront per 64 cells of a row
    const int64_t waves = ((int64_t(gd.nx) + 63) / 64) * gd.ny * gd.nz;
    const int64_t bytes = buffer_lines_bytes<LAT, S>(gd);
    const StepShape sh = step_shape<LAT, S>(bytes, waves, lc.block);
    const StepPolicy sp = step_policy<LAT, S>(bytes);
    const int64_t wpb = sh.threads / 64;
    const dim3 grid(unsigned((waves + wpb - 1) / wpb));
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        return with_policy<LAT, S>(sp.policy, [&](auto P) {
            hipLaunchKernelGGL((step_kernel<LAT, S, decltype(E)::value, decltype(O)::value,
                                            decltype(P)::value>),
                               grid, dim3(sh.threads), sh.lds, lc.stream,
                               static_cast<const S *>(A), static_cast<S *>(B), gd, fd, co, lc.ctr,
                               sweep_of(sp, grid.x, lc.cur));
            return hipGetLastError();
        });
    });
}

template <int LAT, class S>
hipError_t launch_pattern_ls(const void *A, void *B, const GridDims &gd, const LaunchCfg &lc)
{
    // the launch shape of the step (blocks of bx/64 row wavefronts)
    const int64_t waves = ((int64_t(gd.nx) + 63) / 64) * gd.ny * gd.nz;
    const int64_t bytes = buffer_lines_bytes<LAT, S>(gd);
    const StepShape sh = step_shape<LAT, S>(bytes, waves, lc.block);
    const int64_t wpb = sh.threads / 64;
    return with_policy<LAT, S>(step_policy<LAT, S>(bytes).policy, [&](auto P) {
        hipLaunchKernelGGL((pattern_kernel<LAT, S, decltype(P)::value>),
                           dim3(unsigned((waves + wpb - 1) / wpb)), dim3(sh.threads), sh.lds,
                           lc.stream, static_cast<const S *>(A), static_cast<S *>(B), gd);
        return hipGetLastError();
    });
}

// Default block of the multi-grid step: 128 threads.  64 / 128 / 256: 17.8k / 19.1k / 19.7k
// MLUPS on 64 grids of 64^2 to 1024^2 FP32, 17.4k / 18.3k / 19.1k on 64 of 32^2 to 256^2.
// FP64 lists of 449 to 704 tiles: 256, four wavefronts of a block on the four SIMDs of a CU
// and at most one block a CU (us a step, against 128: 456 tiles 6.1 / 6.8, 510 7.7 / 8.1, 538
// 8.2 / 8.8, 598 8.5 / 9.4, 640 8.1 / 8.3, 704 8.3 / 8.8; 448 tiles 7.0 / 6.8, 760 9.9 / 9.9,
// 860 9.5 / 9.0).
template <class S> inline int multi_step_threads(int64_t tiles)
{
    return sizeof(S) == 8 && tiles > 448 && tiles <= 704 ? 256 : 128;
}

template <int LAT, class S>
hipError_t launch_multi_step_ls(int eq, int fo, const BatchLaunch &bl)
{
    if (bl.ntiles <= 0) return hipSuccess;
    const int threads = bl.threads > 0    ? bl.threads
                        : bl.blocks > 0 ? 128
                                        : multi_step_threads<S>(bl.ntiles);
    // one wavefront per tile, or the persistent grid; the kernel strides over
    // the list, so a grid capped at 2^31 - 1 blocks still covers every tile
    const int64_t wpb = threads / 64;
    const int64_t need = (bl.ntiles + wpb - 1) / wpb;
    int64_t grid = bl.blocks > 0 ? std::min(bl.blocks, need) : need;
    grid = std::min<int64_t>(grid, 0x7fffffff);
    const StepPolicy sp = step_policy<LAT, S>(bl.bytes);
    const Sweep sw = sweep_of(sp, bl.ntiles, bl.parity, bl.tile0);
    // FP32 batches of 1 GiB a buffer and more: 8 wavefronts a CU, as in the step (us a
    // step, 128 threads, limited against not: 64 grids of 64^2-1024^2, 3.1 GB, 1155 /
    // 1168, 32 of them, 1.4 GB, 519 / 526, four D3Q39 128^3 476 / 503; 16 grids, 974 MB,
    // 370 / 366: the last round of blocks counts there)
    const bool limit = sizeof(S) == 4 && bl.blocks <= 0 && bl.bytes >= 1024 * MIB;
    const unsigned lds = limit ? STEP_LDS_PER_CU * unsigned(threads) / 512u : 0u;
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        constexpr int EQ = decltype(E)::value, FO = decltype(O)::value;
        if (bl.walls)
            return with_wall_policy(sp.policy, [&](auto P) {
                hipLaunchKernelGGL((multi_step_kernel<LAT, S, EQ, FO, decltype(P)::value, true>),
                                   dim3(unsigned(grid)), dim3(unsigned(threads)), 0, bl.stream,
                                   bl.begin, bl.table, bl.nsims, bl.ntiles, sw);
                return hipGetLastError();
            });
        return with_policy<LAT, S>(sp.policy, [&](auto P) {
            hipLaunchKernelGGL((multi_step_kernel<LAT, S, EQ, FO, decltype(P)::value, false>),
                               dim3(unsigned(grid)), dim3(unsigned(threads)), lds, bl.stream,
                               bl.begin, bl.table, bl.nsims, bl.ntiles, sw);
            return hipGetLastError();
        });
    });
}

template <int LAT, class S>
hipError_t launch_init_ls(int eq, int fo, const double *rho, const double *u, const double *theta,
                          void *A, const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                          const LaunchCfg &lc)
{
    const FieldShape sh = scatter_shape<LAT, S>(gd);
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        return with_walls(lc.walls, [&](auto W) {
            hipLaunchKernelGGL((init_kernel<LAT, S, decltype(E)::value, decltype(O)::value,
                                            decltype(W)::value>),
                               sh.grid, sh.block, sh.lds, lc.stream, rho, u, theta,
                               static_cast<S *>(A), gd, fd, co);
            return hipGetLastError();
        });
    });
}

template <int LAT, class S>
hipError_t launch_rebuild_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                             const ForceDesc &old_force, const ForceDesc &force,
                             const StepCoef &co, const LaunchCfg &lc)
{
    const FieldShape sh = scatter_shape<LAT, S>(gd);
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        hipLaunchKernelGGL((rebuild_kernel<LAT, S, decltype(E)::value, decltype(O)::value>),
                           sh.grid, sh.block, sh.lds, lc.stream, static_cast<const S *>(A),
                           static_cast<S *>(B), gd, old_force, force, co, lc.ctr, lc.cur);
        return hipGetLastError();
    });
}

template <int LAT, class S>
hipError_t launch_moments_ls(const void *A, double *rho, double *u, double *theta,
                             const GridDims &gd, const ForceDesc &fd, const StepCoef &co,
                             const LaunchCfg &lc)
{
    const FieldShape sh = moments_shape<LAT, S>(gd);
    return with_walls(lc.walls, [&](auto W) {
        hipLaunchKernelGGL((moments_kernel<LAT, S, decltype(W)::value>), sh.grid, sh.block, sh.lds,
                           lc.stream, static_cast<const S *>(A), rho, u,
                           theta, gd, fd, co, lc.walls);
        return hipGetLastError();
    });
}

template <int LAT, class S>
hipError_t launch_heat_flux_ls(int eq, int fo, const void *A, double *q, const GridDims &gd,
                               const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc)
{
    const FieldShape sh = field_shape(gd, 256, 0);
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        return with_walls(lc.walls, [&](auto W) {
            hipLaunchKernelGGL((heatflux_kernel<LAT, S, decltype(E)::value, decltype(O)::value,
                                                decltype(W)::value>),
                               sh.grid, sh.block, sh.lds, lc.stream,
                               static_cast<const S *>(A), q, gd, fd, co, lc.walls);
            return hipGetLastError();
        });
    });
}

template <int LAT, class S>
hipError_t launch_wall_step_ls(int eq, int fo, const void *A, void *B, const GridDims &gd,
                               const ForceDesc &fd, const StepCoef &co, const LaunchCfg &lc)
{
    // the work split of the periodic step (blocks of bx/64 row wavefronts)
    const int64_t waves = ((int64_t(gd.nx) + 63) / 64) * gd.ny * gd.nz;
    const int64_t bytes = buffer_lines_bytes<LAT, S>(gd);
    const StepShape sh = step_shape<LAT, S>(bytes, waves, lc.block);
    const int64_t wpb = sh.threads / 64;
    const dim3 grid(unsigned((waves + wpb - 1) / wpb));
    return with_eq_fo<LAT>(eq, fo, [&](auto E, auto O) {
        return with_wall_policy(step_policy<LAT, S>(bytes).policy, [&](auto P) {
            hipLaunchKernelGGL((wall_step_kernel<LAT, S, decltype(E)::value, decltype(O)::value,
                                                 decltype(P)::value>),
                               grid, dim3(sh.threads), sh.lds, lc.stream,
                               static_cast<const S *>(A), static_cast<S *>(B), gd, fd, co,
                               lc.walls, lc.ctr, lc.cur);
            return hipGetLastError();
        });
    });
}

template <int LAT>
hipError_t launch_wall_setup_l(int eq, const double *theta, const double *uw, int64_t ny,
                               double *e, hipStream_t stream)
{
    hipError_t r = hipErrorInvalidValue;
    static_for<2, Lattice<LAT>::MAXEQ + 1>([&](auto E) {
        if (eq == decltype(E)::value) {
            hipLaunchKernelGGL((wall_setup_kernel<LAT, decltype(E)::value>), dim3(1), dim3(64), 0,
                               stream, theta[0], theta[1], uw[0], uw[1], ny, e);
            r = hipGetLastError();
        }
    });
    return r;
}

template <int LAT>
hipError_t launch_wall_mass_l(int storage, const void *A, const GridDims &gd, const StepCoef &co,
                              const LaunchCfg &lc)
{
    const int64_t ncol = int64_t(gd.nx) * gd.nz;
    const dim3 grid(unsigned((ncol + 255) / 256)), block(256);
    if (storage == 0)
        hipLaunchKernelGGL((wall_mass_kernel<LAT, double>), grid, block, 0, lc.stream,
                           static_cast<const double *>(A), gd, co, lc.walls);
    else if (storage == 1)
        hipLaunchKernelGGL((wall_mass_kernel<LAT, float>), grid, block, 0, lc.stream,
                           static_cast<const float *>(A), gd, co, lc.walls);
    else
        hipLaunchKernelGGL((wall_mass_kernel<LAT, __half>), grid, block, 0, lc.stream,
                           static_cast<const __half *>(A), gd, co, lc.walls);
    return hipGetLastError();
}

template <int LAT>
hipError_t launch_totals_l(int storage, const void *A, double *partials, double *out_dev,
                           const GridDims &gd, const StepCoef &co, hipStream_t stream)
{
    const DivU32 by_nx = make_divu32(uint32_t(gd.nx));
    if (storage == 0)
        hipLaunchKernelGGL((totals_stage1<LAT, double>), dim3(TOTALS_BLOCKS), dim3(256), 0, stream,
                           static_cast<const double *>(A), partials, gd, by_nx);
    else if (storage == 1)
        hipLaunchKernelGGL((totals_stage1<LAT, float>), dim3(TOTALS_BLOCKS), dim3(256), 0, stream,
                           static_cast<const float *>(A), partials, gd, by_nx);
    else
        hipLaunchKernelGGL((totals_stage1<LAT, __half>), dim3(TOTALS_BLOCKS), dim3(256), 0, stream,
                           static_cast<const __half *>(A), partials, gd, by_nx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((totals_stage2<LAT>), dim3(1), dim3(1024), 0, stream, partials, out_dev,
                       gd, co);
    return hipGetLastError();
}

}  // namespace lbm
