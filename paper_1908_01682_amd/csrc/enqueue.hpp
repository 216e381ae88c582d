// Launch sequences of one IDIC step shared by the library's entry points:
// binning (counting sort into canonical (cell, id) order), gas density, and
// the fused force + predictor + cell solve + update kernel.
#pragma once

#include "binning.hpp"
#include "host.hpp"
#include "line.hpp"
#include "sph.hpp"
#include "tiles.hpp"

namespace tfsph_host {

inline int ntiles_of(int ncell) { return (ncell + kScanTile - 1) / kScanTile; }

inline int default_cells_per_block(int dim) { return dim == 1 ? 128 : (dim == 2 ? 64 : 32); }
// upper bound of tfsph_set_cells_per_block: the block's cell solves sit in LDS
// next to the staged particle records (under 64 KiB in FP64)
constexpr int kMaxCellsPerBlock = 256;

// zero the cell counts of a phase pair: once per workspace, before its first binning
template <typename R>
inline tfsph_status enqueue_zero_counts(int ncell, Sorted<R> &Sg, Sorted<R> &Sd, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks_for(ncell)), dim3(kBlock), 0, st, Sg.count, ncell, Sd.count, ncell);
    LAUNCH_CHECK("fill_zero");
    return TFSPH_OK;
}

// slot claims of both phases from the caller's arrays (the counts must be zero)
template <typename R>
inline tfsph_status enqueue_count(int ng, int nd, int ncell, const Phase<R> &Pg, const Phase<R> &Pd, Sorted<R> &Sg,
                                  Sorted<R> &Sd, const Flags &F, hipStream_t st)
{
    const int bg = blocks_for(ng), bd = blocks_for(nd);
    if (bg + bd == 0) return TFSPH_OK;
    hipLaunchKernelGGL(k_count, dim3(bg + bd), dim3(kBlock), 0, st, Pg.cell, ng, Sg.count, Sg.slot, Pd.cell, nd,
                       Sd.count, Sd.slot, bg, ncell, F.word);
    LAUNCH_CHECK("count");
    return TFSPH_OK;
}

// whether the scan of a grid leaves the counts for the scatter to clear (k_scan_one)
inline bool scan_keeps_counts(int ncell) { return ncell <= kScanOneCells; }

// exclusive scans of both histograms into the cell offsets; the counts are zero afterwards
// or, with scan_keeps_counts(), untouched
template <typename R>
inline tfsph_status enqueue_scan(int ncell, Sorted<R> &Sg, Sorted<R> &Sd, int *partial, hipStream_t st)
{
    if (scan_keeps_counts(ncell)) {
        hipLaunchKernelGGL(k_scan_one, dim3((ncell + kScanOneTile - 1) / kScanOneTile, 2), dim3(kScanOneThreads), 0, st,
                           Sg.count, Sd.count, ncell, Sg.start, Sd.start);
        LAUNCH_CHECK("scan_one");
        return TFSPH_OK;
    }
    const int ntiles = ntiles_of(ncell);
    hipLaunchKernelGGL(k_scan_reduce, dim3(ntiles, 2), dim3(kBlock), 0, st, Sg.count, Sd.count, ncell, partial, ntiles);
    LAUNCH_CHECK("scan_reduce");
    const int inline_prefix = ntiles <= kScanInlineTiles ? 1 : 0;
    if (!inline_prefix) {
        hipLaunchKernelGGL(k_scan_top, dim3(1, 2), dim3(kBlock), 0, st, partial, ntiles, Sg.start, Sd.start, ncell);
        LAUNCH_CHECK("scan_top");
    }
    hipLaunchKernelGGL(k_scan_down, dim3(ntiles, 2), dim3(kBlock), 0, st, Sg.count, Sd.count, ncell, partial, ntiles,
                       Sg.start, Sd.start, inline_prefix);
    LAUNCH_CHECK("scan_down");
    return TFSPH_OK;
}

// Runs and LDS of the fused 1D step (line.hpp); LDS 0 where the step takes the separate launches.
// Those serve problems of fewer than kLineLeast particles a phase: all of them may crowd in a few
// cells, whose neighbour loops are one workgroup's in a run (1500 of 1500 in one cell: 1480 us a
// step fused, 538 separate; even 20 / 28).
constexpr int kLineLeast = 2048;
template <typename R>
inline size_t line_step_lds(const Geom<R> &G, int ng, int nd, bool mass_d, int &n_runs)
{
    const int cells = line_cells(G.win[0], double(ng) / G.ncell);
    n_runs = (G.ncell + cells - 1) / cells;
    if (ng < kLineLeast && nd < kLineLeast) return 0;
    return line_lds<R>(ng, nd, G.ncell, G.win[0], n_runs, n_runs, mass_d);
}

// One fused 1D step in n_runs runs and lds bytes (line_step_lds()).  claimed: the previous step claimed this one's slots;
// claim: so does this step for the next one.
template <typename R>
inline tfsph_status enqueue_line(int ng, int nd, const Geom<R> &G, const Phys<R> &Ph, const Phase<R> &Pg,
                                 const Phase<R> &Pd, Sorted<R> &Sg, Sorted<R> &Sd, int *partial, const Flags &F, int n_runs,
                                 size_t lds, bool claimed, bool claim, hipStream_t st)
{
    tfsph_status r = TFSPH_OK;
    if (!claimed) r = enqueue_count<R>(ng, nd, G.ncell, Pg, Pd, Sg, Sd, F, st);
    if (r == TFSPH_OK) r = enqueue_scan<R>(G.ncell, Sg, Sd, partial, st);
    if (r != TFSPH_OK) return r;
    const int bg = blocks_for(ng), bd = blocks_for(nd);
    if (bg + bd > 0) {
        hipLaunchKernelGGL(k_line_scatter<R>, dim3(bg + bd), dim3(kBlock), 0, st, G, Pg, Sg, Pd, Sd, bg,
                           scan_keeps_counts(G.ncell) ? 1 : 0, n_runs);
        LAUNCH_CHECK("line_scatter");
    }
    if (Sg.has_mass)
        hipLaunchKernelGGL((k_line_step<R, kForceIsoMass>), dim3(n_runs), dim3(kBlock), lds, st, G, Ph, Sg, Sd, Pg, Pd,
                           F, n_runs, lds, claim ? 1 : 0);
    else
        hipLaunchKernelGGL((k_line_step<R, kForceIsoUniform>), dim3(n_runs), dim3(kBlock), lds, st, G, Ph, Sg, Sd, Pg,
                           Pd, F, n_runs, lds, claim ? 1 : 0);
    LAUNCH_CHECK("line_step");
    return TFSPH_OK;
}

// count + scan + scatter + rank/gather of both phases into the workspace:
// counting sort of both phases into (cell, id) order.  The counts must be zero
// on entry (enqueue_zero_counts() once, then every binning leaves them zero).
template <typename R>
inline tfsph_status enqueue_bin(int ng, int nd, const Geom<R> &G, const Phase<R> &Pg, const Phase<R> &Pd,
                                Sorted<R> &Sg, Sorted<R> &Sd, int *partial, const Flags &F, hipStream_t st)
{
    const int ncell = G.ncell;
    const int bg = blocks_for(ng), bd = blocks_for(nd);
    tfsph_status r = enqueue_count<R>(ng, nd, ncell, Pg, Pd, Sg, Sd, F, st);
    if (r == TFSPH_OK) r = enqueue_scan<R>(ncell, Sg, Sd, partial, st);
    if (r != TFSPH_OK) return r;
    if (bg + bd > 0) {
        hipLaunchKernelGGL(k_scatter, dim3(bg + bd), dim3(kBlock), 0, st, Pg.cell, Pg.id, Sg.slot, Sg.start, ng,
                           Sg.tmp_idx, Sg.tmp_id, Pd.cell, Pd.id, Sd.slot, Sd.start, nd, Sd.tmp_idx, Sd.tmp_id, bg, ncell,
                           scan_keeps_counts(ncell) ? Sg.count : nullptr, Sd.count);
        LAUNCH_CHECK("scatter");
        hipLaunchKernelGGL(k_rank_gather<R>, dim3(bg + bd), dim3(kBlock), 0, st, G, Pg, Sg, Pd, Sd, bg, F.word);
        LAUNCH_CHECK("rank_gather");
    }
    return TFSPH_OK;
}


// kernel variant: 0 (auto) takes the matrix-core support test where the window
// allows it; 1 = window scans (neighbour masks when S.nmask is set)
template <typename R, int DIM>
inline tfsph_status enqueue_density(const Geom<R> &G, const Phys<R> &Ph, const Sorted<R> &S, int want_frc,
                                    hipStream_t st, int variant = 0)
{
    if (S.n == 0) return TFSPH_OK;
    if constexpr (DIM == 3) {
        if (variant == TFSPH_VARIANT_AUTO && tile_density(G, S.n, want_frc && S.nmask)) {
            hipLaunchKernelGGL((k_density_tiles<R>), dim3(blocks_for(S.n)), dim3(kBlock), 0, st, G, Ph, S, want_frc);
            LAUNCH_CHECK("density_tiles");
            return TFSPH_OK;
        }
    }
    hipLaunchKernelGGL((k_density<R, DIM>), dim3(blocks_for(S.n)), dim3(kBlock), 0, st, G, Ph, S, want_frc);
    LAUNCH_CHECK("density");
    return TFSPH_OK;
}

// Explicit gas terms and predictor v~, one thread per gas particle.  The
// pair loop has a launch of its own: a block that owns whole cells holds a
// varying number of particles, and the few past a multiple of the block size
// would take a whole extra round of the pair loop.
template <typename R, int DIM>
inline tfsph_status enqueue_force(const Geom<R> &G, const Phys<R> &Ph, const Sorted<R> &Sg, const Phase<R> &Pg,
                                  hipStream_t st)
{
    if (Sg.n == 0) return TFSPH_OK;
    const dim3 grid(blocks_for(Sg.n)), block(kBlock);
    if (Ph.av || Ph.eos != 0)
        hipLaunchKernelGGL((k_gas_predict<R, DIM, kForceGeneral>), grid, block, 0, st, G, Ph, Sg, Pg);
    else if (Sg.has_mass)
        hipLaunchKernelGGL((k_gas_predict<R, DIM, kForceIsoMass>), grid, block, 0, st, G, Ph, Sg, Pg);
    else
        hipLaunchKernelGGL((k_gas_predict<R, DIM, kForceIsoUniform>), grid, block, 0, st, G, Ph, Sg, Pg);
    LAUNCH_CHECK("gas_predict");
    return TFSPH_OK;
}

// Cell sums, implicit solve, particle update, move and carry.
template <typename R, int DIM>
inline tfsph_status enqueue_update(const Geom<R> &G, const Phys<R> &Ph, const Sorted<R> &Sg, const Sorted<R> &Sd,
                                   const Phase<R> &Pg, const Phase<R> &Pd, const Flags &F, int cpb, hipStream_t st)
{
    const int nblocks = (G.ncell + cpb - 1) / cpb;
    const size_t lds = update_lds_bytes<R>(cpb);
    hipLaunchKernelGGL((k_update<R, DIM>), dim3(nblocks), dim3(kBlock), lds, st, G, Ph, Sg, Sd, Pg, Pd, F, cpb, nblocks);
    LAUNCH_CHECK("update");
    return TFSPH_OK;
}

}  // namespace tfsph_host
