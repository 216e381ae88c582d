// The 1D IDIC step after the histogram in two launches: a scatter of whole
// records into cell ranges, and one kernel that orders, sums, solves and moves.
//
// What bounds it: 1D steps are memory and latency bound (10 window candidates a
// particle).  As separate launches (rank + gather, density, force, update) every
// particle's fields went through memory four times, 240 bytes a particle and
// step, and each launch waited on its own chain of dependent loads.  Here a
// workgroup owns a run of cells and loads them with 2 W cells on either side (W
// the window): it ranks the particles by id in LDS, computes the density of its
// cells and W halo cells, the force and predictor of its own cells, their drag
// solve, and writes the moved particles: 76 bytes a particle, and the halo of 8
// cells costs 6% of a run of 128.  The neighbour loops read LDS.  us a step,
// separate -> fused, FP32: 5000 + 5000 particles 29 -> 21, 1e6 + 1e6 114 -> 77;
// 256 uneven waves (5.4M particles, flattened batch) 292 -> 182.
//
// Everything is computed by the device functions of the separate launches on a
// local copy of the grid (cells renumbered, neighbour order kept), so results
// are bitwise theirs.  Runs are cut by particles (line_cut()).  A run whose particles
// do not fit the LDS of the launch, or that holds a crowded cell, works in the global
// workspace instead, with wider loops; runs share halo particles there, and
// write equal values for them.
#pragma once

#include <algorithm>

#include "binning.hpp"
#include "sph.hpp"

namespace tfsph {

// waves per SIMD of the FP32 kernels: six spill (256 uneven waves 0.215 ms a step against 0.189)
constexpr int kLineWaves = 5;

template <typename R> struct V2;
template <> struct V2<float> { using T = float2; };
template <> struct V2<double> { using T = double2; };

// Record of a particle on its way into its cell range: (off, vel), with
// per-particle masses (off, vel, m, 0).
template <typename R>
__device__ __forceinline__ void line_scatter_one(const Geom<R> &G, const Phase<R> &P, const Sorted<R> &S, int i)
{
    const int c = safe_cell(P.cell[i], G.ncell);
    const int slot = S.slot[i], id = P.id[i];
    const R o = P.off[0][i], v = P.vel[0][i];
    const int pos = S.start[c] + slot;
    S.tmp_id[pos] = id;
    if (S.has_mass) {
        reinterpret_cast<R4<R> *>(S.rec)[pos] = mk4<R>(o, v, P.mass[i], R(0));
    } else {
        typename V2<R>::T q;
        q.x = o;
        q.y = v;
        reinterpret_cast<typename V2<R>::T *>(S.rec)[pos] = q;
    }
}

template <typename R>
__device__ __forceinline__ R4<R> line_record(const Phase<R> &P, const Sorted<R> &S, int pos)
{
    if (S.has_mass) return reinterpret_cast<const R4<R> *>(S.rec)[pos];
    const typename V2<R>::T q = reinterpret_cast<const typename V2<R>::T *>(S.rec)[pos];
    return mk4<R>(q.x, q.y, P.m_uniform, R(0));
}

// The runs of cells of the workgroups: run k of n_runs holds the cells runs[k] .. runs[k + 1] - 1.
// They are cut by particles, so that crowded cells do not make one workgroup's serial work
// of a share of the problem: key(c) counts the gas before cell c three times (two neighbour
// loops), the dust once and the cells line_cell_weight() times (which bounds the cells of a
// run), width is the average key of a run, and cell c belongs to run (key(c) + key(c + 1)) / 2
// / width: a cell of more than two widths has a run to itself, and the runs that it spans
// are empty.  us a step, runs of equal cells -> these (separate launches), 1e5 + 1e5
// particles, 2 of a phase per cell: even 27 -> 29 (38); 90% of the dust in a tenth of the box 71 ->
// 41 (55); 90% of both 330 -> 75 (97); 95% in a fiftieth 4889 -> 285 (310); 5000 dust particles
// in a cell 7298 -> 439 (550); 300 gas particles in a cell 273 -> 225 (202), 1000 1361 -> 765 (620): the
// neighbour loops of a cell stay one workgroup's, which is the limit of this form.
__host__ __device__ inline unsigned line_cell_weight(int ng, int nd, int ncell)
{
    const unsigned w = (3u * unsigned(ng) + unsigned(nd)) / 4u / unsigned(ncell);
    return w < 1u ? 1u : w;
}

__host__ __device__ inline unsigned line_run_width(int ng, int nd, int ncell, int n_runs)
{
    return (3u * unsigned(ng) + unsigned(nd) + line_cell_weight(ng, nd, ncell) * unsigned(ncell)) / unsigned(n_runs) + 1u;
}

// the runs that start at the cells first, first + stride, ... (one past the last cell included)
template <typename R>
__device__ __forceinline__ void line_cut(const Geom<R> &G, const Sorted<R> &Sg, const Sorted<R> &Sd, int n_runs, int first,
                                         int stride)
{
    const unsigned w = line_cell_weight(Sg.n, Sd.n, G.ncell), width = line_run_width(Sg.n, Sd.n, G.ncell, n_runs);
    auto key = [&](int c) { return 3u * unsigned(Sg.start[c]) + unsigned(Sd.start[c]) + w * unsigned(c); };
    auto run_of = [&](int c) { return int((key(c) + key(c + 1)) / 2u / width); };
    for (int c = first; c <= G.ncell; c += stride) {
        const int last = c < G.ncell ? run_of(c) : n_runs;
        for (int k = c > 0 ? run_of(c - 1) + 1 : 0; k <= last; ++k) Sg.runs[k] = c;
    }
}

template <typename R>
__global__ void __launch_bounds__(kBlock)
k_line_scatter(Geom<R> G, Phase<R> Pg, Sorted<R> Sg, Phase<R> Pd, Sorted<R> Sd, int blocks_g, int clear, int n_runs)
{
    clear_counts(clear ? Sg.count : nullptr, Sd.count, G.ncell);
    const bool gas = int(blockIdx.x) < blocks_g;
    const int i = (gas ? blockIdx.x : blockIdx.x - blocks_g) * kBlock + threadIdx.x;
    if (gas) {
        if (i < Sg.n) line_scatter_one(G, Pg, Sg, i);
    } else {
        if (i < Sd.n) line_scatter_one(G, Pd, Sd, i);
    }
    line_cut(G, Sg, Sd, n_runs, blockIdx.x * kBlock + threadIdx.x, gridDim.x * kBlock);
}

// LDS of a run of `own` cells with ng gas particles (halo included) and nd dust
// particles; with base set, the local views.  The gas id scratch shares the
// predictor's bytes, the dust id scratch and the cell solves the force records';
// dust offsets and (per-particle) masses stand alone, no loop reads dust records.
template <typename R>
__host__ __device__ inline size_t line_carve(unsigned char *base, int own, int halo, int ng, int nd, bool mass_d, Sorted<R> &Lg,
                                             Sorted<R> &Ld, R *&off_d, R *&m_d, CellSolve<R> *&cs)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char *p = base + off;
        off += (bytes + 15) / 16 * 16;
        return p;
    };
    size_t most = sizeof(R4<R>) * (ng + kPad);
    if (most < sizeof(CellSolve<R>) * own) most = sizeof(CellSolve<R>) * own;
    if (most < sizeof(int) * nd) most = sizeof(int) * nd;
    unsigned char *shared = take(most);
    Lg.frc = reinterpret_cast<R4<R> *>(shared);
    cs = reinterpret_cast<CellSolve<R> *>(shared);
    Lg.pos = reinterpret_cast<R4<R> *>(take(sizeof(R4<R>) * (ng + kPad)));
    off_d = reinterpret_cast<R *>(take(sizeof(R) * nd));
    m_d = mass_d ? reinterpret_cast<R *>(take(sizeof(R) * nd)) : nullptr;
    Lg.vel[0] = reinterpret_cast<R *>(take(sizeof(R) * ng));
    Lg.vt[0] = reinterpret_cast<R *>(take(sizeof(R) * ng));
    Lg.tmp_id = reinterpret_cast<int *>(Lg.vt[0]);
    Lg.rho = reinterpret_cast<R *>(take(sizeof(R) * ng));
    Lg.id = reinterpret_cast<int *>(take(sizeof(int) * ng));
    Lg.cell = reinterpret_cast<int *>(take(sizeof(int) * ng));
    Lg.energy = nullptr;
    Lg.nmask = nullptr;
    Lg.start = reinterpret_cast<int *>(take(sizeof(int) * (own + 2 * halo + 1)));
    Ld.vel[0] = reinterpret_cast<R *>(take(sizeof(R) * nd));
    Ld.tmp_id = reinterpret_cast<int *>(shared);
    Ld.id = reinterpret_cast<int *>(take(sizeof(int) * nd));
    Ld.cell = reinterpret_cast<int *>(take(sizeof(int) * nd));
    Ld.start = reinterpret_cast<int *>(take(sizeof(int) * (own + 1))) - halo;    // indexed like the gas cells
    Lg.n = ng;
    Ld.n = nd;
    Ld.energy = nullptr;
    Ld.nmask = nullptr;
    Ld.frc = nullptr;
    return off;
}

// first sorted index of cell u, for u up to one period outside the box of nc cells
template <typename R>
__device__ __forceinline__ int line_first(const Sorted<R> &S, int nc, int u)
{
    return u < 0 ? S.start[u + nc] - S.n : (u >= nc ? S.start[u - nc] + S.n : S.start[u]);
}

// The dust of a crowded cell c to its sorted places, by the whole workgroup: ids into kBlock
// equal ranges of their values, then ranks inside a range, so that the ranks of n particles
// take about n^2 / 256 comparisons (5000 in a cell: a step of 3.67 ms -> 0.43).  lds: kBucketInts.  Uses
// the cell's range of slot and tmp_idx.
constexpr int kBucketCell = 512;         // more particles than this go through ranges
constexpr int kBucketInts = 2 * kBlock + kBlock / 64 + 2;
template <typename R>
__device__ __forceinline__ void line_place_buckets(const Phase<R> &P, const Sorted<R> &S, int c, int *lds, unsigned int *flags)
{
    int *begin = lds, *at = lds + kBlock, *range = at + kBlock, *waves = range + 2;
    const int tid = threadIdx.x, b = S.start[c], e = S.start[c + 1];
    __syncthreads();                     // the last cell's lists are done with
    if (tid == 0) {
        range[0] = 0x7fffffff;
        range[1] = -0x7fffffff - 1;
    }
    begin[tid] = 0;
    __syncthreads();
    int lo = 0x7fffffff, hi = -0x7fffffff - 1;
    for (int k = b + tid; k < e; k += kBlock) {
        lo = min(lo, S.tmp_id[k]);
        hi = max(hi, S.tmp_id[k]);
    }
    atomicMin(&range[0], lo);
    atomicMax(&range[1], hi);
    __syncthreads();
    const unsigned first = range[0], width = (unsigned(range[1]) - first) / kBlock + 1;
    auto bucket = [&](int id) { return int((unsigned(id) - first) / width); };
    for (int k = b + tid; k < e; k += kBlock) atomicAdd(&begin[bucket(S.tmp_id[k])], 1);
    __syncthreads();
    int total;
    const int ex = block_exclusive_scan(begin[tid], waves, total);
    begin[tid] = at[tid] = b + ex;
    __syncthreads();
    for (int k = b + tid; k < e; k += kBlock) {
        const int id = S.tmp_id[k];
        const int p = atomicAdd(&at[bucket(id)], 1);
        S.slot[p] = id;
        S.tmp_idx[p] = k;
    }
    __syncthreads();
    for (int p = b + tid; p < e; p += kBlock) {
        const int id = S.slot[p], j = bucket(id);
        const R4<R> q = line_record(P, S, S.tmp_idx[p]);
        const int dst = rank_in_cell(S.slot, begin[j], at[j], id, p, flags);
        S.id[dst] = id;
        S.cell[dst] = c;
        S.pos[dst] = mk4<R>(q.x, R(0), R(0), q.z);
        S.vel[0][dst] = q.y;
    }
}

// The run of cells [c0, c1) of a workgroup.
template <typename R, int KIND>
__device__ __forceinline__ void line_run(const Geom<R> &G, const Phys<R> &Ph, const Sorted<R> &Sg, const Sorted<R> &Sd,
                                         const Phase<R> &Pg, const Phase<R> &Pd, const Flags &F, int c0, int c1,
                                         size_t lds_bytes, bool claim, unsigned char *smem, int &bad, int &one, R &s2)
{
    const int tid = threadIdx.x;
    const int W = G.win[0], H = 2 * W, own = c1 - c0, nl = own + 2 * H, nc = G.nc[0], n = Sg.n;
    auto first_of = [&](int u) { return line_first(Sg, nc, u); };
    const int base = first_of(c0 - H), ng = first_of(c1 + H) - base;
    auto slot_of = [&](int l) {          // global slot of the run's l-th gas slot
        const int t = base + l;
        return t < 0 ? t + n : (t >= n ? t - n : t);
    };
    const int ga = Sg.start[c0], n_own = Sg.start[c1] - ga;
    const int da = Sd.start[c0], nd = Sd.start[c1] - da;
    Sorted<R> Lg{}, Ld{};
    CellSolve<R> *cs;
    R *off_d, *m_d;
    __shared__ int s_long;               // a cell that the loops of the global workspace serve better
    bool local = line_carve<R>(smem, own, H, ng, nd, Sd.has_mass != 0, Lg, Ld, off_d, m_d, cs) <= lds_bytes;
    if (local && (nd > kBucketCell || ng > 2 * kBlock)) {
        if (tid == 0) s_long = 0;
        __syncthreads();
        for (int c = tid - H; c < own + H; c += kBlock) {
            const bool gas = first_of(c0 + c + 1) - first_of(c0 + c) > kBlock;
            if (gas || (c >= 0 && c < own && Sd.start[c0 + c + 1] - Sd.start[c0 + c] > kBucketCell)) s_long = 1;
        }
        __syncthreads();
        local = s_long == 0;
    }

    if (local) {
        Geom<R> Gl = G;
        Gl.nc[0] = Gl.ncell = nl;
        Lg.has_mass = Sg.has_mass;
        for (int c = tid; c <= nl; c += kBlock) Lg.start[c] = first_of(c0 - H + c) - base;
        for (int c = tid; c <= own; c += kBlock) Ld.start[H + c] = Sd.start[c0 + c] - da;
        for (int l = tid; l < ng; l += kBlock) Lg.tmp_id[l] = Sg.tmp_id[slot_of(l)];
        for (int l = tid; l < nd; l += kBlock) Ld.tmp_id[l] = Sd.tmp_id[da + l];
        // the first records of this thread: in flight while the cells are numbered
        R4<R> qg{}, qd{};
        if (tid < ng) qg = line_record(Pg, Sg, slot_of(tid));
        if (tid < nd) qd = line_record(Pd, Sd, da + tid);
        __syncthreads();
        for (int c = tid; c < nl; c += kBlock) {
            for (int k = Lg.start[c]; k < Lg.start[c + 1]; ++k) Lg.cell[k] = c;
            if (c >= H && c < nl - H)
                for (int k = Ld.start[c]; k < Ld.start[c + 1]; ++k) Ld.cell[k] = c;
        }
        __syncthreads();
        for (int l = tid; l < ng; l += kBlock) {
            const R4<R> q = l == tid ? qg : line_record(Pg, Sg, slot_of(l));
            const int c = Lg.cell[l];
            const int dst = rank_in_cell(Lg.tmp_id, Lg.start[c], Lg.start[c + 1], Lg.tmp_id[l], l, F.word);
            Lg.id[dst] = Lg.tmp_id[l];
            Lg.pos[dst] = mk4<R>(q.x, R(0), R(0), q.z);
            Lg.vel[0][dst] = q.y;
        }
        for (int l = tid; l < nd; l += kBlock) {
            const R4<R> q = l == tid ? qd : line_record(Pd, Sd, da + l);
            const int c = Ld.cell[l];
            const int dst = rank_in_cell(Ld.tmp_id, Ld.start[c], Ld.start[c + 1], Ld.tmp_id[l], l, F.word);
            Ld.id[dst] = Ld.tmp_id[l];
            off_d[dst] = q.x;
            if (m_d) m_d[dst] = q.z;
            Ld.vel[0][dst] = q.y;
        }
        // the pair loops read up to kPad records past a range: keep those past the last cell that
        // the density pass (all of them) and the force pass (those with a density) visit finite
        if (tid < kPad) Lg.pos[ng + tid] = mk4<R>(R(0), R(0), R(0), R(0));
        __syncthreads();
        if (tid < kPad) Lg.frc[Lg.start[nl - W] + tid] = mk4<R>(R(0), R(0), R(0), R(0));
        for (int a = Lg.start[W] + tid; a < Lg.start[nl - W]; a += kBlock) density_store<R, 1>(Gl, Ph, Lg, a, 1);
        __syncthreads();
        const int la = Lg.start[H];
        for (int i = tid; i < n_own; i += kBlock) gas_predict<R, 1, KIND>(Gl, Ph, Lg, Pg, la + i);
        __syncthreads();
        for (int c = tid; c < own; c += kBlock) {
            CellSums<R> sums;
            cell_sums_with<R, 1>(
                Ph, Lg.start[H + c], Lg.start[H + c + 1], Ld.start[H + c], Ld.start[H + c + 1],
                [&](int i, R &m, R *v) {
                    m = Lg.pos[i].w;
                    v[0] = Lg.vt[0][i];
                },
                [&](int i, R &m, R *u) {
                    m = m_d ? m_d[i] : Pd.m_uniform;
                    u[0] = Ld.vel[0][i];
                },
                sums);
            one += solve_from_sums<R, 1>(Ph, sums, cs[c]) ? 1 : 0;
        }
        __syncthreads();
        for (int l0 = 0; l0 < max(n_own, nd); l0 += kBlock) {     // every lane of a wave claims (shuffles)
            const int i = l0 + tid;
            int kg = -1, kd = -1;
            R v[3], o[3];
            if (i < n_own) {
                const int l = la + i, a = ga + i, c = Lg.cell[l];
                const R4<R> me = Lg.pos[l];
                const R vt[3] = {Lg.vt[0][l], R(0), R(0)};
                bad |= !gas_advance<R, 1>(G, Ph, c0 + c - H, me, vt, cs[c - H], v, o, kg, s2);
                Pg.vel[0][a] = v[0];
                Pg.off[0][a] = o[0];
                Pg.cell[a] = kg;
                Pg.id[a] = Lg.id[l];
                if (Sg.has_mass && Pg.mass) const_cast<R *>(Pg.mass)[a] = me.w;
                Pg.rho[a] = Lg.rho[l];
            }
            if (i < nd) {
                const int j = da + i, c = Ld.cell[i];
                const R4<R> me = mk4<R>(off_d[i], R(0), R(0), m_d ? m_d[i] : R(0));
                const R u[3] = {Ld.vel[0][i], R(0), R(0)};
                bad |= !dust_advance<R, 1>(G, Ph, c0 + c - H, me, u, cs[c - H], v, o, kd, s2);
                Pd.vel[0][j] = v[0];
                Pd.off[0][j] = o[0];
                Pd.cell[j] = kd;
                Pd.id[j] = Ld.id[i];
                if (Sd.has_mass && Pd.mass) const_cast<R *>(Pd.mass)[j] = me.w;
            }
            if (claim) {
                const int sg = claim_slot(Sg.count, kg);
                const int sd = claim_slot(Sd.count, kd);
                if (i < n_own) Sg.slot[ga + i] = sg;
                if (i < nd) Sd.slot[da + i] = sd;
            }
        }
    } else {
        // in the global workspace: the canonical copy of the run and its halo, then the same phases
        Sorted<R> T = Sg;
        T.nmask = nullptr;
        cs = reinterpret_cast<CellSolve<R> *>(smem);
        int *lsg = reinterpret_cast<int *>(cs + own), *lsd = lsg + nl + 1;
        for (int c = tid; c <= nl; c += kBlock) lsg[c] = first_of(c0 - H + c) - base;
        for (int c = tid; c <= own; c += kBlock) lsd[c] = Sd.start[c0 + c] - da;
        __syncthreads();
        // the cell (0 .. cells - 1) of slot l: the last one that starts at or before it
        auto cell_of = [](const int *st, int cells, int l) {
            int lo = 0, hi = cells;
            while (hi - lo > 1) {
                const int mid = (lo + hi) / 2;
                if (st[mid] <= l) lo = mid;
                else hi = mid;
            }
            return lo;
        };
        auto place = [&](const Phase<R> &P, const Sorted<R> &S, int k, int c) {
            const R4<R> q = line_record(P, S, k);
            const int dst = rank_in_cell<kWideChunk>(S.tmp_id, S.start[c], S.start[c + 1], S.tmp_id[k], k, F.word);
            S.id[dst] = S.tmp_id[k];
            S.cell[dst] = c;
            S.pos[dst] = mk4<R>(q.x, R(0), R(0), q.z);
            S.vel[0][dst] = q.y;
        };
        for (int l = tid; l < ng; l += kBlock) {
            const int u = c0 - H + cell_of(lsg, nl, l);
            place(Pg, Sg, slot_of(l), u < 0 ? u + nc : (u >= nc ? u - nc : u));
        }
        auto by_buckets = [&](int c) {
            const int n_c = lsd[c + 1] - lsd[c];
            return n_c > kBucketCell && n_c <= kMaxRankCell;
        };
        for (int l = tid; l < nd; l += kBlock) {
            const int c = cell_of(lsd, own, l);
            if (!by_buckets(c)) place(Pd, Sd, da + l, c0 + c);
        }
        for (int c = 0; c < own; ++c)
            if (by_buckets(c)) line_place_buckets(Pd, Sd, c0 + c, lsd + own + 1, F.word);
        __syncthreads();
        // (the records after a range may belong to a run that has not placed them yet: not read)
        for (int l = lsg[W] + tid; l < lsg[nl - W]; l += kBlock) density_store<R, 1, false>(G, Ph, T, slot_of(l), 1);
        __syncthreads();
        for (int i = tid; i < n_own; i += kBlock) gas_predict<R, 1, KIND, false>(G, Ph, T, Pg, ga + i);
        __syncthreads();
        for (int c = c0 + tid; c < c1; c += kBlock) one += solve_cell<R, 1>(Ph, T, Sd, c, cs[c - c0]) ? 1 : 0;
        __syncthreads();
        for (int l0 = 0; l0 < max(n_own, nd); l0 += kBlock) {
            const int i = l0 + tid;
            int kg = -1, kd = -1;
            if (i < n_own)
                bad |= !gas_finish<R, 1>(G, Ph, T, Pg, ga + i, cs[T.cell[ga + i] - c0], s2, nullptr, &kg);
            if (i < nd)
                bad |= !dust_finish<R, 1>(G, Ph, Sd, Pd, da + i, cs[Sd.cell[da + i] - c0], s2, nullptr, &kd);
            if (claim) {
                const int sg = claim_slot(Sg.count, kg);
                const int sd = claim_slot(Sd.count, kd);
                if (i < n_own) Sg.slot[ga + i] = sg;
                if (i < nd) Sd.slot[da + i] = sd;
            }
        }
    }
}

// The cells [c0, c1) of a run; none of a problem without particles, whose runs are not cut.
template <typename R>
__device__ __forceinline__ void line_cells_of(const Sorted<R> &Sg, const Sorted<R> &Sd, int run, int &c0, int &c1)
{
    const bool cut = Sg.n + Sd.n > 0;
    c0 = cut ? Sg.runs[run] : 0;
    c1 = cut ? Sg.runs[run + 1] : 0;
}

template <typename R, int KIND>
__device__ __forceinline__ void line_block(const Geom<R> &G, const Phys<R> &Ph, const Sorted<R> &Sg, const Sorted<R> &Sd,
                                           const Phase<R> &Pg, const Phase<R> &Pd, const Flags &F, int c0, int c1,
                                           size_t lds_bytes, bool claim, unsigned char *smem)
{
    __shared__ int s_bad, s_one;
    if (threadIdx.x == 0) { s_bad = 0; s_one = 0; }
    int bad = 0, one = 0;
    R s2 = signal_floor(Ph);
    if (c0 < c1)
        line_run<R, KIND>(G, Ph, Sg, Sd, Pg, Pd, F, c0, c1, lds_bytes, claim, smem, bad, one, s2);
    publish_speed(Ph, F, s2);
    if (bad) atomicOr(&s_bad, 1);
    if (one) atomicAdd(&s_one, one);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_bad) atomicOr(F.word, 1u);
        if (s_one) {
            atomicOr(F.word, 2u);
            atomicAdd(F.one_phase, (unsigned long long)s_one);
        }
    }
}

template <typename R, int KIND>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? kLineWaves : 4)))
k_line_step(Geom<R> G, Phys<R> Ph, Sorted<R> Sg, Sorted<R> Sd, Phase<R> Pg, Phase<R> Pd, Flags F, int n_runs,
            size_t lds_bytes, int claim)
{
    extern __shared__ __align__(16) unsigned char smem_line[];     // 16-byte records from the first byte on
    int c0, c1;
    line_cells_of(Sg, Sd, xcd_block(n_runs), c0, c1);
    line_block<R, KIND>(G, Ph, Sg, Sd, Pg, Pd, F, c0, c1, lds_bytes, claim != 0, smem_line);
}

// Cells of a run: with its halo one gas particle a thread on average, so no phase
// takes a second round for a few particles (half as many cells: 1e6 + 1e6 particles
// 95 us a step against 72).
inline int line_cells(int win, double per_gas)
{
    const int cells = per_gas > 0.0 ? int(kBlock / per_gas) - 4 * win : 128;
    return cells < 16 ? 16 : (cells > 256 ? 256 : cells);
}

// Gas particles a cell, on average, up to which the fused step is taken: the halo of a run is
// 4 W cells whatever they hold, so where cells hold many, most of its densities are computed
// twice.  us a step, fused / separate, FP32 1e5 + 1e5 particles: 4 a cell 33 / 44, with 90% of
// both phases in a tenth of the box 112 / 148; 10 a cell 43 / 58 and 343 / 284; 20 a cell 103 /
// 87 and 1216 / 550.  FP64 launches of more than one round of workgroups hold less: 1e6 + 1e6
// particles, 2 a cell 122 / 144 and 535 / 508, 4 a cell 145 / 170 and 1099 / 690.
constexpr double kLineGasPerCell = 4.0, kLineGasPerCellMany = 2.5;

// LDS of a launch of all_runs runs, some of them of a problem of ng + nd particles cut in n_runs:
// what lets all of them be resident at once, where that is at least 1.6 times an average run's
// need, otherwise 1.6 times it (as fast as 1.35 times; twice: 1e6 + 1e6 particles 79 -> 86 us a
// step).  0 where the step takes the separate launches: crowded averages, and problems whose
// keys (line_cut()) do not fit 31 bits.
template <typename R>
inline size_t line_lds(int64_t ng, int64_t nd, int ncell, int win, int n_runs, int64_t all_runs, bool mass_d)
{
    const double per_gas = double(ng) / ncell, per_dust = double(nd) / ncell, cells = double(ncell) / n_runs;
    if (3 * ng + nd + 2 * int64_t(ncell) >= int64_t(1) << 30) return 0;
    const double g = per_gas * (cells + 4 * win) * 1.6 + 16, d = per_dust * cells * 1.6 + 16;
    if (g + d > 1e5) return 0;
    Sorted<R> Lg{}, Ld{};
    CellSolve<R> *cs;
    R *off_d, *m_d;
    const size_t need = line_carve<R>(nullptr, int(cells) + 1, 2 * win, int(g), int(d), mass_d, Lg, Ld, off_d, m_d, cs);
    // the lists of the longest run, for one that works in global memory
    const size_t own = line_run_width((int)ng, (int)nd, ncell, n_runs) / line_cell_weight((int)ng, (int)nd, ncell) + 2;
    const size_t least = (sizeof(CellSolve<R>) + 2 * sizeof(int)) * own + (4 * win + kBucketInts) * sizeof(int) + 64;
    const int64_t per_cu = (all_runs + 255) / 256;
    // (allocated in steps of 1280 bytes; the static variables take a few of the last one)
    const size_t room = per_cu <= 5 ? size_t(128 / per_cu) * 1280 - 64 : 0;
    if (per_gas > (sizeof(R) == 8 && room == 0 ? kLineGasPerCellMany : kLineGasPerCell)) return 0;
    const size_t lds = std::max(std::max(need, least), room);
    return lds > 144 * 1024 ? (std::max(need, least) > 144 * 1024 ? 0 : 144 * 1024) : lds;
}

}  // namespace tfsph
