// Whole IDIC steps of one small problem inside one workgroup, with the sorted
// copy of both phases, the histograms and the cell solves in LDS.
//
// What bounds it: a problem of a few hundred particles has no work to fill the
// chip; eight launches a step cost 27 us of launch latency, and one workgroup
// on global memory waits for a cache round trip in every one of its dozen
// phases (36 us a step).  In LDS a phase costs a barrier and a few LDS
// latencies, so the step is bound by its own serial chain.  A thread keeps its
// particles (at most kSmallOwn of each phase) in registers between the steps,
// so the permutation of a step is register -> sorted LDS slot and the caller's
// arrays are read once and written once per call.  1D wave of 200 + 200 particles in
// FP64: 28 us a step in eight launches, 6.8 here.
//
// Every particle and cell goes through the device functions of the
// multi-launch step with the same neighbour order, so results are bitwise its.
#pragma once

#include "binning.hpp"
#include "sph.hpp"

namespace tfsph {

constexpr int kSmallBlock = 1024;        // most threads of the workgroup
constexpr int kSmallOwn = 2;             // particles of a phase per thread
constexpr size_t kSmallLds = 159 * 1024; // dynamic LDS of a workgroup (160 KiB per CU)

// Threads of the workgroup: one per particle of the larger phase up to 1024,
// beyond that two particles per thread on the fewest waves.
inline int small_block(int ng, int nd)
{
    int n = ng > nd ? ng : nd;
    if (n > kSmallBlock) n = (n + kSmallOwn - 1) / kSmallOwn;
    n = (n + 63) / 64 * 64;
    return n < 64 ? 64 : n;
}

// The general force loop keeps energies (also for an isothermal gas with
// viscosity, which never reads them): which arrays exist is known at compile time.
constexpr bool small_energy(int kind) { return kind != kForceIsoUniform && kind != kForceIsoMass; }

// Lay the LDS arrays out from `base` (null: count bytes only).  The id scratch
// of the binning shares the gas predictor's bytes, and the cell solves share the
// force records': each is dead before the other is written.
template <typename R, int DIM, int KIND>
__host__ __device__ inline size_t small_carve(unsigned char *base, int ng, int nd, int ncell, int mask_rows,
                                              Sorted<R> &Sg, Sorted<R> &Sd, CellSolve<R> *&cs, R *&en2)
{
    constexpr int dim = DIM;
    constexpr bool energy = small_energy(KIND);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char *p = base + off;
        off += (bytes + 15) / 16 * 16;
        return p;
    };
    Sg.n = ng;
    Sd.n = nd;
    Sg.pos = reinterpret_cast<R4<R> *>(take(sizeof(R4<R>) * (ng + kPad)));
    Sd.pos = reinterpret_cast<R4<R> *>(take(sizeof(R4<R>) * (nd + kPad)));
    const size_t frc = sizeof(R4<R>) * (ng + kPad), sol = sizeof(CellSolve<R>) * ncell;
    unsigned char *shared = take(frc > sol ? frc : sol);
    Sg.frc = reinterpret_cast<R4<R> *>(shared);
    cs = reinterpret_cast<CellSolve<R> *>(shared);
    Sd.frc = nullptr;
    for (int d = 0; d < 3; ++d) {
        Sg.vel[d] = d < dim ? reinterpret_cast<R *>(take(sizeof(R) * ng)) : nullptr;
        Sg.vt[d] = d < dim ? reinterpret_cast<R *>(take(sizeof(R) * ng)) : nullptr;
        Sd.vel[d] = d < dim ? reinterpret_cast<R *>(take(sizeof(R) * nd)) : nullptr;
        Sd.vt[d] = nullptr;
    }
    Sg.tmp_id = reinterpret_cast<int *>(Sg.vt[0]);
    Sd.tmp_id = reinterpret_cast<int *>(take(sizeof(int) * nd));
    Sg.rho = reinterpret_cast<R *>(take(sizeof(R) * ng));
    Sd.rho = nullptr;
    Sg.energy = energy ? reinterpret_cast<R *>(take(sizeof(R) * ng)) : nullptr;
    en2 = energy ? reinterpret_cast<R *>(take(sizeof(R) * ng)) : nullptr;
    Sd.energy = nullptr;
    Sg.cell = reinterpret_cast<int *>(take(sizeof(int) * ng));
    Sd.cell = reinterpret_cast<int *>(take(sizeof(int) * nd));
    Sg.id = reinterpret_cast<int *>(take(sizeof(int) * ng));
    Sd.id = reinterpret_cast<int *>(take(sizeof(int) * nd));
    Sg.nmask = DIM > 1 ? reinterpret_cast<unsigned long long *>(take(sizeof(unsigned long long) * mask_rows * ng))
                         : nullptr;
    Sd.nmask = nullptr;
    Sg.count = reinterpret_cast<int *>(take(sizeof(int) * 2 * ncell));     // gas cells, then dust cells
    Sd.count = Sg.count + ncell;
    Sg.start = reinterpret_cast<int *>(take(sizeof(int) * (ncell + 1)));
    Sd.start = reinterpret_cast<int *>(take(sizeof(int) * (ncell + 1)));
    Sg.rec = Sd.rec = nullptr;
    Sg.slot = Sd.slot = Sg.src = Sd.src = Sg.tmp_idx = Sd.tmp_idx = nullptr;
    return off;
}

// exclusive scan of one int per thread for any blockDim.x <= 1024 (wave64)
__device__ __forceinline__ int block_scan_any(int v, int *lds_waves, int &total)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = (blockDim.x + 63) >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) lds_waves[wave] = x;
    __syncthreads();
    int pre = 0;
    total = 0;
    for (int w = 0; w < nwaves; ++w) {
        const int t = lds_waves[w];
        if (w < wave) pre += t;
        total += t;
    }
    __syncthreads();
    return pre + x - v;
}

// A thread's particles of one phase between the steps.
template <typename R, int DIM>
struct SmallOwn {
    int cell[kSmallOwn], id[kSmallOwn];
    R off[kSmallOwn][DIM], vel[kSmallOwn][DIM], m[kSmallOwn], e[kSmallOwn], rho[kSmallOwn];
};

template <typename R, int DIM>
__device__ __forceinline__ void small_load(const Geom<R> &G, const Phase<R> &P, bool energy, SmallOwn<R, DIM> &O,
                                           unsigned int *bad_cell)
{
#pragma unroll
    for (int q = 0; q < kSmallOwn; ++q) {
        const int i = threadIdx.x + q * blockDim.x;
        if (i >= P.n) continue;
        const int raw = P.cell[i];
        O.cell[q] = safe_cell(raw, G.ncell);
        if (bad_cell && O.cell[q] != raw) atomicOr(bad_cell, 4u);
        O.id[q] = P.id[i];
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            O.off[q][d] = P.off[d][i];
            O.vel[q][d] = P.vel[d][i];
        }
        O.m[q] = P.mass ? P.mass[i] : P.m_uniform;
        if (energy) O.e[q] = P.energy[i];
    }
}

// Rank of each own particle by id inside its cell, then its fields to the sorted slot.
template <typename R, int DIM>
__device__ __forceinline__ void small_place(const Sorted<R> &S, const SmallOwn<R, DIM> &O)
{
#pragma unroll
    for (int q = 0; q < kSmallOwn; ++q) {
        if (int(threadIdx.x + q * blockDim.x) >= S.n) continue;
        const int b = S.start[O.cell[q]], e = S.start[O.cell[q] + 1];
        int dst = b;
        for (int k = b; k < e; ++k) dst += S.tmp_id[k] < O.id[q] ? 1 : 0;
        S.cell[dst] = O.cell[q];
        S.id[dst] = O.id[q];
        S.pos[dst] = mk4<R>(O.off[q][0], DIM > 1 ? O.off[q][DIM > 1 ? 1 : 0] : R(0), R(0), O.m[q]);
#pragma unroll
        for (int d = 0; d < DIM; ++d) S.vel[d][dst] = O.vel[q][d];
        if (S.energy) S.energy[dst] = O.e[q];
    }
}

template <typename R, int DIM>
__device__ __forceinline__ void small_store(const Sorted<R> &S, const Phase<R> &P, const SmallOwn<R, DIM> &O, bool rho,
                                            bool energy)
{
#pragma unroll
    for (int q = 0; q < kSmallOwn; ++q) {
        const int a = threadIdx.x + q * blockDim.x;
        if (a >= S.n) continue;
        P.cell[a] = O.cell[q];
        P.id[a] = O.id[q];
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            P.off[d][a] = O.off[q][d];
            P.vel[d][a] = O.vel[q][d];
        }
        if (S.has_mass && P.mass) const_cast<R *>(P.mass)[a] = O.m[q];
        if (energy) P.energy[a] = O.e[q];
        if (rho) P.rho[a] = O.rho[q];
    }
}

// n_steps steps of the problem (Pg, Pd) by the whole workgroup.  one / bad count one-phase
// cells and non-finite values, s2 is raised to the largest squared signal speed.
template <typename R, int DIM, int KIND>
__device__ __forceinline__ void small_steps(const Geom<R> &G, const Phys<R> &Ph, const Phase<R> &Pg, const Phase<R> &Pd,
                                            bool mass_g, bool mass_d, int mask_rows, int n_steps,
                                            unsigned char *smem, int *lds_waves, unsigned int *bad_cell, int &one,
                                            int &bad, R &s2)
{
    const int tid = threadIdx.x, nt = blockDim.x, ncell = G.ncell;
    Sorted<R> Sg, Sd;
    CellSolve<R> *cs;
    R *en2;
    small_carve<R, DIM, KIND>(smem, Pg.n, Pd.n, ncell, mask_rows, Sg, Sd, cs, en2);
    const bool energy = small_energy(KIND) && Ph.eos != 0;
    Sg.has_mass = mass_g;
    Sd.has_mass = mass_d;
    Phase<R> Pe = Pg;            // gas_predict() writes the new energy here
    Pe.energy = en2;
    SmallOwn<R, DIM> og, od;
    small_load<R, DIM>(G, Pg, energy, og, bad_cell);
    small_load<R, DIM>(G, Pd, false, od, bad_cell);

    for (int s = 0; s < n_steps; ++s) {
        for (int c = tid; c < 2 * ncell; c += nt) Sg.count[c] = 0;
        __syncthreads();
        int sg[kSmallOwn], sd[kSmallOwn];
#pragma unroll
        for (int q = 0; q < kSmallOwn; ++q) {
            if (tid + q * nt < Sg.n) sg[q] = atomicAdd(Sg.count + og.cell[q], 1);
            if (tid + q * nt < Sd.n) sd[q] = atomicAdd(Sd.count + od.cell[q], 1);
        }
        __syncthreads();
        {   // both histograms in one scan: the dust cells follow the gas cells, whose total is n_gas
            const int per = (2 * ncell + nt - 1) / nt;
            const int c0 = min(tid * per, 2 * ncell), c1 = min(c0 + per, 2 * ncell);
            int sum = 0, total;
            for (int c = c0; c < c1; ++c) sum += Sg.count[c];
            int ex = block_scan_any(sum, lds_waves, total);
            for (int c = c0; c < c1; ++c) {
                if (c < ncell) Sg.start[c] = ex;
                else Sd.start[c - ncell] = ex - Sg.n;
                ex += Sg.count[c];
            }
            if (tid == 0) {
                Sg.start[ncell] = Sg.n;
                Sd.start[ncell] = Sd.n;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSmallOwn; ++q) {
            if (tid + q * nt < Sg.n) Sg.tmp_id[Sg.start[og.cell[q]] + sg[q]] = og.id[q];
            if (tid + q * nt < Sd.n) Sd.tmp_id[Sd.start[od.cell[q]] + sd[q]] = od.id[q];
        }
        __syncthreads();
        small_place<R, DIM>(Sg, og);
        small_place<R, DIM>(Sd, od);
        // everything lives in LDS until the update: no register is held across the pair loops
        og = SmallOwn<R, DIM>{};
        od = SmallOwn<R, DIM>{};
        // the pair loops read up to kPad records past the end: keep them finite
        if (tid < kPad) Sg.pos[Sg.n + tid] = Sg.frc[Sg.n + tid] = Sd.pos[Sd.n + tid] = mk4<R>(R(0), R(0), R(0), R(0));
        __syncthreads();
        for (int a = tid; a < Sg.n; a += nt) density_store<R, DIM>(G, Ph, Sg, a, 1);
        __syncthreads();
        for (int a = tid; a < Sg.n; a += nt) gas_predict<R, DIM, KIND>(G, Ph, Sg, Pe, a);
        __syncthreads();
        for (int c = tid; c < ncell; c += nt) one += solve_cell<R, DIM>(Ph, Sg, Sd, c, cs[c]) ? 1 : 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSmallOwn; ++q) {
            const int a = tid + q * nt;
            R vt[3], v[3], o[3];
            if (a < Sg.n) {
                const int c = Sg.cell[a];
                const R4<R> me = Sg.pos[a];
#pragma unroll
                for (int d = 0; d < DIM; ++d) vt[d] = Sg.vt[d][a];
                bad |= !gas_advance<R, DIM>(G, Ph, c, me, vt, cs[c], v, o, og.cell[q], s2);
#pragma unroll
                for (int d = 0; d < DIM; ++d) {
                    og.off[q][d] = o[d];
                    og.vel[q][d] = v[d];
                }
                og.id[q] = Sg.id[a];
                og.m[q] = me.w;
                og.rho[q] = Sg.rho[a];
                if (energy) {
                    og.e[q] = en2[a];
                    s2 = fmax(s2, Ph.ggm1 * og.e[q]);
                }
            }
            if (a < Sd.n) {
                const int c = Sd.cell[a];
                const R4<R> me = Sd.pos[a];
#pragma unroll
                for (int d = 0; d < DIM; ++d) vt[d] = Sd.vel[d][a];
                bad |= !dust_advance<R, DIM>(G, Ph, c, me, vt, cs[c], v, o, od.cell[q], s2);
#pragma unroll
                for (int d = 0; d < DIM; ++d) {
                    od.off[q][d] = o[d];
                    od.vel[q][d] = v[d];
                }
                od.id[q] = Sd.id[a];
                od.m[q] = me.w;
            }
        }
        // the next step writes the sorted arrays again only after two more barriers
    }
    small_store<R, DIM>(Sg, Pg, og, true, energy);
    small_store<R, DIM>(Sd, Pd, od, false, false);
}

// n_steps steps of one problem: grid of one workgroup.
template <typename R, int DIM, int KIND>
__global__ void __launch_bounds__(kSmallBlock)
k_small_steps(Geom<R> G, Phys<R> Ph, Phase<R> Pg, Phase<R> Pd, int mass_g, int mass_d, int mask_rows, int n_steps,
              Flags F)
{
    extern __shared__ unsigned char smem_raw[];
    __shared__ int lds_waves[kSmallBlock / 64];
    __shared__ int s_bad, s_one;
    if (threadIdx.x == 0) { s_bad = 0; s_one = 0; }
    int bad = 0, one = 0;
    R s2 = signal_floor(Ph);
    small_steps<R, DIM, KIND>(G, Ph, Pg, Pd, mass_g != 0, mass_d != 0, mask_rows, n_steps, smem_raw, lds_waves,
                              F.word, one, bad, s2);
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

}  // namespace tfsph
