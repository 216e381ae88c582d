// Host side of the one-workgroup step (small.hpp): which problems take it, and
// its launch.
#include "../../include/tfsph.h"

#include <hip/hip_runtime.h>

#include "host.hpp"
#include "small.hpp"

using namespace tfsph;
using namespace tfsph_host;

namespace {

template <typename R, int DIM, int KIND>
size_t carve_bytes(int ng, int nd, int ncell, int mask_rows)
{
    Sorted<R> Sg{}, Sd{};
    CellSolve<R> *cs;
    R *en2;
    return small_carve<R, DIM, KIND>(nullptr, ng, nd, ncell, mask_rows, Sg, Sd, cs, en2);
}

template <typename R, int DIM, int KIND>
tfsph_status launch(const tfsph_params *p, const tfsph_state *s, size_t lds, int n_steps, const Flags &F, hipStream_t st)
{
    const Geom<R> G = make_geom<R>(p);
    const Phys<R> Ph = make_phys<R>(p);
    const Phase<R> Pg = make_phase<R>(s->gas, DIM), Pd = make_phase<R>(s->dust, DIM);
    hipLaunchKernelGGL((k_small_steps<R, DIM, KIND>), dim3(1), dim3(small_block(Pg.n, Pd.n)), lds, st, G, Ph, Pg, Pd,
                       s->gas.mass != nullptr, s->dust.mass != nullptr, mask_rows_of(p), n_steps, F);
    LAUNCH_CHECK("small_steps");
    return TFSPH_OK;
}

// f(real type, dimension, force-loop kind) of a problem with dim <= 2
template <typename Fn>
auto with_types(const tfsph_params *p, bool gas_mass, Fn &&f)
{
    const int kind = (p->eos != TFSPH_ISOTHERMAL || p->av_alpha != 0.0 || p->av_beta != 0.0)
                         ? kForceGeneral
                         : (gas_mass ? kForceIsoMass : kForceIsoUniform);
    auto by_kind = [&](auto r, auto dim) {
        switch (kind) {
        case kForceGeneral: return f(r, dim, IntC<kForceGeneral>{});
        case kForceIsoMass: return f(r, dim, IntC<kForceIsoMass>{});
        default: return f(r, dim, IntC<kForceIsoUniform>{});
        }
    };
    if (p->precision == TFSPH_F64) return p->dim == 1 ? by_kind(0.0, IntC<1>{}) : by_kind(0.0, IntC<2>{});
    return p->dim == 1 ? by_kind(0.0f, IntC<1>{}) : by_kind(0.0f, IntC<2>{});
}

}  // namespace

size_t tfsph_host::small_step_lds(const tfsph_params *p, const tfsph_state *s)
{
    if (p->scheme != TFSPH_SCHEME_IDIC || p->dim > 2) return 0;
    const int64_t ng = s->gas.n, nd = s->dust.n, most = kSmallParticles;
    if (ng > most || nd > most || ng + nd == 0) return 0;
    const int rows = mask_rows_of(p);
    if (p->dim == 2 && rows == 0) return 0;
    double cand = double(ng) / ncell_of(p);          // window candidates of a particle
    for (int d = 0; d < p->dim; ++d) cand *= 2 * window_of(p, d) + 1;
    if (double(ng) * cand > (p->precision == TFSPH_F64 ? kSmallPairsF64 : kSmallPairsF32)) return 0;
    if (ncell_of(p) > 16 * kSmallOwn * kSmallBlock) return 0;
    const size_t lds = with_types(p, s->gas.mass != nullptr, [&](auto r, auto dim, auto kind) {
        return carve_bytes<decltype(r), decltype(dim)::value, decltype(kind)::value>((int)ng, (int)nd, ncell_of(p), rows);
    });
    return lds <= kSmallLds ? lds : 0;
}

tfsph_status tfsph_host::enqueue_small_steps(const tfsph_params *p, const tfsph_state *s, size_t lds, int n_steps,
                                             const Flags &F, hipStream_t st)
{
    for (int done = 0; done < n_steps; done += kSmallSteps) {
        const int k = n_steps - done < kSmallSteps ? n_steps - done : kSmallSteps;
        const tfsph_status r = with_types(p, s->gas.mass != nullptr, [&](auto r, auto dim, auto kind) {
            return launch<decltype(r), decltype(dim)::value, decltype(kind)::value>(p, s, lds, k, F, st);
        });
        if (r != TFSPH_OK) return r;
    }
    return TFSPH_OK;
}
