// Support test of the 3D window scans on the matrix cores.
//
// A particle of a 3D problem with cells of one support radius has 216 window
// candidates and about 30 neighbours.  Scanning them one by one with the exact
// kernel term (24 VALU instructions and a 16-byte load each, every lane its own
// cell range) bound the density pass by VALU issue and by the L1 return path
// (343 us on the 128^3 box).  Here a wave first finds which candidates can lie
// inside the support: the scaled squared distance of 32 targets to 32 candidates
// is a product of small matrices,
//   (|a - b|^2 - R^2) / 2 = (|b|^2 / 2) 1 - a . b + 1 (|a|^2 - R^2) / 2,
// with K = 8 half-precision columns (x, y, z, |b|^2/2 in two parts, and the
// target's constant in two parts), one 32x32x8 MFMA per 32 candidates.  The
// sign bits of the results are the neighbour bits: one v_alignbit per result
// and v_permlane32_swap bring each target's bits into its own lane.  Each half
// wave has 32 targets, consecutive in the sorted order, so their windows in one
// row of cells are one run of candidates (plus the cells wrapped around the box),
// loaded once, coalesced: about 48 candidates for targets in 4 cells (64 targets
// on one run of 80 left three quarters of the results unused).
//
// The test is an inclusion test only: R exceeds the support by a bound on the
// rounding of the half-precision coordinates, so every pair inside the support
// is kept, and the exact term, evaluated by walk_bits() for the kept ones in
// the scan's own order, is zero for the few others.  The sums are those of the
// scan bit for bit.  128^3 box after 100 steps, scan -> tiles: gas density 352 -> 333 us
// (FP32), MK gas drag 807 -> 613, MK dust drag 639 -> 483; FP64 64^3 step 215 -> 186.
// The density pass issues VALU instructions in three quarters of the slots (4490 a wave over the
// first hundred steps of the box), the drag sums in two thirds; by the listing about 190 a row (36 of
// the test itself per 64 candidates, 64 sign bits) and 39 per visited neighbour.
// Coordinates are relative to the middle of the wave's run of cells, in units of the
// support radius 2h.
#pragma once

#include "sph.hpp"

namespace tfsph {

constexpr int kTileWaves = 4;        // waves per SIMD of the FP32 kernels
// Widest run of cells (along x) of the targets that share one origin: 16 cells
// keep |x| within 9 cells, of at most 2 units each (tile_windows()): 18, where a
// half-precision step is 2^-6.  The inclusion radius grows with it (tile_groups()).
// Wider spread targets form further groups.
constexpr int kTileSpan = 15;
constexpr int kTileGroups = 3;       // groups of targets per wave; any left over scan their windows
constexpr int kTileRun = 512;        // longest candidate run of a group and row

using Half2 = __attribute__((ext_vector_type(2))) _Float16;
using Half4 = __attribute__((ext_vector_type(4))) _Float16;
using Acc16 = __attribute__((ext_vector_type(16))) float;

__device__ __forceinline__ unsigned pack_half(_Float16 a, _Float16 b)
{
    Half2 h;
    h.x = a;
    h.y = b;
    return __builtin_bit_cast(unsigned, h);
}

__device__ __forceinline__ Half4 half4_of(unsigned lo, unsigned hi)
{
    const uint64_t v = (uint64_t(hi) << 32) | lo;
    return __builtin_bit_cast(Half4, v);
}

// lanes 0..31 of p and q into x (p low, q low as the upper half), lanes 32..63 into y
__device__ __forceinline__ void swap_halves(unsigned p, unsigned q, unsigned &x, unsigned &y)
{
    auto r = __builtin_amdgcn_permlane32_swap(p, q, false, false);
    x = r[0];
    y = r[1];
}

// sign bits of the 16 results of a lane, result r at bit r
__device__ __forceinline__ unsigned sign_bits(const Acc16 &d)
{
    unsigned w = 0;
#pragma unroll
    for (int r = 15; r >= 0; --r) w = __builtin_amdgcn_alignbit(w, __float_as_uint(d[r]), 31);
    return w;
}

// Matrix columns of a point: a candidate has (x, y, z, c_hi | c_lo, 1, 1, 0) with
// c = |b|^2 / 2, a target (-x, -y, -z, 1 | 1, c_hi, c_lo, 0) with c = (|a|^2 - R^2) / 2;
// the first four come from lanes 0..31, the others from lanes 32..63, and c is kept to
// 22 bits in two halves.  The squared norm is that of the rounded coordinates.
__device__ __forceinline__ void tile_halves(float x, float y, float z, _Float16 h[3], float &norm2)
{
    h[0] = _Float16(x);
    h[1] = _Float16(y);
    h[2] = _Float16(z);
    const float fx = float(h[0]), fy = float(h[1]), fz = float(h[2]);
    norm2 = fx * fx + fy * fy + fz * fz;
}

// One group of targets per half wave (32 lanes): a run of cells of one row.  The
// members of [2] are wave-uniform, one per half; on[h] is false for a half
// without targets.
struct TileGroups {
    bool on[2];
    int cy[2], cz[2], cx0[2], cx1[2];
    Half4 b[2];                 // matrix operands of the halves' targets
    bool in;                    // this lane's target belongs to its half's group
    unsigned long long lanes;   // lanes of both groups
};

// The first group of each half among the lanes of todo (not empty).
template <typename R>
__device__ __forceinline__ void tile_groups(const Geom<R> &G, unsigned long long todo, int cx, int cy, int cz,
                                            const R oa[3], TileGroups &T)
{
    const int lane = threadIdx.x & 63;
    const float s = 0.5f * float(G.inv_h);
    const float sx = float(G.delta[0]) * s;
    T.lanes = 0;
    bool in_half[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned mine = unsigned(todo >> (32 * h));
        T.on[h] = mine != 0;
        const int first = 32 * h + (mine ? __builtin_ctz(mine) : 0);
        T.cx0[h] = __builtin_amdgcn_readlane(cx, first);
        T.cy[h] = __builtin_amdgcn_readlane(cy, first);
        T.cz[h] = __builtin_amdgcn_readlane(cz, first);
        in_half[h] = (lane >> 5) == h && ((todo >> lane) & 1) && cy == T.cy[h] && cz == T.cz[h] && cx >= T.cx0[h] &&
                     cx - T.cx0[h] <= kTileSpan;
        const unsigned long long group = __ballot(in_half[h]);
        T.cx1[h] = __builtin_amdgcn_readlane(cx, group ? 63 - __builtin_clzll(group) : 0);
        T.lanes |= group;
    }
    T.in = in_half[0] || in_half[1];
    const int x0 = lane < 32 ? T.cx0[0] : T.cx0[1], x1 = lane < 32 ? T.cx1[0] : T.cx1[1];
    const float mid = 0.5f * float(x0 + x1 + 1);
    // a bound on the distance error: half an ulp (2^-11 of the value) per coordinate of either
    // point, and 0.002 for the single-precision steps and the inclusion margin kMaskQ
    const float mx = (0.5f * float(x1 - x0 + 1) + 1.0f) * sx;
    const float my = 2.0f * float(G.delta[1]) * s, mz = 2.0f * float(G.delta[2]) * s;
    const float rad = 1.002f + 0.0009765625f * __builtin_amdgcn_sqrtf(mx * mx + my * my + mz * mz);
    _Float16 h[3];
    float n2;
    tile_halves((float(cx) - mid) * sx + float(oa[0]) * s, float(oa[1]) * s, float(oa[2]) * s, h, n2);
    const float c = 0.5f * (n2 - rad * rad);
    const _Float16 c_hi = _Float16(c);
    const _Float16 c_lo = _Float16(c - float(c_hi));
    const _Float16 one = _Float16(1.0f), zero = _Float16(0.0f);
    unsigned b0x, b0y, b1x, b1y;
    swap_halves(pack_half(-h[0], -h[1]), pack_half(one, c_hi), b0x, b1x);
    swap_halves(pack_half(-h[2], one), pack_half(c_lo, zero), b0y, b1y);
    T.b[0] = half4_of(b0x, b0y);
    T.b[1] = half4_of(b1x, b1y);
}

// Bits of the candidates of one row (dy, dz) of the groups' windows for each target:
// bit k of a lane is the k-th candidate of its row (cells cx - 1 .. cx + 1 in
// order), bs0 the first index of its cell cx - 1 and len the number of candidates.
// False when a run is too long (the caller scans).
template <typename R>
__device__ __forceinline__ bool tile_row(const Geom<R> &G, const TileGroups &T, int dy, int dz, int cx, int bs0, int len,
                                         const int *__restrict__ start, const int *__restrict__ cell,
                                         const R4<R> *__restrict__ data, unsigned long long &bits)
{
    const int nx = G.nc[0];
    const int lane = threadIdx.x & 63;
    // the run of a group in walking order: [cell nx - 1 wrapped to the left] [cells lo..hi]
    // [cell 0 wrapped to the right]
    int row[2], s_left[2], s_mid[2], s_right[2], n_left[2], n_lm[2], n_run[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        n_run[h] = 0;
        n_left[h] = 0;
        s_mid[h] = 0;
        if (!T.on[h]) continue;
        row[h] = nx * (wrap_once(T.cy[h] + dy, G.nc[1]) + G.nc[1] * wrap_once(T.cz[h] + dz, G.nc[2]));
        const bool left = T.cx0[h] == 0, right = T.cx1[h] == nx - 1;
        const int lo = left ? 0 : T.cx0[h] - 1, hi = right ? nx - 1 : T.cx1[h] + 1;
        s_mid[h] = start[row[h] + lo];
        s_left[h] = start[row[h] + nx - 1];
        s_right[h] = start[row[h]];
        n_left[h] = left ? start[row[h] + nx] - s_left[h] : 0;
        n_lm[h] = n_left[h] + start[row[h] + hi + 1] - s_mid[h];
        n_run[h] = n_lm[h] + (right ? start[row[h] + 1] - s_right[h] : 0);
    }
    const int n_most = max(n_run[0], n_run[1]);
    if (n_most > kTileRun) return false;
    // position of the lane's first candidate in its group's run
    const int v_first = cx == 0 ? 0 : bs0 + (lane < 32 ? n_left[0] - s_mid[0] : n_left[1] - s_mid[1]);
    // matrix row rho belongs to candidate 16 hi + r of result r (see sign_bits()): the lane
    // that supplies row rho loads that candidate
    const int rho = lane & 31;
    const int mine = (lane & 32) + 16 * ((rho >> 2) & 1) + 4 * (rho >> 3) + (rho & 3);
    const float s = 0.5f * float(G.inv_h);
    const float sx = float(G.delta[0]) * s, yd = float(dy) * float(G.delta[1]) * s, zd = float(dz) * float(G.delta[2]) * s;
    const _Float16 one = _Float16(1.0f), zero = _Float16(0.0f);
    bits = 0;
    for (int v0 = 0; v0 < n_most; v0 += 64) {
        unsigned w[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (v0 >= n_run[h]) continue;
            const int v = min(v0 + mine, n_run[h] - 1);
            const bool in_left = v < n_left[h], in_right = v >= n_lm[h];
            const int idx = v + (in_left ? s_left[h] : (in_right ? s_right[h] - n_lm[h] : s_mid[h] - n_left[h]));
            const R4<R> q = data[idx];
            const int u = cell[idx] - row[h] + (in_left ? -nx : (in_right ? nx : 0));
            const float mid = 0.5f * float(T.cx0[h] + T.cx1[h] + 1);
            _Float16 x[3];
            float n2;
            tile_halves((float(u) - mid) * sx + float(q.x) * s, float(q.y) * s + yd, float(q.z) * s + zd, x, n2);
            const float c = 0.5f * n2;
            const _Float16 c_hi = _Float16(c);
            const _Float16 c_lo = _Float16(c - float(c_hi));
            unsigned a0x, a0y, a1x, a1y;
            swap_halves(pack_half(x[0], x[1]), pack_half(c_lo, one), a0x, a1x);
            swap_halves(pack_half(x[2], c_hi), pack_half(one, zero), a0y, a1y);
            const Acc16 none = {};
            w[h][0] = sign_bits(__builtin_amdgcn_mfma_f32_32x32x8f16(half4_of(a0x, a0y), T.b[h], none, 0, 0, 0));
            if (v0 + 32 < n_run[h])
                w[h][1] = sign_bits(__builtin_amdgcn_mfma_f32_32x32x8f16(half4_of(a1x, a1y), T.b[h], none, 0, 0, 0));
        }
        unsigned l0, h0, l1, h1;
        swap_halves(w[0][0], w[1][0], l0, h0);
        swap_halves(w[0][1], w[1][1], l1, h1);
        const unsigned long long word = (uint64_t(l1 | (h1 << 16)) << 32) | (l0 | (h0 << 16));
        const int sh = v0 - v_first;
        if (sh >= 0) bits |= sh < 64 ? word << (sh & 63) : 0ull;
        else bits |= sh > -64 ? word >> ((-sh) & 63) : 0ull;
    }
    bits &= len >= 64 ? ~0ull : (1ull << (len & 63)) - 1ull;
    return true;
}

// The pairs of rows of a 3D window of one cell on each side, as for_window_pairs(),
// with the neighbour bits of each pair: fn(i, bs, be, ry0, rz0, P, shift, full, m),
// where m is a superset of the candidates inside the support (P, shift as
// pair_segments()); full marks a pair of more than kMaskBits candidates (every
// candidate has to be visited, m means nothing).  Every lane of the wave must call
// it, in the sorted order of its particles; start, cell and data belong to the
// candidates' phase.
template <typename R, typename Fn>
__device__ __forceinline__ void for_tile_pairs(const Geom<R> &G, int cx, int cy, int cz, const R oa[3],
                                               const int *__restrict__ start, const int *__restrict__ cell,
                                               const R4<R> *__restrict__ data, Fn &&fn)
{
    const int lane = threadIdx.x & 63;
    const R cut = R(kMaskQ) * G.h;
    const R cut2 = cut * cut;
    auto inside = [&](int, const R4<R> &, R rx, R ry, R rz, bool ok) {
        return ok && rx * rx + ry * ry + rz * rz < cut2;
    };
    TileGroups T0;               // the first groups serve every pair of rows
    tile_groups<R>(G, ~0ull, cx, cy, cz, oa, T0);
    for_window_pairs<R, 3, 1>(G, cx, cy, cz, oa, start, [&](int i, auto &bs, auto &be, const R *ry0, const R *rz0) {
        int P[6], shift[6];
        const int n_pair = pair_segments<3>(bs, be, P, shift);
        const bool full = n_pair > kMaskBits;
        const int len[2] = {P[3], n_pair - P[3]};
        unsigned long long m = 0;
        // bits of the targets of T; false when a run is too long
        auto rows = [&](const TileGroups &T) {
            unsigned long long bits[2] = {0ull, 0ull};
            bool done = true;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int l = t ? 8 - i : i;
                if (t == 1 && l == i) break;
                int dy, dz;
                row_offsets(l, 1, 1, dy, dz);
                done = done && tile_row<R>(G, T, dy, dz, cx, bs[t][0], len[t], start, cell, data, bits[t]);
            }
            if (done && T.in) m = bits[0] | (len[0] < 64 ? bits[1] << (len[0] & 63) : 0ull);
            return done;
        };
        unsigned long long todo = ~0ull;
        if (rows(T0)) todo &= ~T0.lanes;
        for (int g = 1; g < kTileGroups && todo; ++g) {
            TileGroups T;
            tile_groups<R>(G, todo, cx, cy, cz, oa, T);
            if (!rows(T)) break;
            todo &= ~T.lanes;
        }
        if (((todo >> lane) & 1) && !full) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    m |= visit_range_bits<R, 3>(bs[t][k], be[t][k], data, oa[0] - R(k - 1) * G.delta[0], ry0[t], rz0[t],
                                                t ? P[3 + k] : P[k], inside);
        }
        fn(i, bs, be, ry0, rz0, P, shift, full, m);
    });
}

// Visit the candidates of the window that lie inside the support (and a few
// more, whose terms are zero) in the order of for_window(): fn(b, q, rx, ry, rz,
// valid).  With mask the bits of each pair of rows are stored at mask[i stride]
// when store is set.
template <typename R, typename Fn>
__device__ __forceinline__ void for_tile_support(const Geom<R> &G, int cx, int cy, int cz, const R oa[3],
                                                 const int *__restrict__ start, const int *__restrict__ cell,
                                                 const R4<R> *__restrict__ data, unsigned long long *mask, int stride,
                                                 bool store, Fn &&fn)
{
    R rx0[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) rx0[k] = oa[0] - R(k - 1) * G.delta[0];
    const bool rows_contiguous = __ballot(cx < 1 || cx + 1 >= G.nc[0]) == 0ull;
    for_tile_pairs<R>(G, cx, cy, cz, oa, start, cell, data,
                      [&](int i, auto &bs, auto &be, const R *ry0, const R *rz0, const int (&P)[6],
                          const int (&shift)[6], bool full, unsigned long long m) {
                          if (mask && store) mask[size_t(i) * stride] = m;
                          if (full) {
#pragma unroll
                              for (int t = 0; t < 2; ++t)
#pragma unroll
                                  for (int k = 0; k < 3; ++k)
                                      visit_range<R, 3>(bs[t][k], be[t][k], data, rx0[k], ry0[t], rz0[t], fn);
                          } else if (rows_contiguous) {
                              walk_bits<R, 3, 3, true, R>(m, P, shift, rx0, ry0, rz0, data, fn);
                          } else {
                              walk_bits<R, 3, 3, false, R>(m, P, shift, rx0, ry0, rz0, data, fn);
                          }
                      });
}

// k_density for 3D windows of one cell: the support test above, then the kernel
// term for the kept candidates.  Every lane takes part (lanes past the end
// repeat the last particle and store nothing).
template <typename R>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? kTileWaves : 3)))
k_density_tiles(Geom<R> G, Phys<R> Ph, Sorted<R> S, int want_frc)
{
    const int a0 = xcd_block(gridDim.x) * kBlock + threadIdx.x;
    const bool live = a0 < S.n;
    const int a = live ? a0 : S.n - 1;
    int cx, cy, cz;
    cell_coords<3>(G, S.cell[a], cx, cy, cz);
    const R4<R> me = S.pos[a];
    const R oa[3] = {me.x, me.y, me.z};
    R acc = R(0);
    for_tile_support<R>(G, cx, cy, cz, oa, S.start, S.cell, S.pos, want_frc && S.nmask ? S.nmask + a : nullptr, S.n, live,
                        [&](int, const R4<R> &q, R rx, R ry, R rz, bool ok) { density_add(G, q, rx, ry, rz, ok, acc); });
    if (!live) return;
    density_finish<R>(G, Ph, S, a, me, acc * G.wnorm, want_frc);
}

// Whether 3D pair sums between a phase of `least` and one of `most` particles take the tile path: a
// window of one cell per axis, cells at most four smoothing lengths wide (coarser ones would
// widen the rounding bound, and scans of such windows are rare), and on average at most 55
// candidates per pair of rows (6 cells): near kMaskBits = 64 many pairs are visited whole
// and the test is wasted.  IDIC step, us, tiles / scan: 2.2^3 particles per cell (64 per pair) 138.5 /
// 131.1, 2.1^3 (56) 114.4 / 113.5 (MK 238 / 259), 2.05^3 (51) 104.7 / 110.8.  Few candidates leave the
// matrices empty: at least 38 per pair in FP32, 25 in FP64.  Tiles / scan by particles per cell, MK step
// 80^3 FP32: 1 385 / 219, 3 434 / 376, 5 482 / 474, 6 504 / 523, 7 529 / 570; IDIC 100^3 FP32: 5 346 / 338, 6 350 /
// 346, 7 365 / 378; MK 32^3 FP64: 3 185 / 162, 4 184 / 181, 5 189 / 194; IDIC 64^3 FP64: 1 164 / 139, 3 160 / 172.
constexpr double kTilePairMost = 55.0;
template <typename R>
constexpr double tile_pair_least() { return sizeof(R) == 4 ? 38.0 : 25.0; }
template <typename R>
inline bool tile_windows(const Geom<R> &G, int least, int most)
{
    if (G.dim != 3 || 6.0 * most > kTilePairMost * G.ncell || 6.0 * least < tile_pair_least<R>() * G.ncell) return false;
    for (int d = 0; d < 3; ++d)
        if (G.win[d] != 1 || G.delta[d] > R(4) * G.h) return false;
    return true;
}

// Whether the density pass of n particles takes the tile kernel (masks: it records them).
// The FP32 form holds 4 waves per SIMD against 7 of the scan: up to 7 per SIMD the scan runs in
// one round, and the tile kernel is at best as fast.  Without masks (dust) the scan saves their
// stores and loses to the tiles only while the dust is even.  us a launch, tiles / scan,
// box of n^3 particles fresh and after 100 steps, gas: 32^3 30.3 / 27.1 and 33.2 / 33.7; 45^3
// 49.8 / 45.7, 40.7 / 41.9; 64^3 53.4 / 54.2, 53.5 / 52.7; 72^3 74.7 / 73.0, 80.5 / 71.1; 80^3 (8000
// waves) 93.6 / 117, 96.7 / 107; 96^3 146 / 162, 150 / 153; 128^3 318 / 361, 333 / 352.  Dust: 64^3
// 49.3 / 48.7, 59.6 / 48.3; 96^3 140 / 151, 184 / 152; 128^3 298 / 330, 402 / 352.  FP64 holds few
// waves either way: 32^3 33 / 38 and 37 / 49, 64^3 77 / 113 and 83 / 121, dust 75 / 96 and 96 / 113.
constexpr int kScanWaves = 7 * 4 * 256;      // 7 per SIMD of 256 CUs
template <typename R>
inline bool tile_density(const Geom<R> &G, int n, bool masks)
{
    const int waves = n / 64 + (n % 64 != 0);
    return tile_windows(G, n, n) && (sizeof(R) == 8 || (masks && waves > kScanWaves));
}

}  // namespace tfsph
