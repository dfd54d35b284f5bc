// hmc_sweep_kernels.hip -- a whole standard sweep (both colours of Table A1 and
// the cone-angle rule of the sweep before) in one launch, for lattices too
// small to fill the chip.
//
// Such a lattice's sweep costs its launches: a red pass, a black pass and a
// finalize took 4.2, 4.2 and 4.6 us at 16^3 to 64^3 (MI355X), hardly more than
// the three launches' own latencies, while the vector units idle.  Here a
// work-group updates the black sites of a tile (ry rows of zc planes) and
// recomputes for itself every red site they touch: the red sites of the tile,
// one row more on both sides and the tile's rows of the planes below and above.
// The random numbers are keyed by site and the arithmetic is update_site's,
// so a red site comes out the same in every work-group that computes it, and
// the sweep is that of the two passes bit for bit.  Nothing is updated in
// place: a sweep reads one copy of the spins and writes the other
// (DevLattice::spins and the scratch of the constrained sweeps in turn; a call
// of an odd number of sweeps begins with a plain copy, so that it too ends in
// DevLattice::spins).
//
// The cone angle of a sweep needs the acceptances of the whole lattice in the
// sweep before.  Every work-group sums the counts that the launch before
// left (a few loads, in flight with the spins'), and one work-group more does
// that sweep's finalize beside the others.  What two launches in a row share
// is kept twice, by the parity of the launch, so that none overwrites what
// another work-group of it still reads.  The records are folded in one order
// in every sweep, so a chain does not depend on how calls divide it.
//
// What bounds a launch at 16^3 to 48^3 is latency: of 3.7 us inside the kernel
// (FP32, unsampled, before the cone table went into the slots) 2.3 are two or
// three loads behind one another that miss every cache after the launch
// boundary, 0.8 the red and 0.7 the black update of one site per thread.
#include "hmc_pass.hpp"

namespace hmc {

namespace {

// Work-group size, and sites of old black and of new red spins in LDS.  FP32:
// 75 KB, two work-groups of eight waves to a compute unit; FP64: the same
// bytes for two of four waves, whose update takes twice the registers.
template <typename R> struct TileCap;
template <> struct TileCap<float> { static constexpr int threads = 512, black = 4096, red = 2304; };
template <> struct TileCap<double> { static constexpr int threads = 256, black = 2048, red = 1280; };

// Most tiles of a launch, two to a compute unit.  Every tile sums their counts,
// a thread kMostTiles / work-group size of them.
constexpr int kMostTiles = 512;

// n / d for n * d < 2^32, d >= 2
struct Div {
    uint32_t d, m;
    __device__ __forceinline__ uint32_t of(uint32_t n) const { return __umulhi(n, m); }
};

Div div_by(uint32_t d) { return Div{d, (uint32_t)((1ull << 32) / d) + 1u}; }

// What a launch leaves for the next one: its cone angle and sweep number, and
// the cone table's entries one degree up and down, one of which the next
// launch takes (so its table look-up does not wait for its angle).
template <typename R>
struct SweepSlot {
    int32_t theta;
    uint32_t sweep;
    R up, down;
};
static_assert(offsetof(SweepSlot<float>, up) == 8 && offsetof(SweepSlot<double>, down) == 16, "slot layout");

template <typename R>
struct SweepArgs {
    R* dst;              // component array j of colour c at dst + (3c + j) * pitch / sizeof(R)
    size_t pitch;
    uint32_t ry, zc, nyt, ntile;
    Div hx;
    SweepSlot<R>* slot;  // [2]
    uint32_t* cnt;       // [2][ntile]
    double* part;        // [2][kObsRows][ntile]
    uint32_t parity;     // of this launch
    int32_t first;       // no launch before this one in the call
    int32_t fin;         // finalize flags of a sweep
    double T, N;
    R scale;
};

__device__ __forceinline__ uint32_t wrap(int32_t v, uint32_t n)
{
    return v < 0 ? (uint32_t)(v + (int32_t)n) : ((uint32_t)v >= n ? (uint32_t)v - n : (uint32_t)v);
}

// Spins in LDS, one array per component at a fixed distance.
template <typename R, int S>
struct Lds {
    R* p;
    __device__ __forceinline__ V3<R> get(uint32_t e) const { return V3<R>{p[e], p[S + e], p[2 * S + e]}; }
    __device__ __forceinline__ void put(uint32_t e, const V3<R>& v) const
    {
        p[e] = v.x;
        p[S + e] = v.y;
        p[2 * S + e] = v.z;
    }
};

// The neighbour sum of a site of colour C at LDS entry e of the other colour's
// tile (rows of hx, planes of pl), in the order of the passes; o0 receives
// the same-index partner.
template <typename R, int S, bool MASK>
__device__ __forceinline__ V3<R> tile_neighbours(const Lds<R, S>& o, uint32_t e, uint32_t kx, uint32_t p, uint32_t hx,
                                                 uint32_t pl, bool below, bool above, uint32_t zbound, uint32_t mb,
                                                 V3<R>& o0)
{
    const uint32_t ed = p ? (kx == hx - 1 ? e + 1 - hx : e + 1) : (kx == 0 ? e + hx - 1 : e - 1);
    o0 = o.get(e);
    const V3<R> xd = o.get(ed), ym = o.get(e - hx), yp = o.get(e + hx);
    V3<R> zm = o.get(e - pl), zp = o.get(e + pl);
    if (zbound) {
        if (below) zm = across_z(zm, zbound);
        if (above) zp = across_z(zp, zbound);
    }
    if (MASK) {
        const V3<R> xm = p ? o0 : xd, xp = p ? xd : o0;
        const R w0 = (mb & 1u) ? R(1) : R(0), w1 = (mb & 2u) ? R(1) : R(0);
        const R w2 = (mb & 4u) ? R(1) : R(0), w3 = (mb & 8u) ? R(1) : R(0);
        const R w4 = (mb & 16u) ? R(1) : R(0), w5 = (mb & 32u) ? R(1) : R(0);
        return V3<R>{((((w0 * xm.x + w1 * xp.x) + w2 * ym.x) + w3 * yp.x) + w4 * zm.x) + w5 * zp.x,
                     ((((w0 * xm.y + w1 * xp.y) + w2 * ym.y) + w3 * yp.y) + w4 * zm.y) + w5 * zp.y,
                     ((((w0 * xm.z + w1 * xp.z) + w2 * ym.z) + w3 * yp.z) + w4 * zm.z) + w5 * zp.z};
    }
    return V3<R>{((((o0.x + xd.x) + ym.x) + yp.x) + zm.x) + zp.x,
                 ((((o0.y + xd.y) + ym.y) + yp.y) + zm.y) + zp.y,
                 ((((o0.z + xd.z) + ym.z) + yp.z) + zm.z) + zp.z};
}

// The finalize of the last sweep of a call, by the work-group size that does the others.
template <typename R>
__global__ __launch_bounds__(TileCap<R>::threads) void sweep_finalize_kernel(DevState* st, const double* part,
                                                                             const uint32_t* cnt, uint32_t n, int fin,
                                                                             double T, double N)
{
    __shared__ double tot[kObsRows];
    __shared__ unsigned long long totc;
    fold_sweep<TileCap<R>::threads, kObsRows>(st, part, cnt, n, fin, T, N, tot, &totc);
}

// The six component arrays, from one copy to the other.
__global__ __launch_bounds__(kThreads) void copy_spins_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                              uint32_t n)
{
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) dst[i] = src[i];
}

template <typename R, bool OBS, bool MASK>
__global__ __launch_bounds__(TileCap<R>::threads) void sweep_kernel(const KArgs<R> a, const SweepArgs<R> f)
{
    constexpr int NT = TileCap<R>::threads, SB = TileCap<R>::black, SR = TileCap<R>::red, NW = NT / 64;
    constexpr int NB = SB / NT, NR = (SR + NT - 1) / NT;      // black loads and red sites per thread
    constexpr int NC = kMostTiles / NT;                       // counts per thread
    static_assert(SB % NT == 0 && kMostTiles % NT == 0, "black sites and counts per thread");
    __shared__ __align__(16) R smem[3 * (SB + SR)];
    __shared__ double tot[kObsRows];
    __shared__ unsigned long long totc;
    __shared__ uint32_t wacc[NW], wtot[NW];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t prev = f.parity ^ 1u;
    if (blockIdx.x == f.ntile) {
        fold_sweep<NT, kObsRows>(a.st, f.part + (size_t)prev * kObsRows * f.ntile, f.cnt + (size_t)prev * f.ntile, f.ntile, f.fin,
                       f.T, f.N, tot, &totc);
        return;
    }
    const uint32_t tile = xcd_remap(blockIdx.x, f.ntile);
    const uint32_t hx = a.hx, ny = a.ny, nz = a.nz;
    const uint32_t zt = tile / f.nyt, yt = tile - zt * f.nyt;
    const int32_t y0 = (int32_t)(yt * f.ry), z0 = (int32_t)(zt * f.zc);
    const uint32_t ry = min(f.ry, ny - (uint32_t)y0), zn = min(f.zc, nz - (uint32_t)z0);

    // the counts of the launch before, summed below: they move the angle one up or down
    // (added up only after the spins' loads have left; the first launch of a
    // call reads counts that nobody wrote and does not use them)
    uint32_t cq[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u)
        cq[u] = f.cnt[(size_t)prev * f.ntile + min(t + (uint32_t)u * NT, f.ntile - 1u)];
    // (through a buffer resource: as vector loads, which nothing waits for
    // before their use; scalar loads held up every load behind them)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(f.slot + prev, 0, (int)sizeof(SweepSlot<R>),
                                                                        kBufferConfig);
    const uint32_t left_theta = __builtin_amdgcn_raw_buffer_load_b32(rs, 0u, 0u, 0);
    const uint32_t left_sweep = __builtin_amdgcn_raw_buffer_load_b32(rs, 4u, 0u, 0);
    const R left_up = Gm<R>::ld(rs, 8u, 0u), left_down = Gm<R>::ld(rs, 8u + (uint32_t)sizeof(R), 0u);

    const Arrays<R> g(a);
    const Lds<R, SB> lb{smem};
    const Lds<R, SR> lr{smem + 3 * SB};
    // old black spins: the tile, two rows and two planes more on every side
    // (every load leaves before the first is waited for)
    const uint32_t rb = ry + 4u, plb = rb * hx, nb_all = plb * (zn + 4u);
    const uint32_t mrb = (uint32_t)((1ull << 32) / rb) + 1u;
    V3<R> v[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if ((uint32_t)i * NT < nb_all) {
            const uint32_t e = min(t + (uint32_t)i * NT, nb_all - 1u);
            const uint32_t rp = f.hx.of(e), kx = e - rp * hx;
            const uint32_t j = __umulhi(rp, mrb), row = rp - j * rb;
            const uint32_t z = wrap(z0 - 2 + (int32_t)j, nz), y = wrap(y0 - 2 + (int32_t)row, ny);
            v[i] = g.get(1, (kx + hx * (y + ny * z)) * (uint32_t)sizeof(R), 0);
        }
    }
    // the red sites this thread updates: first those of the tile's planes with
    // a row more on both sides, then the tile's rows of the planes below and above
    const uint32_t rr = ry + 2u, plr = rr * hx, inner = plr * zn, nr_all = inner + 2u * ry * hx;
    const uint32_t mrr = (uint32_t)((1ull << 32) / rr) + 1u;
    V3<R> so[NR];
    uint32_t at[NR];         // row, plane and x of the site: j | row << 8 | kx << 16
    uint32_t mk[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if ((uint32_t)i * NT < nr_all) {
            const uint32_t r = min(t + (uint32_t)i * NT, nr_all - 1u);
            const bool in = r < inner;
            const uint32_t rp = f.hx.of(in ? r : r - inner), kx = (in ? r : r - inner) - rp * hx;
            // plane z0 - 1 + j, row y0 - 1 + row
            const uint32_t q = __umulhi(rp, mrr);
            const uint32_t j = in ? q + 1u : (rp < ry ? 0u : zn + 1u);
            const uint32_t row = in ? rp - q * rr : (rp < ry ? rp : rp - ry) + 1u;
            at[i] = j | row << 8 | kx << 16;
            const uint32_t z = wrap(z0 - 1 + (int32_t)j, nz), y = wrap(y0 - 1 + (int32_t)row, ny);
            const uint32_t k = kx + hx * (y + ny * z);
            so[i] = g.get(0, k * (uint32_t)sizeof(R), 0);
            mk[i] = MASK ? a.mask[0][k] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const uint32_t e = t + (uint32_t)i * NT;
        if ((uint32_t)i * NT < nb_all && e < nb_all) lb.put(e, v[i]);
    }
    int32_t up, down;
    uint32_t sweep;
    R c1_up, c1_down;
    if (f.first) {
        up = down = a.st->theta;
        sweep = (uint32_t)a.st->sweep;
        c1_up = c1_down = a.c1tab[up];
    } else {
        const int32_t theta = __builtin_amdgcn_readfirstlane((int)left_theta);
        up = min(theta + 1, 180);
        down = max(theta - 1, 1);
        sweep = (uint32_t)__builtin_amdgcn_readfirstlane((int)left_sweep) + 1u;
        c1_up = left_up;
        c1_down = left_down;
    }
    {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < NC; ++u) c += t + (uint32_t)u * NT < f.ntile ? cq[u] : 0u;
        c = wave_sum(c);                       // N < 2^32
        if (lane == 0) wacc[wave] = c;
    }
    __syncthreads();
    // the rule of finalize_body (the first launch of a call takes the angle as it is)
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) before += wacc[w];
    const bool more = 2.0 * (double)before > f.N;
    const R c1 = more ? c1_up : c1_down;
    if (blockIdx.x == 0 && t == 0) {
        const int32_t theta = more ? up : down;
        f.slot[f.parity] = SweepSlot<R>{theta, sweep, a.c1tab[min(theta + 1, 180)], a.c1tab[max(theta - 1, 1)]};
    }

    uint32_t nacc = 0;
    Acc acc;
    Part<R> part;
    auto& pa = site_acc<R>(acc, part);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const uint32_t r = t + (uint32_t)i * NT;
        if (r < nr_all) {
            const uint32_t j = at[i] & 255u, row = at[i] >> 8 & 255u, kx = at[i] >> 16;
            const uint32_t z = wrap(z0 - 1 + (int32_t)j, nz), y = wrap(y0 - 1 + (int32_t)row, ny);
            const uint32_t k = kx + hx * (y + ny * z), p = (y + z) & 1u;
            V3<R> o0;
            const V3<R> nb = tile_neighbours<R, SB, MASK>(lb, ((j + 1u) * rb + row + 1u) * hx + kx, kx, p, hx, plb,
                                                          z == 0, z == nz - 1, a.zbound, mk[i], o0);
            const Rand4 rn = philox(sweep, 2u * k + p, 0u, a.inst, a.key0, a.key1);
            uint32_t ok = 0;
            const V3<R> s = update_site<R, false>(a.m, so[i], nb, o0, rn, c1, f.scale, ok, pa);
            lr.put((j * rr + row) * hx + kx, s);
            if (j - 1u < zn && row - 1u < ry) {          // of the tile
                nacc += ok;
                R* d = f.dst + k;
                const size_t pitch = f.pitch / sizeof(R);
                d[0] = s.x;
                d[pitch] = s.y;
                d[2 * pitch] = s.z;
            }
        }
    }
    __syncthreads();
    const uint32_t tp = ry * hx, nt = tp * zn;
    const uint32_t mry = ry > 1u ? (uint32_t)((1ull << 32) / ry) + 1u : 0u;
    for (uint32_t b = t; b < nt; b += NT) {
        const uint32_t rp = f.hx.of(b), kx = b - rp * hx;
        const uint32_t j = ry > 1u ? __umulhi(rp, mry) : rp, row = rp - j * ry;
        const uint32_t z = (uint32_t)z0 + j, y = (uint32_t)y0 + row;
        const uint32_t k = kx + hx * (y + ny * z), p = (y + z + 1u) & 1u;
        V3<R> o0;
        const uint32_t mb = MASK ? a.mask[1][k] : 0u;
        const V3<R> nb = tile_neighbours<R, SR, MASK>(lr, ((j + 1u) * rr + row + 1u) * hx + kx, kx, p, hx, plr, z == 0,
                                                      z == nz - 1, a.zbound, mb, o0);
        const V3<R> s = lb.get(((j + 2u) * rb + row + 2u) * hx + kx);
        const Rand4 rn = philox(sweep, 2u * k + p, 1u, a.inst, a.key0, a.key1);
        const V3<R> n = update_site<R, OBS>(a.m, s, nb, o0, rn, c1, f.scale, nacc, pa);
        const size_t pitch = f.pitch / sizeof(R);
        R* d = f.dst + 3 * pitch + k;
        d[0] = n.x;
        d[pitch] = n.y;
        d[2 * pitch] = n.z;
    }
    if constexpr (OBS) flush_part(acc, pa);
    // the tile's record
    uint32_t* cnt = f.cnt + (size_t)f.parity * f.ntile + tile;
    if constexpr (OBS) {
        static_assert(kObsRows * NT * sizeof(double) <= sizeof(smem), "the record's sums change places in the tile");
        const double v[kObsRows] = {acc.M[0], acc.M[1], acc.M[2], acc.ex, acc.eu, acc.ec, acc.ez};
        __syncthreads();                      // the tile's spins have been read
        write_record<NT, kObsRows>(v, nacc, f.part + (size_t)f.parity * kObsRows * f.ntile + tile, f.ntile, cnt,
                                   reinterpret_cast<double*>(smem), wtot);
    } else {
        const uint32_t na = wave_sum(nacc);
        if (lane == 0) wtot[wave] = na;
        __syncthreads();
        if (t == 0) {
            uint32_t tot = 0;
            for (int w = 0; w < NW; ++w) tot += wtot[w];
            *cnt = tot;
        }
    }
}

// The tiles of a lattice, and the space they need behind the copy of the spins.
struct Tiles {
    int ry = 0, zc = 0;
    uint32_t nyt = 0, n = 0;
    double cost = 0.0;           // of a launch, cycles
    size_t bytes = 0;
};

// Rows and planes of a tile, at most kMaxTileEdge.  A launch takes the vector work of its tiles, one
// compute unit each at a time (a red site about 550 cycles of a wave, a black
// one with its sums about 700), and per round of two tiles to a compute unit
// the latency of the loads and the reductions, about 3 us.
constexpr int kMaxTileEdge = 16;

// Equal parts of n rows or planes: their edges up to kMaxTileEdge, and how many parts.
struct Parts {
    uint32_t edge[kMaxTileEdge], parts[kMaxTileEdge];
    int count = 0;
};

Parts parts_of(uint32_t n)
{
    Parts p;
    for (uint32_t e = 1; e <= (uint32_t)kMaxTileEdge && e <= n; ++e) {
        const uint32_t parts = (n + e - 1) / e;
        if ((n + parts - 1) / parts != e) continue;
        p.edge[p.count] = e;
        p.parts[p.count++] = parts;
    }
    return p;
}

// (The divisions stand outside the double loop: inside it they took a new lattice
// 1 us of the host's time.)
template <typename R>
Tiles tiles_for(const DevLattice& d)
{
    using Cap = TileCap<R>;
    constexpr double kRed = sizeof(R) == 4 ? 550.0 : 1300.0, kBlack = sizeof(R) == 4 ? 700.0 : 1500.0, kRound = 7000.0;
    const uint32_t hx = (uint32_t)d.hx;
    const Parts y = parts_of((uint32_t)d.ny), z = parts_of((uint32_t)d.nz);
    Tiles best;
    for (int i = 0; i < y.count; ++i) {
        const uint32_t ry = y.edge[i];
        for (int j = 0; j < z.count; ++j) {
            const uint32_t zc = z.edge[j];
            if ((ry + 4) * (zc + 4) * hx > (uint32_t)Cap::black || (ry + 2) * (zc + 2) * hx > (uint32_t)Cap::red) break;
            const uint32_t red = ((ry + 2) * zc + 2 * ry) * hx, black = ry * zc * hx;
            const double work = ((red + 63) / 64 * kRed + (black + 63) / 64 * kBlack) / 4;
            const uint32_t n = y.parts[i] * z.parts[j];
            const double c = (n + 255) / 256 * work + (n + 511) / 512 * kRound;
            if (best.ry == 0 || c < best.cost) {
                best.cost = c;
                best.ry = (int)ry;
                best.zc = (int)zc;
                best.nyt = y.parts[i];
                best.n = n;
            }
        }
    }
    best.bytes = 2 * (size_t)best.n * (kObsRows * sizeof(double) + sizeof(uint32_t)) + 2 * sizeof(SweepSlot<R>);
    return best;
}

template <typename R>
bool plan_go(const DevLattice& d, SweepPlan* plan)
{
    // cycles of the passes of a sweep: unsampled, sampled; of a launch and per spin
    constexpr double kPasses[2] = {sizeof(R) == 4 ? 10500.0 : 12000.0, sizeof(R) == 4 ? 11800.0 : 12000.0};
    constexpr double kPassesSpin[2] = {sizeof(R) == 4 ? 0.0085 : 0.021, sizeof(R) == 4 ? 0.0095 : 0.021};
    const Tiles tl = tiles_for<R>(d);
    const size_t spins = 6 * d.pitch;
    const size_t room = 16 * (size_t)d.Nc * sizeof(R);       // the constrained scratch: at least this
    if (tl.n == 0 || tl.n > (uint32_t)kMostTiles || spins + tl.bytes > room) return false;
    for (int obs = 0; obs < 2; ++obs) plan->pays[obs] = tl.cost <= kPasses[obs] + kPassesSpin[obs] * (double)d.N;
    plan->ry = tl.ry;
    plan->zc = tl.zc;
    plan->ntile = (int32_t)tl.n;
    return true;
}

template <typename R, bool OBS>
void sweep_go(const DevLattice& d, const SweepPlan& p, const KArgs<R>& a, const SweepArgs<R>& f, hipStream_t s)
{
    const uint32_t grid = f.ntile + (f.first ? 0u : 1u);
    if (d.mask) sweep_kernel<R, OBS, true><<<grid, TileCap<R>::threads, 0, s>>>(a, f);
    else sweep_kernel<R, OBS, false><<<grid, TileCap<R>::threads, 0, s>>>(a, f);
}

// Behind the copy of the spins in the scratch: the partial sums, the slots, the counts.
template <typename R>
SweepArgs<R> args_for(const DevLattice& d, const SweepPlan& p, int launch, bool obs, double T)
{
    SweepArgs<R> f;
    f.pitch = d.pitch;
    f.ry = (uint32_t)p.ry;
    f.zc = (uint32_t)p.zc;
    f.nyt = cdiv((uint64_t)d.ny, (uint64_t)p.ry);
    f.ntile = (uint32_t)p.ntile;
    f.hx = div_by((uint32_t)d.hx);
    f.part = reinterpret_cast<double*>(static_cast<char*>(d.aos) + 6 * d.pitch);
    f.slot = reinterpret_cast<SweepSlot<R>*>(f.part + 2 * (size_t)kObsRows * f.ntile);
    f.cnt = reinterpret_cast<uint32_t*>(f.slot + 2);
    f.parity = (uint32_t)launch & 1u;
    f.first = launch == 0;
    f.fin = kFinCounts | (obs ? (kFinObs | kFinSample) : 0);
    f.T = T;
    f.N = (double)d.N;
    f.scale = Prim<R>::scale_for(T);
    f.dst = nullptr;
    return f;
}

template <typename R>
void run_go(const DevLattice& d, const SweepPlan& p, int launch, bool to_copy, bool obs, double T, hipStream_t s)
{
    SweepArgs<R> f = args_for<R>(d, p, launch, obs, T);
    DevLattice src = d;
    if (!to_copy) src.spins = d.aos;
    f.dst = static_cast<R*>(to_copy ? d.aos : d.spins);
    const auto a = make_args<R>(src);
    if (obs) sweep_go<R, true>(d, p, a, f, s);
    else sweep_go<R, false>(d, p, a, f, s);
}

template <typename R>
void finalize_go(const DevLattice& d, const SweepPlan& p, int launch, bool obs, double T, hipStream_t s)
{
    const SweepArgs<R> f = args_for<R>(d, p, launch, obs, T);
    sweep_finalize_kernel<R><<<1, TileCap<R>::threads, 0, s>>>(d.st, f.part + (size_t)f.parity * kObsRows * f.ntile,
                                                               f.cnt + (size_t)f.parity * f.ntile, f.ntile, f.fin, T,
                                                               f.N);
}

}  // namespace

// One launch pays while the work it repeats costs less than the launches it
// saves: up to a number of spins, and below it where the launch (tiles_for) costs
// no more cycles than the passes in their default shape.  Long rows leave room for
// tiles of a row or two only, which recompute three to five red sites for one.
// The lines of sampled and unsampled sweeps differ (an unsampled sweep sums
// integers only, so it leaves the same state either way; sampled ones keep to one
// form, for the order of their sums).  Measured on MI355X, us per sampled sweep (in
// brackets unsampled) against those passes, each of which carries the finalize of
// the sweep before: FP32 32^3 6.4 for 9.5 (5.8 for 7.8), 64^3 8.4 for 11.7 (7.7 for
// 8.6), 84^3 12.1 for 14.5 (11.5 for 12.4); FP64 32^3 7.2 for 10.5 (6.6 for 9.5),
// 66^3 14.1 for 16.6 (13.1 for 15.2).  Where the cost draws the line: FP32 128 x 128
// x 32 12.6 for 14.8 (11.9 for 10.8); sampled only 256 x 32 x 32 11.2 for 12.2 (10.4 for
// 9.3), 128 x 68 x 68 13.8 for 14.4 (12.8 for 12.4); passes 160 x 60 x 60 14.6 for 14.6
// (13.7 for 12.6), 200 x 50 x 50 18.0 for 14.5 (17.0 for 10.7), 272 x 32 x 64 20.3 for
// 14.8 (19.0 for 12.9); FP64 60^3 12.5 for 12.9 (11.7 for 11.6), passes 96 x 64 x 40 15.1
// for 13.3 (13.9 for 12.0).  Above the spins' line it lost already to passes with a
// finalize launch each: FP32 112^3 27.3 for 25.6, FP64 80^3 25.8 for 25.4.
bool sweep_plan(const DevLattice& d, SweepPlan* plan)
{
    constexpr int64_t kMost[2] = {600000, 300000};          // spins, FP32 and FP64
    if (d.hx < 2 || d.nz < 2 || d.N > kMost[d.precision == 32 ? 0 : 1]) return false;
    return d.precision == 32 ? plan_go<float>(d, plan) : plan_go<double>(d, plan);
}

hipError_t launch_sweep_copy(const DevLattice& d, hipStream_t s)
{
    const uint32_t n = (uint32_t)(6 * d.pitch / sizeof(uint4));
    const uint32_t full = cdiv((uint64_t)n, kThreads);
    copy_spins_kernel<<<full < 2048u ? full : 2048u, kThreads, 0, s>>>(static_cast<const uint4*>(d.spins),
                                                                     static_cast<uint4*>(d.aos), n);
    return hipGetLastError();
}

hipError_t launch_sweep(const DevLattice& d, const SweepPlan& p, int launch, bool to_copy, bool obs, double T,
                        hipStream_t s)
{
    if (d.precision == 32) run_go<float>(d, p, launch, to_copy, obs, T, s);
    else run_go<double>(d, p, launch, to_copy, obs, T, s);
    return hipGetLastError();
}

hipError_t launch_sweep_finalize(const DevLattice& d, const SweepPlan& p, int launch, bool obs, double T, hipStream_t s)
{
    if (d.precision == 32) finalize_go<float>(d, p, launch, obs, T, s);
    else finalize_go<double>(d, p, launch, obs, T, s);
    return hipGetLastError();
}

}  // namespace hmc
