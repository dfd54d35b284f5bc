// hmc_kernels.hip -- gfx950 kernels of the parallel Metropolis sweeps
// (Lepadatu et al., arXiv:2103.03517, Sec. 2, Tables A1 and A2).
//
// Spin storage: colour-split structure of arrays.  Site (x, y, z) has colour
// c = (x + y + z) & 1 (red = 0) and colour index k = (x + nx*(y + ny*z)) / 2;
// its components live in s[c][0..2][k].  Within a colour, k = kx + hx*(y +
// ny*z) with hx = nx/2, and the x-partner with the same k is the other colour.
// Every kernel reads one colour as neighbours and writes only the other, so a
// colour pass has no read/write overlap (Sec. 2: the two sets do not
// interact in Eq. 2).
//
// Global memory is accessed through buffer resources: the per-plane offset
// travels in a scalar register, so the per-column offsets are computed once,
// and out-of-range accesses are dropped by the hardware.
#include "hmc_pass.hpp"

namespace hmc {

// In-plane windows or tiles of the colour pass.  Tiles: the width (a row cut
// into equal parts) and height that cost least, where a site costs its own
// accesses and its tile's share of the halo (a third: the caches hold most of
// it), and threads without a site cost as much as others.  Parts are 48 to 127
// sites: wide enough for runs of lines, and with one halo site per thread.  Two
// thirds of the threads of a one-site shape have a site at least, so a pass
// has no more work-groups than a workspace holds records for (max_blocks_for:
// twice as many as full ones; launch_pass checks it).
PassGeom pass_geometry(int hx, int ny, int spt)
{
    const uint32_t most = (uint32_t)kThreads * (uint32_t)spt;
    PassGeom best{};
    if (geometry_of(hx) != 0) {
        best.n = cdiv((uint64_t)hx * ny, most);
        best.entries = most + 2u * (uint32_t)hx;
        return best;
    }
    double cost = 0.0;
    for (uint32_t parts = cdiv((uint64_t)hx, 127); parts <= (uint32_t)hx / 48u; ++parts) {
        const uint32_t tx = cdiv((uint64_t)hx, parts);
        uint32_t ty = most / tx;
        if (ty > (uint32_t)kThreads - 2u * tx) ty = (uint32_t)kThreads - 2u * tx;
        if (ty > (uint32_t)ny) ty = (uint32_t)ny;
        ty = cdiv((uint64_t)ny, cdiv((uint64_t)ny, ty));                 // equal rows
        const uint32_t ntx = cdiv((uint64_t)hx, tx), nty = cdiv((uint64_t)ny, ty);
        const double used = (double)hx * ny / ((double)ntx * nty * most);
        const double halo = (2.0 * tx + ty) / ((double)tx * ty);
        const double c = (1.0 + halo / 3.0) / used;
        if (best.tx == 0 || c < cost) {
            cost = c;
            best.tx = tx;
            best.ty = ty;
            best.ntx = ntx;
            best.n = ntx * nty;
            best.entries = (ty + 2u) * tx + ty + 1u;                     // and one spare
        }
    }
    return best;
}

size_t pass_lds_bytes(const DevLattice& d, int spt)
{
    const size_t e = d.precision == 32 ? LdsPlane<float>::bytes_per_entry : LdsPlane<double>::bytes_per_entry;
    const size_t b = 2 * (size_t)pass_geom(d, spt).entries * e;
    return b < 1024 ? 1024 : b;
}

// (the line is that of a window of whole rows, which the pass once kept)
bool pass_shape_ok(int precision, int hx, int spt)
{
    const size_t e = precision == 32 ? LdsPlane<float>::bytes_per_entry : LdsPlane<double>::bytes_per_entry;
    return 2 * ((size_t)kThreads * spt + 2 * (size_t)hx) * e <= kMaxLds;
}

// The per-sweep finalize, one work-group of 1024 threads: all of them sum
// the counts, the first 256 fold the records (or the group sums left by
// fold_groups_kernel in l2).  A lone work-group has no occupancy to gain, so
// the register budget of four waves per SIMD goes to loads in flight.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
void finalize_kernel(DevState* st, const double* part, uint32_t stride, const uint32_t* red, const uint32_t* black,
                     uint32_t nred, uint32_t nblack, uint32_t npart, const double* l2, int fin, double T, double N)
{
    __shared__ double scratch[kFinScratch];
    finalize_body<1024>(st, part, stride, red, black, nred, nblack, npart, l2, fin, T, N, scratch);
}

// Work-group g: the sum S_g of record group g (the order of finalize_body),
// its first nrows components stored at l2[g * kNumPart ..].
__global__ __launch_bounds__(kGroupThreads) void fold_groups_kernel(const double* part, uint32_t stride,
                                                                    uint32_t npart, uint32_t nrows, double* l2)
{
    __shared__ double scratch[5 * kNumPart];
    if (nrows == (uint32_t)kTorqueRows)
        group_sums<kGroupThreads, kTorqueRows>(part, stride, npart, blockIdx.x, blockIdx.x + 1u, scratch,
                                               scratch + 4 * kNumPart);
    else
        group_sums<kGroupThreads, kObsRows>(part, stride, npart, blockIdx.x, blockIdx.x + 1u, scratch,
                                            scratch + 4 * kNumPart);
    if (threadIdx.x < nrows) l2[(size_t)blockIdx.x * kNumPart + threadIdx.x] = scratch[4 * kNumPart + threadIdx.x];
}

// ---------------------------------------------------------------------------
// Set-up of a lattice's workspace: the chain state (zeroed, cone angle
// theta0) and the cone table 1 - cos(theta), both precisions, from values
// passed by argument (so nothing is copied from host memory).
// ---------------------------------------------------------------------------
struct C1Table {
    double d[181];
    float f[181];
};

__global__ __launch_bounds__(kThreads) void setup_kernel(DevState* st, int theta0, const C1Table tab, double* c1d,
                                                         float* c1f)
{
    const uint32_t t = threadIdx.x;
    if (t < 181) {
        c1d[t] = tab.d[t];
        c1f[t] = tab.f[t];
    }
    uint32_t* w = reinterpret_cast<uint32_t*>(st);
    for (uint32_t i = t; i < sizeof(DevState) / 4; i += kThreads) w[i] = 0u;
    __syncthreads();
    if (t == 0) st->theta = theta0;
}

hipError_t launch_setup(const DevLattice& d, const double* c1d_host, int theta0, void* c1_dev, hipStream_t s)
{
    C1Table tab;
    for (int i = 0; i < 181; ++i) {
        tab.d[i] = c1d_host[i];
        tab.f[i] = (float)c1d_host[i];
    }
    double* c1d = static_cast<double*>(c1_dev);
    float* c1f = reinterpret_cast<float*>(c1d + 181);
    setup_kernel<<<1, kThreads, 0, s>>>(d.st, theta0, tab, c1d, c1f);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Initial spins: along a direction, or uniform on the sphere from Philox
// tag 4 (z = 2 u0 - 1, azimuth 2 pi u1).  The sites are dealt to the XCDs as the
// measurement deals them, which follows and finds part of them in its L2 (hmc_init_lattice
// of 128^3 random FP64 44.3 us with sites in launch order, 33.5 so, FP32 33.4 and
// 27.8; MI355X).
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(kThreads) void init_kernel(const KArgs<R> a, int mode, R d0, R d1, R d2,
                                                       double width)
{
    const uint32_t k = xcd_remap(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
    const int c = blockIdx.y;
    if (k >= a.Nc) return;
    V3<R> s{d0, d1, d2};
    if (mode == 2) {
        // one wall across z: the T = 0 profile (sech u, 0, -tanh u)
        const uint32_t z = k / a.P;
        const double u = M_PI * ((double)z - (0.5 * (double)a.nz - 0.5)) / width;
        s = V3<R>{(R)(1.0 / cosh(u)), R(0), (R)(-tanh(u))};
    }
    if (mode == 1) {
        const uint32_t r = k / a.hx;
        const uint32_t y = r % a.ny, z = r / a.ny;
        const uint32_t site = 2u * k + ((y + z + (uint32_t)c) & 1u);
        const Rand4 rn = philox(0u, site, 4u, a.inst, a.key0, a.key1);
        const R zc = R(2) * Prim<R>::u01(rn.r0) - R(1);
        const R rho = Prim<R>::sqrt_(R(1) - zc * zc);
        R sp, cp;
        Prim<R>::sincos_turns(Prim<R>::u01(rn.r1), &sp, &cp);
        s = V3<R>{rho * cp, rho * sp, zc};
    }
    a.s[c][0][k] = s.x;
    a.s[c][1][k] = s.y;
    a.s[c][2][k] = s.z;
}


// ---------------------------------------------------------------------------
// Constrained sweep (Table A2).  A constrained call works on an AoS copy of
// the spins (one 4-vector per site, both colours), made on entry and copied
// back on exit.  Before each colour's pair pass a stencil kernel writes, for
// every site of that colour in site order, a record of its spin and the sum
// of its six neighbours (32 bytes FP32, 64 FP64; the other colour does not
// change during the pass, so the sums are exact).  A pair then needs its two
// records -- the first read in site order, the partner's at a random
// address, the pairing being a random permutation: one cache line per pair
// instead of seven sites -- and writes its new spins into the AoS copy.
// ---------------------------------------------------------------------------
template <typename R> struct Vec4T;
template <> struct Vec4T<float> { using type = float4; };
template <> struct Vec4T<double> { using type = double4; };
template <typename R> using Vec4 = typename Vec4T<R>::type;

template <typename R>
struct Rec {
    Vec4<R> s;    // spin (w unused)
    Vec4<R> nb;   // sum of the six neighbours (other colour)
};

template <typename R>
__device__ __forceinline__ V3<R> v3(const Vec4<R>& q)
{
    return V3<R>{q.x, q.y, q.z};
}

template <typename R>
__device__ __forceinline__ Vec4<R> v4(const V3<R>& v)
{
    Vec4<R> q;
    q.x = v.x;
    q.y = v.y;
    q.z = v.z;
    q.w = R(0);
    return q;
}

#ifndef HMC_PAIR_BLOCKS
#define HMC_PAIR_BLOCKS 512      // most work-groups of the pair pass
#endif
#ifndef HMC_PAIR_TILE_BLOCKS
#define HMC_PAIR_TILE_BLOCKS 2   // blocks of 256 colour indices per pair-pass tile
#endif
constexpr uint32_t kPairTile = HMC_PAIR_TILE_BLOCKS * kThreads;

// the smallest power of two >= n
constexpr uint32_t ring_size(uint32_t n)
{
    uint32_t r = 1;
    while (r < n) r *= 2;
    return r;
}

#ifndef HMC_NB_BLOCKS
#define HMC_NB_BLOCKS 2048       // most work-groups of the record stencil
#endif

// SoA -> AoS (to_aos) or AoS -> SoA, both colours; aos[c * Nc + k].
template <typename R, bool TO_AOS>
__global__ __launch_bounds__(kThreads) void aos_copy_kernel(const KArgs<R> a, Vec4<R>* aos)
{
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
    const int c = blockIdx.y;
    if (k >= a.Nc) return;
    Vec4<R>* q = aos + (size_t)c * a.Nc + k;
    if (TO_AOS) {
        *q = v4<R>(V3<R>{a.s[c][0][k], a.s[c][1][k], a.s[c][2][k]});
    } else {
        const Vec4<R> v = *q;
        a.s[c][0][k] = v.x;
        a.s[c][1][k] = v.y;
        a.s[c][2][k] = v.z;
    }
}

// Colour indices of the six neighbours (other colour) of colour index k of
// colour C, in the order x-, x+, y-, y+, z-, z+.
template <int C>
__device__ __forceinline__ void neighbour_indices(uint32_t k, uint32_t hx, uint32_t ny, uint32_t nz, uint32_t P,
                                                  uint32_t (&nb)[6], bool& zm_wraps, bool& zp_wraps)
{
    const uint32_t kx = k % hx, r = k / hx;
    const uint32_t y = r % ny, z = r / ny;
    const uint32_t p = (y + z + (uint32_t)C) & 1u;
    const uint32_t row = k - kx;
    const uint32_t d = p ? (kx == hx - 1 ? row : k + 1) : (kx == 0 ? row + hx - 1 : k - 1);
    const uint32_t fz = P * z, inpl = kx + hx * y;
    nb[0] = p ? k : d;
    nb[1] = p ? d : k;
    nb[2] = kx + hx * (y == 0 ? ny - 1 : y - 1) + fz;
    nb[3] = kx + hx * (y == ny - 1 ? 0 : y + 1) + fz;
    nb[4] = inpl + P * (z == 0 ? nz - 1 : z - 1);
    nb[5] = inpl + P * (z == nz - 1 ? 0 : z + 1);
    zm_wraps = z == 0;
    zp_wraps = z == nz - 1;
}

// Records of colour C over work-groups b, b + count, ... of the launch:
// site k's spin and the sum of its neighbours (the other colour's AoS spins).
template <typename R, int C>
__device__ __forceinline__ void records_range(const KArgs<R>& a, const Vec4<R>* aos, Rec<R>* rec, uint32_t b,
                                              uint32_t count)
{
    const Vec4<R>* other = aos + (size_t)(1 - C) * a.Nc;
    const Vec4<R>* own = aos + (size_t)C * a.Nc;
    for (uint32_t k = b * kThreads + threadIdx.x; k < a.Nc; k += count * kThreads) {
        uint32_t id[6];
        bool wm, wp;
        neighbour_indices<C>(k, a.hx, a.ny, a.nz, a.P, id, wm, wp);
        V3<R> v[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) v[i] = v3<R>(other[id[i]]);
        if (a.zbound) {
            if (wm) v[4] = across_z(v[4], a.zbound);
            if (wp) v[5] = across_z(v[5], a.zbound);
        }
        if (a.mask[C]) {
            const uint32_t mb = a.mask[C][k];
#pragma unroll
            for (int i = 0; i < 6; ++i)
                if (!((mb >> i) & 1u)) v[i] = V3<R>{R(0), R(0), R(0)};
        }
        const V3<R> nb{((((v[0].x + v[1].x) + v[2].x) + v[3].x) + v[4].x) + v[5].x,
                       ((((v[0].y + v[1].y) + v[2].y) + v[3].y) + v[4].y) + v[5].y,
                       ((((v[0].z + v[1].z) + v[2].z) + v[3].z) + v[4].z) + v[5].z};
        Rec<R> r;
        r.s = own[k];
        r.nb = v4<R>(nb);
        rec[k] = r;
    }
}

template <typename R, int C>
__global__ __launch_bounds__(kThreads) void records_kernel(const KArgs<R> a, const Vec4<R>* aos, Rec<R>* rec)
{
    records_range<R, C>(a, aos, rec, blockIdx.x, gridDim.x);
}

// The end of one constrained sweep and the start of the next in one launch:
// work-group 0 runs the per-sweep finalize (the records of the two pair
// passes, nrec rows each), the others write the colour-0 records of the next
// sweep, which need only the spins.  The finalize and the records touch
// disjoint memory, so the finalize runs in the shadow of the stencil.
template <typename R>
__global__ __launch_bounds__(kThreads) void finalize_records_kernel(const KArgs<R> a, const Vec4<R>* aos, Rec<R>* rec,
                                                                    uint32_t nrec, int fin, double T, double N)
{
    // the pair passes write at most 2 x HMC_PAIR_BLOCKS records: one group
    static_assert(2 * HMC_PAIR_BLOCKS <= kGroupRecords, "the fused finalize folds one group of records");
    __shared__ double scratch[kFinScratch];
    if (blockIdx.x == 0) {
        finalize_body<kThreads>(a.st, a.part, a.cnt_stride, a.cnt, a.cnt + a.cnt_stride, nrec, nrec, 2 * nrec, nullptr, fin, T, N, scratch);
        return;
    }
    records_range<R, 0>(a, aos, rec, blockIdx.x - 1, gridDim.x - 1);
}

// Feistel domain of the shuffle of N_c indices: 2*half bits, the smallest
// even width covering N_c.
struct Shuffle {
    uint32_t half, mask;
};

static inline Shuffle shuffle_for(uint32_t n)
{
    uint32_t bits = 2;
    while (bits < 32 && (1ull << bits) < n) bits += 2;
    Shuffle f;
    f.half = bits / 2;
    f.mask = f.half >= 32 ? 0xFFFFFFFFu : ((1u << f.half) - 1u);
    return f;
}

// Per-sweep constants of a pair pass.
template <typename R>
struct PairCtx {
    Model<R> m;
    V3<R> ec;
    R c1, scale, invML;
    double ML;
    uint32_t sweep, inst, key0, key1;
};

// The pair move of Table A2 on pair k = (i, j) of colour C, with the records
// ri, rj of its two spins: cone move of S_i, compensation of the transverse
// change by S_j (perpendicular to eC; the parallel part from the length),
// M_L ratio and Jacobian, Metropolis test with exp(-(dE_i + dE_j)/T); on
// acceptance both new spins go to the AoS copy.  OBS adds the one-site terms
// of both final spins (and in the black pass their exchange with their final
// red neighbours).
template <typename R, int C, bool OBS, typename A>
__device__ __forceinline__ void pair_move(const PairCtx<R>& x, Vec4<R>* own, uint32_t k, uint32_t ia, uint32_t ja,
                                          const Rec<R>& ri, const Rec<R>& rj, uint32_t& nacc, A& acc)
{
    const Model<R>& m = x.m;
    const V3<R>& ec = x.ec;
    const V3<R> si = v3<R>(ri.s), nbi = v3<R>(ri.nb);
    const V3<R> sj = v3<R>(rj.s), nbj = v3<R>(rj.nb);
    const Rand4 rn = philox(x.sweep, k, 2u + (uint32_t)C, x.inst, x.key0, x.key1);
    const V3<R> ti = cone_move(si, Prim<R>::u01(rn.r0), Prim<R>::u01(rn.r1), x.c1);

    const R pi_old = dot(si, ec), pi_new = dot(ti, ec), pj_old = dot(sj, ec);
    V3<R> pj;
    pj.x = (sj.x - pj_old * ec.x) + (si.x - pi_old * ec.x) - (ti.x - pi_new * ec.x);
    pj.y = (sj.y - pj_old * ec.y) + (si.y - pi_old * ec.y) - (ti.y - pi_new * ec.y);
    pj.z = (sj.z - pj_old * ec.z) + (si.z - pi_old * ec.z) - (ti.z - pi_new * ec.z);
    const R q = dot(sj, sj) - dot(pj, pj);
    bool ok = q > R(0);
    const R pj_new = (pj_old >= R(0) ? R(1) : R(-1)) * Prim<R>::sqrt_(ok ? q : R(1));
    const V3<R> tj{pj.x + pj_new * ec.x, pj.y + pj_new * ec.y, pj.z + pj_new * ec.z};
    // (M_L'/M_L)^2 with M_L' = |M_L| + change along eC
    const R xr = ((pi_new + pj_new) - pi_old - pj_old) * x.invML;
    ok = ok && (R(1) + xr > R(0)) && (x.ML != 0.0);
    const V3<R> hi{m.J * nbi.x + m.h.x, m.J * nbi.y + m.h.y, m.J * nbi.z + m.h.z};
    const V3<R> hj{m.J * nbj.x + m.h.x, m.J * nbj.y + m.h.y, m.J * nbj.z + m.h.z};
    const R dE = delta_e(m, si, ti, hi) + delta_e(m, sj, tj, hj);
    const R ratio = (R(1) + xr) * (R(1) + xr) * fabs(pj_old / pj_new);
    ok = ok && (Prim<R>::u01(rn.r2) < ratio * Prim<R>::boltzmann(dE, x.scale));
    const V3<R> fi = ok ? ti : si;
    const V3<R> fj = ok ? tj : sj;
    if (ok) {
        own[ia] = v4<R>(ti);
        own[ja] = v4<R>(tj);
        nacc += 2;
    }
    if (OBS) {
        if (C == 1) acc.ex += (-m.J * dot(fi, nbi)) + (-m.J * dot(fj, nbj));
        add_site<R, true>(acc, m, fi);
        add_site<R, true>(acc, m, fj);
    }
}

// Pair pass of colour C.  The shuffled order pi of the colour indices is a
// keyed bijection evaluated inline (nothing is stored); pair k is
// (pi(2k), pi(2k+1)) (N_c is even: nx and ny are).  A work-group scans tiles
// of kPairTile consecutive colour indices a (blocks of 256); a is the first
// spin of pair pi^-1(a)/2 when pi^-1(a) is even, and such pairs are queued in
// LDS in scan order (blocks in order, wave ballots, waves in order), so the
// queue never depends on scheduling; a tile takes one ballot round, two
// barriers, for all of its blocks.
// The queue is a ring in LDS drained in rounds of 256 pairs, one per thread,
// and what is left of it stays for the next tile: every lane runs a pair
// move, and the first record of each pair is read near site order (only the
// partner's is a random gather).  M_L is the moment along eC at the
// start of the sweep (one value for both colours, as in the paper).  The sums take
// the one-site terms of both final spins of every pair; since pi is a
// bijection every site is covered once, and in the black pass every bond once
// through its black end.  Results go to row part_base + block (red pass: rows
// 0 .., black pass: rows grid ..).
template <typename R, int C>
__global__ __launch_bounds__(kThreads) void pair_kernel(const KArgs<R> a, Vec4<R>* aos, const Rec<R>* rec,
                                                        const V3<R> ec, const Shuffle f, const R scale,
                                                        const uint32_t part_base)
{
    constexpr uint32_t kU = kPairTile / kThreads;            // indices per thread and tile
    constexpr uint32_t kTrip = kPairTile;                    // indices scanned per tile
    constexpr uint32_t kRing = ring_size(kThreads - 1 + kTrip);  // queue ring: 255 left + kTrip new
    static_assert((kRing & (kRing - 1)) == 0 && kRing >= kThreads - 1 + kTrip, "queue ring too small");
    constexpr int kWaves = kThreads / 64;
    __shared__ uint32_t qa[kRing], qj[kRing], qk[kRing];
    __shared__ double buf[kTorqueRows * kThreads];
    __shared__ uint32_t wtot[kWaves];
    __shared__ uint32_t wcnt[kU][kWaves];
    Vec4<R>* own = aos + (size_t)C * a.Nc;
    PairCtx<R> x;
    x.m = a.m;
    x.ec = ec;
    x.sweep = (uint32_t)a.st->sweep;
    x.c1 = a.c1tab[a.st->theta];
    x.scale = scale;
    const double* M = a.st->M;
    x.ML = M[0] * (double)ec.x + M[1] * (double)ec.y + M[2] * (double)ec.z;
    x.invML = (R)(1.0 / fabs(x.ML));
    x.inst = a.inst;
    x.key0 = a.key0;
    x.key1 = a.key1;
    const Rand4 key = philox(x.sweep, 0u, 5u + (uint32_t)C, a.inst, a.key0, a.key1);

    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t tiles = (a.Nc + kTrip - 1u) / kTrip;
    uint32_t nacc = 0;
    Acc acc;
    Part<R> part;                                            // FP32 spins: the thread's sums, then FP64
    auto& pa = site_acc<R>(acc, part);
    // pairs queued and pairs taken so far, the same in every thread; the
    // queue holds entries head .. tail - 1 at their positions modulo kRing
    uint32_t head = 0, tail = 0;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        uint32_t ia[kU], ja[kU], k[kU];
        bool first[kU];
        uint64_t ball[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            ia[u] = tile * kTrip + u * kThreads + t;
            first[u] = false;
            ja[u] = 0;
            k[u] = 0;
            if (ia[u] < a.Nc) {
                const uint32_t pos = unshuffle_index(ia[u], a.Nc, f.half, f.mask, key);
                first[u] = (pos & 1u) == 0u;
                if (first[u]) {
                    ja[u] = shuffle_index(pos + 1u, a.Nc, f.half, f.mask, key);
                    k[u] = pos >> 1;
                }
            }
            ball[u] = __ballot(first[u]);
            if (lane == 0) wcnt[u][wave] = (uint32_t)__popcll(ball[u]);
        }
        // every wave has left the previous tile's queue reads: the slots past
        // tail are free
        __syncthreads();
        // appended in scan order: index block u = 0 (waves in order), then u = 1
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            uint32_t off = tail, total = tail;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                off += (uint32_t)w < wave ? wcnt[u][w] : 0u;
                total += wcnt[u][w];
            }
            if (first[u]) {
                const uint32_t e = (off + (uint32_t)__popcll(ball[u] & below)) & (kRing - 1u);
                qa[e] = ia[u];
                qj[e] = ja[u];
                qk[e] = k[u];
            }
            tail = total;
        }
        __syncthreads();
        for (; tail - head >= kThreads; head += kThreads) {
            const uint32_t e = (head + t) & (kRing - 1u);
            const uint32_t i = qa[e], j = qj[e];
            pair_move<R, C, true>(x, own, qk[e], i, j, rec[i], rec[j], nacc, pa);
        }
    }
    if (t < tail - head) {
        const uint32_t e = (head + t) & (kRing - 1u);
        const uint32_t i = qa[e], j = qj[e];
        pair_move<R, C, true>(x, own, qk[e], i, j, rec[i], rec[j], nacc, pa);
    }
    flush_part(acc, pa);
    const double v[kTorqueRows] = {acc.M[0], acc.M[1], acc.M[2], acc.ex, acc.eu,
                                   acc.ec,   acc.ez,   acc.tq[0], acc.tq[1], acc.tq[2]};
    // (in place of a wave sum of every row in every wave: a pass 24.4 us for 25.0 at
    // 128^3 FP32, 26.8 for 27.7 at 96^3 FP64; MI355X)
    write_record<kThreads, kTorqueRows>(v, nacc, a.part + part_base + blockIdx.x, a.cnt_stride,
                                        a.cnt + (size_t)C * a.cnt_stride + blockIdx.x, buf, wtot);
}

// ---------------------------------------------------------------------------
// Constrained sweeps of small lattices: one thread per pair, which reads the
// neighbours of both its spins from the AoS copy (cached, at these sizes)
// instead of records, so that a sweep is its two pair passes.  The red pass
// folds the records of the sweep before in every work-group (the moment and
// the counts: all the next sweep needs), while one work-group more does the
// whole finalize; what the passes of a sweep share goes through a slot, and
// slots and records are kept twice, by the parity of the sweep.  What bounds a
// pass is latency: one update deep, a wave to a SIMD.
// ---------------------------------------------------------------------------
template <typename R>
struct PairSlot {
    double ML;
    int32_t theta;
    uint32_t sweep;
    R c1, up, down;      // the cone table at theta and one degree up and down
};
static_assert(offsetof(PairSlot<float>, c1) == 16 && offsetof(PairSlot<double>, c1) == 16, "slot layout");

template <typename R>
struct PairArgs {
    V3<R> ec;
    Shuffle f;
    R scale;
    uint32_t nblk;       // work-groups of a pass; a sweep leaves 2 nblk records
    PairSlot<R>* slot;   // [2]
    uint32_t* cnt;       // [2][2 nblk]
    double* part;        // [2][kTorqueRows][2 nblk]
    uint32_t parity;     // of this sweep in the call
    int32_t first, fin;
    double T, N;
};

// The record (spin, neighbour sum) of colour index k of colour C from the AoS copy.
template <typename R, int C>
__device__ __forceinline__ Rec<R> record_of(const KArgs<R>& a, const Vec4<R>* aos, uint32_t k)
{
    const Vec4<R>* other = aos + (size_t)(1 - C) * a.Nc;
    uint32_t id[6];
    bool wm, wp;
    neighbour_indices<C>(k, a.hx, a.ny, a.nz, a.P, id, wm, wp);
    V3<R> v[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = v3<R>(other[id[i]]);
    Rec<R> r;
    r.s = aos[(size_t)C * a.Nc + k];
    if (a.zbound) {
        if (wm) v[4] = across_z(v[4], a.zbound);
        if (wp) v[5] = across_z(v[5], a.zbound);
    }
    if (a.mask[C]) {
        const uint32_t mb = a.mask[C][k];
#pragma unroll
        for (int i = 0; i < 6; ++i)
            if (!((mb >> i) & 1u)) v[i] = V3<R>{R(0), R(0), R(0)};
    }
    r.nb = v4<R>(V3<R>{((((v[0].x + v[1].x) + v[2].x) + v[3].x) + v[4].x) + v[5].x,
                       ((((v[0].y + v[1].y) + v[2].y) + v[3].y) + v[4].y) + v[5].y,
                       ((((v[0].z + v[1].z) + v[2].z) + v[3].z) + v[4].z) + v[5].z});
    return r;
}

template <typename R, int C>
__global__ __launch_bounds__(kThreads) void pair_direct_kernel(const KArgs<R> a, Vec4<R>* aos, const PairArgs<R> f)
{
    __shared__ double buf[kTorqueRows * kThreads];
    __shared__ double tot[kTorqueRows];
    __shared__ unsigned long long totc;
    __shared__ uint32_t wtot[kThreads / 64];
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, nrec = 2u * f.nblk;
    const uint32_t prev = f.parity ^ 1u;
    const double* before = f.part + (size_t)prev * kTorqueRows * nrec;
    const uint32_t* cnt_before = f.cnt + (size_t)prev * nrec;
    if (C == 0 && blockIdx.x == f.nblk) {
        fold_sweep<kThreads, kTorqueRows>(a.st, before, cnt_before, nrec, f.fin, f.T, f.N, tot, &totc);
        return;
    }
    // what the sweep before left, and the first records of the fold below (all
    // as vector loads, which hold up nothing before their use)
    const bool head = C == 0 && !f.first;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(f.slot + (C == 0 ? prev : f.parity), 0,
                                                                        (int)sizeof(PairSlot<R>), kBufferConfig);
    const double left_ML = Gm<double>::ld(rs, 0u, 0u);
    const int32_t left_theta = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, 8u, 0u, 0);
    const uint32_t left_sweep = __builtin_amdgcn_raw_buffer_load_b32(rs, 12u, 0u, 0);
    constexpr uint32_t rr = sizeof(R);
    const R left_c1 = Gm<R>::ld(rs, 16u, 0u), left_up = Gm<R>::ld(rs, 16u + rr, 0u), left_down = Gm<R>::ld(rs, 16u + 2u * rr, 0u);
    double fq[8];
    uint32_t cq[8];
    if (head) {
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint32_t i = min(u * 64u + lane, nrec - 1u);
            fq[u] = wave < 3 ? before[(size_t)(kMx + wave) * nrec + i] : 0.0;
            cq[u] = wave < 3 ? 0u : cnt_before[i];
        }
    }
    PairCtx<R> x;
    x.m = a.m;
    x.ec = f.ec;
    x.scale = f.scale;
    x.inst = a.inst;
    x.key0 = a.key0;
    x.key1 = a.key1;
    int32_t theta = 0;
    if (C == 0 && f.first) {
        theta = a.st->theta;
        x.sweep = (uint32_t)a.st->sweep;
    } else {
        x.sweep = (uint32_t)__builtin_amdgcn_readfirstlane((int)left_sweep) + (C == 0 ? 1u : 0u);
    }
    // the pair and its records, whose loads pass behind the fold
    const Rand4 key = philox(x.sweep, 0u, 5u + (uint32_t)C, a.inst, a.key0, a.key1);
    const uint32_t k = blockIdx.x * kThreads + t;
    const bool act = k < a.Nc / 2u;
    const uint32_t i = shuffle_index(act ? 2u * k : 0u, a.Nc, f.f.half, f.f.mask, key);
    const uint32_t j = shuffle_index(act ? 2u * k + 1u : 1u, a.Nc, f.f.half, f.f.mask, key);
    const Rec<R> ri = record_of<R, C>(a, aos, i), rj = record_of<R, C>(a, aos, j);
    if (C == 1) {
        x.ML = left_ML;
        x.c1 = left_c1;
    } else {
        double M[3];
        if (f.first) {
            for (int e = 0; e < 3; ++e) M[e] = a.st->M[e];
            x.c1 = a.c1tab[theta];
        } else {
            // the moment and the counts, as fold_sweep folds them (at most 512 records)
            if (wave < 3) {
                double s = 0.0;
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u) s += u * 64u + lane < nrec ? fq[u] : 0.0;
                s = wave_sum(s);
                if (lane == 0) tot[wave] = s;
            } else {
                uint32_t c = 0;
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u) c += u * 64u + lane < nrec ? cq[u] : 0u;
                c = wave_sum(c);
                if (lane == 0) totc = c;
            }
            __syncthreads();
            const bool more = 2.0 * (double)(long long)totc > f.N;
            theta = more ? min(left_theta + 1, 180) : max(left_theta - 1, 1);
            x.c1 = more ? left_up : left_down;
            for (int e = 0; e < 3; ++e) M[e] = tot[e];
        }
        x.ML = M[0] * (double)f.ec.x + M[1] * (double)f.ec.y + M[2] * (double)f.ec.z;
        if (blockIdx.x == 0 && t == 0)
            f.slot[f.parity] = PairSlot<R>{x.ML, theta, x.sweep, x.c1, a.c1tab[min(theta + 1, 180)],
                                           a.c1tab[max(theta - 1, 1)]};
    }
    x.invML = (R)(1.0 / fabs(x.ML));
    uint32_t nacc = 0;
    Acc acc;
    Part<R> part;
    auto& pa = site_acc<R>(acc, part);
    if (act) pair_move<R, C, true>(x, aos + (size_t)C * a.Nc, k, i, j, ri, rj, nacc, pa);
    flush_part(acc, pa);
    const double v[kTorqueRows] = {acc.M[0], acc.M[1], acc.M[2], acc.ex, acc.eu,
                                   acc.ec,   acc.ez,   acc.tq[0], acc.tq[1], acc.tq[2]};
    const uint32_t b = (uint32_t)C * f.nblk + blockIdx.x;
    write_record<kThreads, kTorqueRows>(v, nacc, f.part + (size_t)f.parity * kTorqueRows * nrec + b, nrec,
                                        f.cnt + (size_t)f.parity * nrec + b, buf, wtot);
}

// The finalize of the last sweep of a call.
__global__ __launch_bounds__(kThreads) void pair_direct_finalize_kernel(DevState* st, const double* part,
                                                                        const uint32_t* cnt, uint32_t n, int fin,
                                                                        double T, double N)
{
    __shared__ double tot[kTorqueRows];
    __shared__ unsigned long long totc;
    fold_sweep<kThreads, kTorqueRows>(st, part, cnt, n, fin, T, N, tot, &totc);
}

template <typename R>
__global__ __launch_bounds__(kThreads) void measure_kernel(const KArgs<R> a, const uint32_t zc)
{
    __shared__ double scratch[8 * kNumPart];
    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    Acc acc;
    measure_column<R>(a, zc, b * kThreads + threadIdx.x, acc);
    block_end<R, true>(a, 1, b, 0u, acc, scratch);
}

// Mean spin of every z plane (both colours), for wall profiles: work-group z
// sums the 2P spins of plane z in a fixed order and writes the mean to
// out[3z .. 3z+2].
template <typename R>
__global__ __launch_bounds__(kThreads) void plane_mean_kernel(const KArgs<R> a, double* out)
{
    __shared__ double scratch[5 * 3];
    const Arrays<R> g(a);
    const uint32_t z = blockIdx.x;
    const uint32_t off = a.P * (uint32_t)sizeof(R) * z;
    double v[3] = {0.0, 0.0, 0.0};
    for (uint32_t q = threadIdx.x; q < a.P; q += kThreads) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const V3<R> s = g.get(c, q * (uint32_t)sizeof(R), off);
            v[0] += (double)s.x;
            v[1] += (double)s.y;
            v[2] += (double)s.z;
        }
    }
    block_sum<3>(v, scratch);
    if (threadIdx.x < 3) out[3 * (size_t)z + threadIdx.x] = scratch[threadIdx.x] / (2.0 * (double)a.P);
}

// Spins of sites 2k and 2k + 1 between doubles in site order, S[3 i + a], and the
// component arrays; on the way in each vector is divided by its length (zero
// or non-finite ones are kept), rounded as separate multiplications and
// additions.  The host's loops over sites did this at 0.3 us per hundred
// sites, each way; now the copy over the bus is the time: 96^3 FP32, in and out
// with a measurement between, 4.9 ms before, 2.0 now (MI355X; 1.8 the copies).
template <typename R, bool IN>
__global__ __launch_bounds__(kThreads) void site_order_kernel(const KArgs<R> a, double* xyz)
{
#pragma clang fp contract(off)
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
    if (k >= a.Nc) return;
    const uint32_t r = k / a.hx;
    const uint32_t y = r % a.ny, z = r / a.ny;
#pragma unroll
    for (uint32_t p = 0; p < 2; ++p) {
        double* v = xyz + 6 * (size_t)k + 3 * p;
        const uint32_t c = (y + z + p) & 1u;
        if (IN) {
            const double n2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
            const double inv = (n2 > 0.0 && isfinite(n2)) ? 1.0 / sqrt(n2) : 1.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) (c ? a.s[1][i] : a.s[0][i])[k] = (R)(v[i] * inv);
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i] = (double)(c ? a.s[1][i] : a.s[0][i])[k];
        }
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

template <typename R>
static void site_order_go(const DevLattice& d, double* xyz, bool in, hipStream_t s)
{
    const uint32_t grid = cdiv((uint64_t)d.Nc, kThreads);
    if (in) site_order_kernel<R, true><<<grid, kThreads, 0, s>>>(make_args<R>(d), xyz);
    else site_order_kernel<R, false><<<grid, kThreads, 0, s>>>(make_args<R>(d), xyz);
}

hipError_t launch_site_order(const DevLattice& d, double* xyz, bool in, hipStream_t s)
{
    if (d.precision == 32) site_order_go<float>(d, xyz, in, s);
    else site_order_go<double>(d, xyz, in, s);
    return hipGetLastError();
}

int64_t max_blocks_for(int32_t nx, int32_t ny, int32_t nz)
{
    const uint64_t P = (uint64_t)(nx / 2) * (uint64_t)ny;
    const uint64_t Nc = P * (uint64_t)nz;
    const int64_t pass = (int64_t)cdiv(P, kThreads) * (int64_t)nz;
    const int64_t gather = 2 * (int64_t)cdiv(Nc, kThreads);   // neighbour-sum + pair partials
    return pass > gather ? pass : gather;
}

int64_t pass_blocks(const DevLattice& d, int spt, int zc)
{
    return (int64_t)pass_geom(d, spt).n * (int64_t)cdiv((uint64_t)d.nz, (uint64_t)zc);
}

// The launch shape where none was set.  A step of the march is bound by the
// latency of its loads (about 1.2 us a plane), so a lattice that the last-level
// cache holds takes the shortest slabs whose work-groups still run in one
// round: kRoundBlocks of them (four of 256 threads to a compute unit at FP32,
// two at FP64, whose march holds twice the registers).  One site per thread
// while that leaves short slabs, else two, which share a slab's fixed cost
// (rows above 256 sites, whose tiles are narrow: always one, 1024 x 1024 x 5 with
// masks (1, 5) 51.7 us, (2, 5) 55; 1024 x 512 x 15 (1, 15) 67, (2, 8) 74).
// Measured on MI355X, sampled sweeps, against (2, 16): 32^3 FP32 (1, 1) 13.3
// us for 47.8, 128^3 (1, 4) 27.8 for 51.3, 192^3 (2, 8) 60.7 for 72.6, 256^3
// (2, 16) 110.6 and every other shape above 116; FP64 32^3 (1, 1) 15.3 for
// 72.6, 128^3 (1, 8) 47.3 for 82.5.  Spins that stream from HBM (the
// depth-two march) take 8 planes at FP32 and 32 at FP64: shorter slabs spread
// better (384^3 FP32 2.9 %, 464^3 1.9 % faster than 16 planes), longer ones
// re-read fewer slab ends (256^3 FP64 63.9 G updates/s for 62.8 with 16).
void default_shape(const DevLattice& d, int* spt, int* zc)
{
    const bool wide = !pass_shape_ok(d.precision, d.hx, 2);
    if (pass_deep(d) || (uint64_t)d.N * 3ull * (uint64_t)(d.precision / 8) > kDeepMarchBytes) {
        *spt = wide ? 1 : 2;
        *zc = d.mask ? 16 : (d.precision == 32 ? 8 : 32);
        return;
    }
    constexpr int kRoundBlocks[2] = {1024, 512}, kShortSlab[2] = {4, 8};   // FP32, FP64
    const int p = d.precision == 32 ? 0 : 1;
    for (int s = 1; s <= 2; ++s) {
        const int nqb = (int)pass_geom(d, s).n;
        const int slabs = kRoundBlocks[p] / nqb;                         // as many as one round holds
        const int planes = slabs > 0 ? (int)cdiv((uint64_t)d.nz, (uint64_t)slabs) : d.nz;
        *spt = s;
        *zc = planes < 16 ? planes : 16;
        if (*zc <= kShortSlab[p] || (s == 1 && (wide || geometry_of(d.hx) == 0))) return;
    }
}

// In a batch the other lattices fill the chip, so the slabs are as long as
// re-reading their ends asks for, whatever the batch holds (a lattice's
// result must not depend on its company).  That is a compromise: long slabs leave
// the chip idle where a batch is small, and in (2, 16) a batch that fills exactly
// one round is hard to beat.  Measured on MI355X, us per sampled batch sweep in
// (1, 4), (1, 8), (2, 8) and (2, 16).
//   FP32: 4 x 64^3 21, 27, 38, 62; 24 of 48^3 to 128^3 162, 158, 172, 198; 8 x 128^3
// 116, 113, 117, 109.  Above 128^3 the slabs' ends show: 4 x 160^3 116, 111, 115, 108;
// 2 x 192^3 108, 101, 104, 102; 1 x 224^3 97, 86, 95, 88; 2 x 240^3 244, 231, 248, 262.
// From 14 million spins on a lattice fills the chip alone: 256^3 130, 119, 118, 111.
//   FP64: 4 x 64^3 29, 34, 49, 81 and 16 x 64^3 92, 82, 75, 94, but 32 x 64^3 165, 146,
// 135, 127 (the line is the smaller batches'); 2 x 96^3 50, 45, 55, 90; 16 x 96^3 331, 303,
// 268, 275; 8 x 160^3 756, 684, 591, 573.  Rows of 256 colour sites, where the halo
// of a window is as large as the window: 2 x 512 x 128 x 64 179, 153, 172, 160 and 6 x
// 512 x 64 x 64 323, 296, 291, 278.  Longer ones, in tiles: 4 x 600 x 128 x 64 478, 429, 466,
// 452; 8 x 640 x 64 x 32 202, 178, 203, 226; 1024 x 256 x 32 172, 147 (two sites refused).
void default_batch_shape(const DevLattice& d, int* spt, int* zc)
{
    if ((uint64_t)d.N * 3ull * (uint64_t)(d.precision / 8) > kDeepMarchBytes) {
        default_shape(d, spt, zc);
        return;
    }
    if (d.precision == 32) {
        const bool large = d.N > 14000000;
        *spt = large ? 2 : 1;
        *zc = large ? 16 : (d.N > (int64_t)128 * 128 * 128 ? 8 : 4);
    } else {
        const bool small = d.N <= (int64_t)64 * 64 * 64, tiles = geometry_of(d.hx) == 0;
        *spt = small || tiles ? 1 : 2;
        *zc = small ? 4 : (d.hx < kThreads || tiles ? 8 : 16);
    }
}

// Colour-split bond masks from masks in site order: site i = 2k + p of row
// (y, z) has colour c = (x + y + z) & 1 and colour index k.
__global__ __launch_bounds__(kThreads) void split_masks_kernel(const uint8_t* src, uint8_t* dst, uint32_t Nc,
                                                               uint32_t hx, uint32_t ny)
{
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
    if (k >= Nc) return;
    const uint32_t r = k / hx;
    const uint32_t y = r % ny, z = r / ny;
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c) dst[(size_t)c * Nc + k] = src[2 * (size_t)k + ((y + z + c) & 1u)];
}

hipError_t launch_split_masks(const DevLattice& d, const uint8_t* src, hipStream_t s)
{
    split_masks_kernel<<<cdiv((uint64_t)d.Nc, kThreads), kThreads, 0, s>>>(src, d.mask, (uint32_t)d.Nc,
                                                                             (uint32_t)d.hx, (uint32_t)d.ny);
    return hipGetLastError();
}

hipError_t launch_init(const DevLattice& d, hipStream_t s)
{
    dim3 grid(cdiv((uint64_t)d.Nc, kThreads), 2);
    if (d.precision == 32) {
        auto a = make_args<float>(d);
        init_kernel<float><<<grid, kThreads, 0, s>>>(a, d.init_mode, (float)d.init_dir[0], (float)d.init_dir[1],
                                                     (float)d.init_dir[2], d.init_width);
    } else {
        auto a = make_args<double>(d);
        init_kernel<double><<<grid, kThreads, 0, s>>>(a, d.init_mode, d.init_dir[0], d.init_dir[1], d.init_dir[2],
                                                      d.init_width);
    }
    return hipGetLastError();
}

hipError_t launch_pass(const DevLattice& d, int colour, bool obs, int spt, int zc, double T, const SweepCarry& c,
                       hipStream_t s, int64_t* blocks)
{
    *blocks = pass_blocks(d, spt, zc);
    if (*blocks > d.max_blocks) return hipErrorInvalidValue;
    if (d.mask) return launch_pass_masked(d, colour, obs, spt, zc, T, c, s);
    if (pass_deep(d)) return launch_pass_deep(d, colour, obs, spt, zc, T, c, s);
    return PassLaunch<false, false>::run(d, colour, obs, spt, zc, T, c, s);
}

// What carried sweeps share lies in the two rows of part that no record uses.
uint32_t* red_counts(const DevLattice& d, int sweep)
{
    return sweep & 1 ? reinterpret_cast<uint32_t*>(d.part + (size_t)kTorqueRows * (size_t)d.max_blocks) : d.cnt;
}

PassSlot* carry_slots(const DevLattice& d)
{
    return reinterpret_cast<PassSlot*>(d.part + (size_t)(kTorqueRows + 1) * (size_t)d.max_blocks);
}

// Passes of up to 2048 records: there (masked 1024 x 1024 x 5, one site per thread)
// a sweep still gains 3 us of 52 (MI355X).  In the default shapes more records
// come with lattices whose sweeps take 440 us and more (384^3 FP32), of which a
// finalize is 5, while every work-group would fold more counts.
bool pass_carries(const DevLattice& d, int spt, int zc)
{
    return pass_blocks(d, spt, zc) <= kCarryRecords &&
           2 * sizeof(PassSlot) <= (size_t)d.max_blocks * sizeof(double);
}

template <typename R>
static void constrained_go(const DevLattice& d, int step, const double eC[3], double T, hipStream_t s,
                           int64_t* blocks)
{
    const auto a = make_args<R>(d);
    Vec4<R>* aos = static_cast<Vec4<R>*>(d.aos);
    Rec<R>* rec = reinterpret_cast<Rec<R>*>(aos + 2 * (size_t)d.Nc);
    const uint32_t n = (uint32_t)d.Nc;
    const uint32_t full = cdiv(n, kThreads);
    const uint32_t tiles = cdiv(n, kPairTile);
    const uint32_t pgrid = tiles < (uint32_t)HMC_PAIR_BLOCKS ? tiles : (uint32_t)HMC_PAIR_BLOCKS;
    const uint32_t ngrid = full < (uint32_t)HMC_NB_BLOCKS ? full : (uint32_t)HMC_NB_BLOCKS;
    *blocks = pgrid;
    if (step == kAosIn) {
        aos_copy_kernel<R, true><<<dim3(full, 2), kThreads, 0, s>>>(a, aos);
    } else if (step == kAosOut) {
        aos_copy_kernel<R, false><<<dim3(full, 2), kThreads, 0, s>>>(a, aos);
    } else if (step == kNbRed) {
        records_kernel<R, 0><<<ngrid, kThreads, 0, s>>>(a, aos, rec);
    } else if (step == kNbBlack) {
        records_kernel<R, 1><<<ngrid, kThreads, 0, s>>>(a, aos, rec);
    } else {
        const V3<R> ec{(R)eC[0], (R)eC[1], (R)eC[2]};
        const R scale = Prim<R>::scale_for(T);
        const Shuffle f = shuffle_for(n);
        if (step == kPairRed) pair_kernel<R, 0><<<pgrid, kThreads, 0, s>>>(a, aos, rec, ec, f, scale, 0u);
        else pair_kernel<R, 1><<<pgrid, kThreads, 0, s>>>(a, aos, rec, ec, f, scale, pgrid);
    }
}

hipError_t launch_constrained(const DevLattice& d, int step, const double eC[3], double T, hipStream_t s,
                              int64_t* blocks)
{
    if (d.precision == 32) constrained_go<float>(d, step, eC, T, s, blocks);
    else constrained_go<double>(d, step, eC, T, s, blocks);
    return hipGetLastError();
}

// The scratch of the direct form lies where the records do, behind the AoS copy.
template <typename R>
static PairArgs<R> pair_args(const DevLattice& d, int sweep, const double eC[3], double T, int fin)
{
    PairArgs<R> f;
    f.ec = V3<R>{(R)eC[0], (R)eC[1], (R)eC[2]};
    f.f = shuffle_for((uint32_t)d.Nc);
    f.scale = Prim<R>::scale_for(T);
    f.nblk = cdiv((uint64_t)d.Nc / 2, kThreads);
    f.part = reinterpret_cast<double*>(static_cast<Vec4<R>*>(d.aos) + 2 * (size_t)d.Nc);
    f.slot = reinterpret_cast<PairSlot<R>*>(f.part + 4 * (size_t)kTorqueRows * f.nblk);
    f.cnt = reinterpret_cast<uint32_t*>(f.slot + 2);
    f.parity = (uint32_t)sweep & 1u;
    f.first = sweep == 0;
    f.fin = fin;
    f.T = T;
    f.N = (double)d.N;
    return f;
}

// The direct form up to 64^3 spins: there the lattice's AoS copy stays in the
// L2 caches.  Measured on MI355X, us per sampled sweep, records and queue
// against direct: FP32 16^3 25.8, 14.4; 32^3 21.4, 15.2; 64^3 33.7, 23.8; FP64
// 16^3 28.5, 19.2; 32^3 24.2, 20.7; 64^3 43.5, 29.7.
bool pair_direct(const DevLattice& d)
{
    constexpr int64_t kMost = 64 * 64 * 64;      // spins (512 records: the fold in every work-group takes one round)
    const uint64_t nblk = cdiv((uint64_t)d.Nc / 2, kThreads);
    const uint64_t need = nblk * 4 * (kTorqueRows * sizeof(double) + sizeof(uint32_t)) + 2 * sizeof(PairSlot<double>);
    return d.N <= kMost && need <= (uint64_t)d.Nc * 8 * (uint64_t)(d.precision / 8);
}

template <typename R>
static void pair_direct_go(const DevLattice& d, int colour, int sweep, const double eC[3], double T, int fin, hipStream_t s)
{
    const PairArgs<R> f = pair_args<R>(d, sweep, eC, T, fin);
    const auto a = make_args<R>(d);
    Vec4<R>* aos = static_cast<Vec4<R>*>(d.aos);
    const uint32_t n = 2u * f.nblk;
    if (colour == 0) pair_direct_kernel<R, 0><<<f.nblk + (f.first ? 0u : 1u), kThreads, 0, s>>>(a, aos, f);
    else if (colour == 1) pair_direct_kernel<R, 1><<<f.nblk, kThreads, 0, s>>>(a, aos, f);
    else
        pair_direct_finalize_kernel<<<1, kThreads, 0, s>>>(d.st, f.part + (size_t)f.parity * kTorqueRows * n,
                                                           f.cnt + (size_t)f.parity * n, n, fin, T, f.N);
}

hipError_t launch_pair_direct(const DevLattice& d, int colour, int sweep, const double eC[3], double T, int fin,
                              hipStream_t s)
{
    if (d.precision == 32) pair_direct_go<float>(d, colour, sweep, eC, T, fin, s);
    else pair_direct_go<double>(d, colour, sweep, eC, T, fin, s);
    return hipGetLastError();
}

template <typename R>
static void finalize_records_go(const DevLattice& d, int64_t rec_blocks, int fin, double T, hipStream_t s)
{
    Vec4<R>* aos = static_cast<Vec4<R>*>(d.aos);
    const uint32_t full = cdiv((uint64_t)d.Nc, kThreads);
    const uint32_t ngrid = 1u + (full < (uint32_t)HMC_NB_BLOCKS ? full : (uint32_t)HMC_NB_BLOCKS);
    finalize_records_kernel<R><<<ngrid, kThreads, 0, s>>>(make_args<R>(d), aos,
                                                          reinterpret_cast<Rec<R>*>(aos + 2 * (size_t)d.Nc),
                                                          (uint32_t)rec_blocks, fin, T, (double)d.N);
}

hipError_t launch_finalize_nbsum(const DevLattice& d, int64_t rec_blocks, int fin, double T, hipStream_t s)
{
    if (d.precision == 32) finalize_records_go<float>(d, rec_blocks, fin, T, s);
    else finalize_records_go<double>(d, rec_blocks, fin, T, s);
    return hipGetLastError();
}

hipError_t launch_plane_means(const DevLattice& d, double* out, hipStream_t s)
{
    if (d.precision == 32) plane_mean_kernel<float><<<d.nz, kThreads, 0, s>>>(make_args<float>(d), out);
    else plane_mean_kernel<double><<<d.nz, kThreads, 0, s>>>(make_args<double>(d), out);
    return hipGetLastError();
}

// Planes per thread of the measurement: the shortest slabs that give 512
// work-groups at most, which shares the work-group sums where the chip is not
// filled anyway; above eight planes the shortest that give 2048 (eight to a
// compute unit).  Planes of a few sites take one plane a thread: columns shorter
// than a 32-byte sector would scatter a wave's loads over as many lines as it has
// slabs (MI355X, us per hmc_observables in slabs and so: 2 x 2 x 4000000 FP32 383,
// 119, FP64 380, 158; 2 x 6 x 700000 FP32 87, 77; at the line 4 x 4 x 1000000 FP32 98,
// 120, 2 x 4 x 1000000 FP64 88, 89).  The rule depends on the lattice alone:
// hmc_measure_static and a batch measure with the same grid, so with the same bits.
int measure_planes(const DevLattice& d)
{
    if (d.P * (d.precision / 8) < 32) return 1;
    auto planes = [&](uint64_t blocks) {
        const uint64_t slabs = blocks * kThreads / (uint64_t)d.P;
        return slabs == 0 ? d.nz : (int)cdiv((uint64_t)d.nz, slabs);
    };
    const int few = planes(512), many = planes(2048);
    return few <= 8 ? few : (many > 8 ? many : 8);
}

int64_t measure_blocks(const DevLattice& d)
{
    return (int64_t)cdiv((uint64_t)d.P * cdiv((uint64_t)d.nz, (uint64_t)measure_planes(d)), kThreads);
}

hipError_t launch_measure(const DevLattice& d, hipStream_t s, int64_t* blocks)
{
    const uint32_t grid = (uint32_t)measure_blocks(d), zc = (uint32_t)measure_planes(d);
    if (d.precision == 32) measure_kernel<float><<<grid, kThreads, 0, s>>>(make_args<float>(d), zc);
    else measure_kernel<double><<<grid, kThreads, 0, s>>>(make_args<double>(d), zc);
    *blocks = grid;
    return hipGetLastError();
}

hipError_t launch_finalize(const DevLattice& d, int64_t red_blocks, int64_t black_blocks, int64_t part_blocks,
                           int fin, double T, hipStream_t s, int sweep)
{
    const uint32_t stride = (uint32_t)d.max_blocks;
    const uint32_t G = (uint32_t)cdiv((uint64_t)part_blocks, (uint64_t)kGroupRecords);
    const double* l2 = nullptr;
    if ((fin & kFinObs) && G > kFinGroupsInKernel) {
        // the group sums, in parallel, into the space after the partial rows
        double* g2 = d.part + (size_t)kNumPart * stride;
        const uint32_t nrows = (fin & kFinTorque) ? (uint32_t)kTorqueRows : (uint32_t)kObsRows;
        fold_groups_kernel<<<G, kGroupThreads, 0, s>>>(d.part, stride, (uint32_t)part_blocks, nrows, g2);
        l2 = g2;
    }
    finalize_kernel<<<1, 1024, 0, s>>>(d.st, d.part, stride, red_counts(d, sweep), d.cnt + stride,
                                       (uint32_t)red_blocks, (uint32_t)black_blocks, (uint32_t)part_blocks, l2, fin,
                                       T, (double)d.N);
    return hipGetLastError();
}

}  // namespace hmc
