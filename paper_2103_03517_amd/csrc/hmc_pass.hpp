// hmc_pass.hpp -- device code shared by the kernel translation units:
// kernel arguments, buffer-resource access, LDS planes, fixed-order
// reductions, the per-sweep finalize and the tile of the standard colour
// pass (hmc_kernels.hip launches it for one lattice, hmc_batch_kernels.hip
// for a batch).
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
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include "hmc_device.hpp"
#include "hmc_internal.h"

namespace hmc {

constexpr int32_t kBufferConfig = 0x00020000;   // raw buffer, gfx9-family data format

template <typename R>
struct KArgs {
    R* s[2][3];
    uint32_t hx, ny, nz, P, Nc;
    uint32_t arr_bytes;  // bytes of one component array (range of the buffer resources)
    Model<R> m;
    uint32_t key0, key1, inst;
    DevState* st;
    const R* c1tab;
    double* part;
    uint32_t* cnt;       // [2][cnt_stride]
    uint32_t cnt_stride; // row stride of cnt and of part ([kNumPart][cnt_stride] doubles)
    uint32_t zbound;     // z boundary: 0 periodic, 1 anti-periodic, 2 open
    const uint8_t* mask[2];  // per colour, Nc bytes of active-bond bits (x-, x+, y-, y+, z-, z+), or null
};

template <typename R>
static KArgs<R> make_args(const DevLattice& d)
{
    KArgs<R> a;
    char* base = static_cast<char*>(d.spins);
    for (int c = 0; c < 2; ++c)
        for (int k = 0; k < 3; ++k) a.s[c][k] = reinterpret_cast<R*>(base + (size_t)(3 * c + k) * d.pitch);
    a.hx = (uint32_t)d.hx;
    a.ny = (uint32_t)d.ny;
    a.nz = (uint32_t)d.nz;
    a.P = (uint32_t)d.P;
    a.Nc = (uint32_t)d.Nc;
    a.arr_bytes = (uint32_t)((uint64_t)d.Nc * sizeof(R));
    a.m.J = (R)d.J;
    a.m.Ku = (R)d.Ku;
    a.m.Kc = (R)d.Kc;
    a.m.e = V3<R>{(R)d.eu[0], (R)d.eu[1], (R)d.eu[2]};
    a.m.h = V3<R>{(R)d.h[0], (R)d.h[1], (R)d.h[2]};
    a.key0 = d.key0;
    a.key1 = d.key1;
    a.inst = d.instance;
    a.st = d.st;
    a.c1tab = static_cast<const R*>(d.c1tab);
    a.part = d.part;
    a.cnt = d.cnt;
    a.cnt_stride = (uint32_t)d.max_blocks;
    a.zbound = (uint32_t)d.zbound;
    a.mask[0] = d.mask;
    a.mask[1] = d.mask ? d.mask + d.Nc : nullptr;
    return a;
}

// One lattice of a batch (device table, filled on the host by
// batch_fill_entry): its kernel arguments and its launch shape.
template <typename R>
struct BatchEntry {
    KArgs<R> a;
    PassGeom geom;       // in-plane tiles of the colour pass
    uint32_t zc, nblk;
    uint32_t mzc;        // planes per thread of the measurement
    double N;
};

// ---------------------------------------------------------------------------
// Buffer-resource access to the six component arrays.
// ---------------------------------------------------------------------------
template <typename R> struct Gm;

template <> struct Gm<float> {
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float v)
    {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, 0);
    }
};

template <> struct Gm<double> {
    static __device__ __forceinline__ double ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
    {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, double v)
    {
        using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0u, 0u, 0));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, 0);
    }
};

template <typename R>
__device__ __forceinline__ V3<R> neg(const V3<R>& v)
{
    return V3<R>{-v.x, -v.y, -v.z};
}

// A neighbour seen across the z boundary: its sign flipped (anti-periodic,
// zbound 1) or no bond at all (open, zbound 2).
template <typename R>
__device__ __forceinline__ V3<R> across_z(const V3<R>& v, uint32_t zbound)
{
    return zbound == 1 ? neg(v) : V3<R>{R(0), R(0), R(0)};
}

template <typename R>
struct Arrays {
    __amdgpu_buffer_rsrc_t r[2][3];
    __device__ __forceinline__ explicit Arrays(const KArgs<R>& a)
    {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                r[c][k] = __builtin_amdgcn_make_buffer_rsrc(a.s[c][k], 0, (int)a.arr_bytes, kBufferConfig);
    }
    // spin of colour c at byte offset voff + soff
    __device__ __forceinline__ V3<R> get(int c, uint32_t voff, uint32_t soff) const
    {
        return V3<R>{Gm<R>::ld(r[c][0], voff, soff), Gm<R>::ld(r[c][1], voff, soff), Gm<R>::ld(r[c][2], voff, soff)};
    }
    __device__ __forceinline__ void put(int c, uint32_t voff, uint32_t soff, const V3<R>& v) const
    {
        Gm<R>::st(r[c][0], voff, soff, v.x);
        Gm<R>::st(r[c][1], voff, soff, v.y);
        Gm<R>::st(r[c][2], voff, soff, v.z);
    }
};

// ---------------------------------------------------------------------------
// LDS plane of the other colour: float4 entries for FP32 (one 16-byte access
// per neighbour), three component planes for FP64.
// ---------------------------------------------------------------------------
template <typename R> struct LdsPlane;

template <> struct LdsPlane<float> {
    static constexpr size_t bytes_per_entry = 16;
    static __device__ __forceinline__ void put(unsigned char* p, uint32_t W, uint32_t e, const V3<float>& v)
    {
        (void)W;
        reinterpret_cast<float4*>(p)[e] = make_float4(v.x, v.y, v.z, 0.0f);
    }
    static __device__ __forceinline__ V3<float> get(const unsigned char* p, uint32_t W, uint32_t e)
    {
        (void)W;
        const float4 q = reinterpret_cast<const float4*>(p)[e];
        return V3<float>{q.x, q.y, q.z};
    }
};

template <> struct LdsPlane<double> {
    static constexpr size_t bytes_per_entry = 24;
    static __device__ __forceinline__ void put(unsigned char* p, uint32_t W, uint32_t e, const V3<double>& v)
    {
        double* d = reinterpret_cast<double*>(p);
        d[e] = v.x;
        d[W + e] = v.y;
        d[2 * W + e] = v.z;
    }
    static __device__ __forceinline__ V3<double> get(const unsigned char* p, uint32_t W, uint32_t e)
    {
        const double* d = reinterpret_cast<const double*>(p);
        return V3<double>{d[e], d[W + e], d[2 * W + e]};
    }
};

static inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Work-groups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Renumber them so that XCD x receives one contiguous range of logical
// tiles: neighbouring tiles, whose halos overlap, then share an L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nblk)
{
    const uint32_t per = nblk >> 3, rem = nblk & 7u;
    const uint32_t x = b & 7u, i = b >> 3;
    return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

// ---------------------------------------------------------------------------
// Fixed-order reductions.  Within a wave a DPP tree, across the four waves
// of a work-group in wave order, across work-groups by the finalize kernel in
// the order set out at finalize_body.  The results therefore do not depend
// on scheduling.
// ---------------------------------------------------------------------------
// Cross-lane moves for the wave sum: DPP row operations (gfx9 encodings),
// which run on the vector ALU instead of the LDS crossbar.
constexpr int kDppQuadSwap1 = 0xB1;        // quad_perm [1,0,3,2]: lane i takes lane i ^ 1
constexpr int kDppQuadSwap2 = 0x4E;        // quad_perm [2,3,0,1]: lane i takes lane i ^ 2
constexpr int kDppRowHalfMirror = 0x141;   // lane i takes lane 7 - i within its 8-lane half-row
constexpr int kDppRowMirror = 0x140;       // lane i takes lane 15 - i within its 16-lane row

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}

template <int CTRL, typename T>
__device__ __forceinline__ T dpp_move(T v)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit values");
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp_u32<CTRL>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = dpp_u32<CTRL>((uint32_t)u), hi = dpp_u32<CTRL>((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, lo | (hi << 32));
    }
}

template <typename T>
__device__ __forceinline__ T read_lane(T v, int lane)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane((int)__builtin_bit_cast(uint32_t, v), lane));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
        return __builtin_bit_cast(T, lo | (hi << 32));
    }
}

// Sum over the 64 lanes of a wave (all lanes active), the same on every
// lane: pairs, quads, half-rows and rows by DPP moves (at each step the two
// lanes of a pair add the same two values, so they hold the same sum), then
// the four row sums as (row0 + row1) + (row2 + row3).
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
    v += dpp_move<kDppQuadSwap1>(v);
    v += dpp_move<kDppQuadSwap2>(v);
    v += dpp_move<kDppRowHalfMirror>(v);
    v += dpp_move<kDppRowMirror>(v);
    const T r0 = read_lane(v, 0), r1 = read_lane(v, 16), r2 = read_lane(v, 32), r3 = read_lane(v, 48);
    return (r0 + r1) + (r2 + r3);
}

// Sums NV values over the work-group; the totals land in scratch[0..NV).
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* scratch)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
    __syncthreads();
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < NV; ++i) scratch[NV + wave * NV + i] = v[i];
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += scratch[NV + w * NV + threadIdx.x];
        scratch[threadIdx.x] = s;
    }
    __syncthreads();
}

// The end of a producing launch: work-group b writes its acceptance count
// and (OBS) its partial sums, component e at part[e * cnt_stride + b] (one
// row per component, so the finalize reads each row coalesced): the moment
// and the energies, and with TQ the torque.  They are reduced by
// finalize_kernel, launched next on the same stream (the kernel boundary
// makes them visible).  scratch: at least 5 * kTorqueRows + 2 doubles.
template <typename R, bool OBS, bool TQ = true>
__device__ __forceinline__ void block_end(const KArgs<R>& a, int colour, uint32_t b, uint32_t nacc, const Acc& acc,
                                          double* scratch)
{
    if (OBS) {
        constexpr int NV = TQ ? kTorqueRows : kObsRows;
        double v[NV];
        v[kMx] = acc.M[0];
        v[kMy] = acc.M[1];
        v[kMz] = acc.M[2];
        v[kEexch] = acc.ex;
        v[kEuni] = acc.eu;
        v[kEcub] = acc.ec;
        v[kEzee] = acc.ez;
        if constexpr (TQ) {
            v[kTx] = acc.tq[0];
            v[kTy] = acc.tq[1];
            v[kTz] = acc.tq[2];
        }
        // the count as an integer, its wave sums published by block_sum's barriers
        uint32_t* s32 = reinterpret_cast<uint32_t*>(scratch + 5 * NV);
        const uint32_t c = wave_sum(nacc);
        if ((threadIdx.x & 63) == 0) s32[threadIdx.x >> 6] = c;
        block_sum<NV>(v, scratch);
        if (threadIdx.x < (uint32_t)NV) a.part[(size_t)threadIdx.x * a.cnt_stride + b] = scratch[threadIdx.x];
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int w = 0; w < kThreads / 64; ++w) tot += s32[w];
            a.cnt[(size_t)colour * a.cnt_stride + b] = tot;
        }
    } else {
        uint32_t c = wave_sum(nacc);
        __syncthreads();
        uint32_t* s32 = reinterpret_cast<uint32_t*>(scratch);
        if ((threadIdx.x & 63) == 0) s32[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int w = 0; w < kThreads / 64; ++w) tot += s32[w];
            a.cnt[(size_t)colour * a.cnt_stride + b] = tot;
        }
    }
}

// ---------------------------------------------------------------------------
// Per-sweep finalize: the fixed-order reduction of the work-group results of
// the colour-1 (and, for the counts, colour-0) launch, then Table A1's
// cone-angle rule (one degree up when accepted/N > 1/2, else down, within
// [1, 180]), the sweep counter and on sampled sweeps the shifted FP64
// accumulators of Eq. 6.
//
// The records are folded in one order, whichever kernel folds them.  They
// form groups of 1024 (group g: records 1024g .. 1024g + 1023).  In a group,
// thread t of 256 adds records 1024g + t, + 256, + 512 and + 768 in turn
// (from 0.0); wave_sum adds the threads of each wave and the four wave sums
// are added in wave order (from 0.0), giving the group sum S_g.  The total is
// ((0.0 + S_0) + S_1) + ... .  A group is one round of loads (4 per folded row
// and thread: the 7 rows of M and the energies, 10 with the torque).
// With more than one group the single-lattice path forms the group sums in
// parallel (fold_groups_kernel, one work-group per group) and the finalize
// adds them; the batch and constrained finalizes form them one after the
// other (a 1024-thread work-group would form four per round).
// The counts are integers, summed in any order.
// ---------------------------------------------------------------------------
constexpr int kGroupRecords = 1024;
constexpr int kGroupThreads = 256;
// doubles of shared memory finalize_body needs: the wave sums [16][kNumPart],
// the group sums of a round [4][kNumPart], the totals [kNumPart + 1] and the
// per-wave counts [16]
constexpr int kFinScratch = 16 * kNumPart + 4 * kNumPart + kNumPart + 1 + 16;
// group sums the single-lattice finalize forms itself; above this,
// fold_groups_kernel forms them in parallel first.  One work-group reading
// several groups is bound by what one CU can fetch (measured on MI355X: 24
// us for the 7 groups of a 384^3 pass with 8-plane chunks, against 13 us
// with the parallel fold), so the finalize takes one group at most.
constexpr uint32_t kFinGroupsInKernel = 1;

// The group sums S_g of groups g0, g0 + 1, ... (those below G), one group
// per 256 threads of the work-group, into sg[j * kNumPart ..] for group
// g0 + j (shared memory; wsum holds [NT / 64][kNumPart]).  Every thread of
// the work-group calls it (it holds barriers).
template <int NT, int NR>
__device__ __forceinline__ void group_sums(const double* part, uint32_t stride, uint32_t npart, uint32_t g0,
                                           uint32_t G, double* wsum, double* sg)
{
    constexpr int PG = NT / kGroupThreads;
    const uint32_t t = threadIdx.x, tl = t % (uint32_t)kGroupThreads;
    const uint32_t g = g0 + t / (uint32_t)kGroupThreads;
    if (g < G) {                       // uniform over each 256 threads (whole waves)
        const uint32_t r0 = g * (uint32_t)kGroupRecords + tl;
        double q[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t r = r0 + (uint32_t)(u * kGroupThreads);
            const double* p = part + (r < npart ? r : 0u);     // record 0 always exists
#pragma unroll
            for (int e = 0; e < NR; ++e) q[u][e] = p[(size_t)e * stride];
        }
        // a record past the end adds +0.0, which changes no sum (no partial
        // sum here is ever -0.0), so the loads need no branch
        double v[NR];
#pragma unroll
        for (int e = 0; e < NR; ++e) v[e] = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = r0 + (uint32_t)(u * kGroupThreads) < npart;
#pragma unroll
            for (int e = 0; e < NR; ++e) v[e] += in ? q[u][e] : 0.0;
        }
        // all wave sums first, then one branch for the stores
#pragma unroll
        for (int e = 0; e < NR; ++e) v[e] = wave_sum(v[e]);
        if ((t & 63u) == 0) {
#pragma unroll
            for (int e = 0; e < NR; ++e) wsum[(t >> 6) * kNumPart + e] = v[e];
        }
    }
    __syncthreads();
    if (t < (uint32_t)(PG * NR)) {
        const uint32_t j = t / (uint32_t)NR, e = t % (uint32_t)NR;
        if (g0 + j < G) {
            double x = 0.0;
            for (int w = 0; w < kGroupThreads / 64; ++w)
                x += wsum[((int)j * (kGroupThreads / 64) + w) * kNumPart + (int)e];
            sg[j * kNumPart + e] = x;
        }
    }
    __syncthreads();
}

// The old chain state, one value of each kind per lane of a wave: accumulator i
// in lanes 0..4, that of the anisotropy energy in lane 5, of the torque in
// lanes 7..9; and its update from the totals of a sweep or a measurement by that
// wave.  Read early, it waits with the records' loads.  (One thread's chain of
// loads, divisions and stores took 7000 cycles of a finalize: 13000 for 6000 in
// the launch of a whole 16^3 sweep, MI355X.)
struct StateLanes {
    double shift, sum, sum2;
    int64_t samples, torque_samples, sweep;
    int32_t theta;
    __device__ __forceinline__ void read(const DevState* st)
    {
        const uint32_t lane = threadIdx.x & 63u, i = min(lane, 4u);
        shift = st->shift[i];
        sum = lane == 5 ? st->sum_eanis : (lane >= 7 ? st->sum_torque[min(lane - 7u, 2u)] : st->sum[i]);
        sum2 = st->sum2[i];
        samples = st->samples;
        torque_samples = st->torque_samples;
        theta = st->theta;
        sweep = st->sweep;
    }
    // tot: the totals of the NR folded rows; accepted: with kFinCounts
    template <int NR>
    __device__ __forceinline__ void update(DevState* st, const double* tot, long long accepted, int fin, double T,
                                           double N) const
    {
        const uint32_t lane = threadIdx.x & 63u;
        if ((fin & kFinCounts) && lane == 0) {
            st->accepted_last = accepted;
            if (2.0 * (double)accepted > N) st->theta = theta < 180 ? theta + 1 : theta;
            else st->theta = theta > 1 ? theta - 1 : theta;
            st->sweep = sweep + 1;
        }
        if (!(fin & kFinObs)) return;
        const double row = tot[min(lane, (uint32_t)NR - 1u)];
        if (__ballot(!isfinite(row)) && lane == 0) st->nonfinite = 1;
        double* inst = st->M;                        // M[3], the four energies, the torque[3]
        if (lane < (uint32_t)NR) inst[lane] = row;
        if (!(fin & kFinSample)) return;
        // lane 1, 2, 3: m_x, m_y, m_z; lane 4: E/N; lane 5: (E_uni + E_cub)/N; lanes
        // 7..9: the torque; lane 0: |m|
        double num = lane < 4 ? tot[lane == 0 ? 0u : lane - 1u] : row;
        if (lane == 4) num = tot[kEexch] + tot[kEuni] + tot[kEcub] + tot[kEzee];
        if (lane == 5) num = tot[kEuni] + tot[kEcub];
        double x = num / N;
        const double mx = read_lane(x, 1), my = read_lane(x, 2), mz = read_lane(x, 3);
        const double ml = sqrt(mx * mx + my * my + mz * mz);
        if (lane == 0) x = ml;
        if (lane < 5) {
            const double sh = samples == 0 ? x : shift, d = x - sh;
            if (samples == 0) st->shift[lane] = x;
            st->sum[lane] = sum + d;
            st->sum2[lane] = sum2 + d * d;
        } else if (lane == 5) {
            st->sum_eanis = sum + x;
        } else if (lane == 6) {
            st->samples = samples + 1;
            st->T_sample = T;
            if (NR == kTorqueRows) st->torque_samples = torque_samples + 1;
        } else if (NR == kTorqueRows && lane < 10) {
            st->sum_torque[lane - 7u] = sum + x;
        }
    }
};
static_assert(offsetof(DevState, E_exch) == offsetof(DevState, M) + 24 && offsetof(DevState, E_zee) == offsetof(DevState, M) + 48 &&
                  offsetof(DevState, torque) == offsetof(DevState, M) + 56,
              "M, the energies and the torque lie in the order of the rows");

// The finalize of one lattice by one work-group of NT threads (256 or 1024).
// stride: row stride of part; red, black: the counts of the passes; l2: the group sums computed by
// fold_groups_kernel ([G][kNumPart]), or null when this work-group computes
// them.
template <int NT>
__device__ __forceinline__ void finalize_body(DevState* st, const double* part, uint32_t stride,
                                              const uint32_t* red, const uint32_t* black, uint32_t nred, uint32_t nblack, uint32_t npart, const double* l2,
                                              int fin, double T, double N, double* scratch)
{
    static_assert(NT >= kGroupThreads && NT % 64 == 0 && NT <= 1024, "work-group size");
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    double* wsum = scratch;                                                   // [16][kNumPart]
    double* sg = scratch + 16 * kNumPart;                                     // [4][kNumPart]
    double* tot = sg + 4 * kNumPart;                                          // [kNumPart + 1]
    unsigned long long* wc = reinterpret_cast<unsigned long long*>(tot + kNumPart + 1);   // [NT / 64]
    StateLanes old;
    if (wave == 0) old.read(st);
    if (fin & kFinCounts) {
        // integer sums: any order gives the same total; eight loads in flight
        constexpr int UC = 8;
        const uint32_t nc = nred + nblack;
        unsigned long long c = 0;
        for (uint32_t i = t; i < nc; i += UC * NT) {
            uint32_t w[UC];
#pragma unroll
            for (int u = 0; u < UC; ++u) {
                const uint32_t j = i + (uint32_t)u * NT;
                const uint32_t jj = j < nc ? j : i;                    // always in range
                const uint32_t x = jj < nred ? red[jj] : black[jj - nred];
                w[u] = j < nc ? x : 0u;
            }
#pragma unroll
            for (int u = 0; u < UC; ++u) c += w[u];
        }
        c = wave_sum(c);
        if (lane == 0) wc[wave] = c;
    }
    if (fin & kFinObs) {
        const uint32_t G = (npart + (uint32_t)kGroupRecords - 1u) / (uint32_t)kGroupRecords;
        const bool torque = (fin & kFinTorque) != 0;
        const uint32_t nrows = torque ? (uint32_t)kTorqueRows : (uint32_t)kObsRows;
        if (l2 != nullptr) {
            if (t < (uint32_t)kNumPart) {
                double x = 0.0;
                if (t < nrows)
                    for (uint32_t g = 0; g < G; ++g) x += l2[(size_t)g * kNumPart + t];
                tot[t] = x;
            }
        } else {
            // rounds of NT / 256 groups formed side by side, added in order
            constexpr uint32_t PG = NT / kGroupThreads;
            double run = 0.0;          // threads 0..nrows-1: the running total
            for (uint32_t g0 = 0; g0 < G; g0 += PG) {
                if (torque) group_sums<NT, kTorqueRows>(part, stride, npart, g0, G, wsum, sg);
                else group_sums<NT, kObsRows>(part, stride, npart, g0, G, wsum, sg);
                if (t < nrows)
                    for (uint32_t j = 0; j < PG && g0 + j < G; ++j) run += sg[j * kNumPart + t];
            }
            if (t < (uint32_t)kNumPart) tot[t] = run;
        }
    }
    __syncthreads();
    if (wave != 0) return;
    unsigned long long c = 0;
    if (fin & kFinCounts)
        for (int w = 0; w < NT / 64; ++w) c += wc[w];
    if (fin & kFinTorque) old.update<kTorqueRows>(st, tot, (long long)c, fin, T, N);
    else old.update<kObsRows>(st, tot, (long long)c, fin, T, N);
}

// ---------------------------------------------------------------------------
// The finalize where a launch folds the records of the sweep before beside its
// own work (hmc_sweep_kernels.hip, pair_direct_kernel).
// ---------------------------------------------------------------------------
// Row `row` of n records, by one wave: lane l adds records l, l + 64, ..., then
// the lanes are summed.
__device__ __forceinline__ double fold_row(const double* part, uint32_t row, uint32_t n)
{
    const uint32_t lane = threadIdx.x & 63u;
    const double* p = part + (size_t)row * n;
    double x = 0.0;
    for (uint32_t i0 = 0; i0 < n; i0 += 512u) {
        double q[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) q[u] = p[min(i0 + u * 64u + lane, n - 1u)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) x += i0 + u * 64u + lane < n ? q[u] : 0.0;
    }
    return wave_sum(x);
}

// The counts of n records, by one wave.
__device__ __forceinline__ unsigned long long fold_counts(const uint32_t* cnt, uint32_t n)
{
    unsigned long long c = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 512u) {
        uint32_t q[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) q[u] = cnt[min(i0 + u * 64u + (threadIdx.x & 63u), n - 1u)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) c += i0 + u * 64u + (threadIdx.x & 63u) < n ? q[u] : 0u;
    }
    return wave_sum(c);
}

// The record of a work-group of NT threads: its NV sums, row e at
// row0[e * stride], and its count.  The values change places in LDS (buf: NV * NT
// doubles, free on entry), a wave then sums a row: where a launch is one
// update deep, a tree for every row in every wave (block_sum) was a tenth of it
// (2400 of 23000 cycles of a pair pass at 32^3, MI355X).
template <int NT, int NV>
__device__ __forceinline__ void write_record(const double (&v)[NV], uint32_t nacc, double* row0, size_t stride,
                                             uint32_t* cnt, double* buf, uint32_t* wtot)
{
    constexpr uint32_t NW = NT / 64;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
#pragma unroll
    for (int e = 0; e < NV; ++e) buf[e * NT + t] = v[e];
    const uint32_t c = wave_sum(nacc);
    if (lane == 0) wtot[wave] = c;
    __syncthreads();
#pragma unroll
    for (uint32_t e0 = 0; e0 < (uint32_t)NV; e0 += NW) {
        const uint32_t e = e0 + wave;
        if (e < (uint32_t)NV) {
            double x = 0.0;
#pragma unroll
            for (uint32_t u = 0; u < NW; ++u) x += buf[e * NT + u * 64u + lane];
            x = wave_sum(x);
            if (lane == 0) row0[e * stride] = x;
        }
    }
    if (t == (uint32_t)NT - 1) {
        uint32_t tot = 0;
        for (uint32_t w = 0; w < NW; ++w) tot += wtot[w];
        *cnt = tot;
    }
}

// The finalize of a sweep by a work-group of NT threads: theta rule, sweep
// counter, and by the flags the observables, the torque and the accumulators.
// A wave folds a row (row(e): its sum) or the counts (counts()).  tot: NR doubles
// and totc in shared memory.
template <int NT, int NR, typename Row, typename Counts>
__device__ __forceinline__ void fold_sweep(DevState* st, int fin, double T, double N, double* tot,
                                           unsigned long long* totc, Row row, Counts counts)
{
    constexpr uint32_t NW = NT / 64;
    static_assert(NR == kObsRows || NR == kTorqueRows, "rows of a record");
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    StateLanes old;
    if (wave == 0) old.read(st);
    for (uint32_t e = wave; e <= (uint32_t)NR; e += NW) {
        if (e == (uint32_t)NR) {
            const unsigned long long c = counts();
            if (lane == 0) *totc = c;
        } else if (fin & kFinObs) {
            const double x = row(e);
            if (lane == 0) tot[e] = x;
        }
    }
    __syncthreads();
    if (wave == 0) old.update<NR>(st, tot, (long long)*totc, fin, T, N);
}

// ... from n records: rows of n partials and a row of counts.
template <int NT, int NR>
__device__ __forceinline__ void fold_sweep(DevState* st, const double* part, const uint32_t* cnt, uint32_t n, int fin,
                                           double T, double N, double* tot, unsigned long long* totc)
{
    fold_sweep<NT, NR>(st, fin, T, N, tot, totc, [&](uint32_t e) { return fold_row(part, e, n); },
                       [&] { return fold_counts(cnt, n); });
}

// Records of a row through a buffer resource of its length: what lies past the
// end reads as zero, which changes no sum.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const T* p, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, (int)(n * (uint32_t)sizeof(T)), kBufferConfig);
}

constexpr int kCarryRecords = 2048;

// The total of the n records at p, by one wave: the order of finalize_body,
// whose 256 threads a wave stands for in four steps.  (Eight loads in flight: the
// pass this is part of has no registers for more.)
__device__ __forceinline__ double fold_groups(const double* p, uint32_t n)
{
    const __amdgpu_buffer_rsrc_t r = row_rsrc(p, n);
    const uint32_t lane = threadIdx.x & 63u;
    double total = 0.0, sum = 0.0;
#pragma unroll 1
    for (uint32_t w0 = 0; w0 < 4u * ((n + kGroupRecords - 1u) / kGroupRecords); w0 += 2) {
        const uint32_t v = (w0 / 4u) * (uint32_t)(8 * kGroupRecords) + (w0 % 4u) * 512u + lane * 8u;
        double q[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) q[u] = Gm<double>::ld(r, v + (u >> 1) * 2048u + (u & 1u) * 512u, 0u);
#pragma unroll
        for (uint32_t w = 0; w < 2; ++w) {
            double x = 0.0;
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) x += q[2u * u + w];
            sum += wave_sum(x);
        }
        if (w0 % 4u == 2u) {
            total += sum;
            sum = 0.0;
        }
    }
    return total;
}

// The counts of the n records of two passes, by one wave (at most one a spin, so
// below 2^32).
__device__ __forceinline__ uint32_t fold_pass_counts(const uint32_t* red, const uint32_t* black, uint32_t n)
{
    const __amdgpu_buffer_rsrc_t r = row_rsrc(red, n), b = row_rsrc(black, n);
    const uint32_t v = (threadIdx.x & 63u) * 4u;
    uint32_t c = 0;
#pragma unroll 1
    for (uint32_t u0 = 0; u0 * 64u < n; u0 += 8)
#pragma unroll
        for (uint32_t u = u0; u < u0 + 8; ++u)
            c += __builtin_amdgcn_raw_buffer_load_b32(r, v + u * 256u, 0u, 0) +
                 __builtin_amdgcn_raw_buffer_load_b32(b, v + u * 256u, 0u, 0);
    return wave_sum(c);
}

// ---------------------------------------------------------------------------
// Sweeps that follow each other in one call, where a pass leaves at most 2048
// records: the red pass of the next sweep does what a finalize launch would.
// Each of its work-groups sums the counts of the sweep before (its own next
// cone angle; the loads pass behind those of the march's first planes), and one
// work-group more runs the whole finalize meanwhile.  What the passes of a sweep
// share goes through a slot; slots and the red counts are kept twice, by the
// parity of the sweep in the call, so that no launch writes what its own
// work-groups read.  Against a finalize launch per sweep (MI355X,
// us a sampled sweep in the default shapes): FP32 96^3 20.5 -> 17.4, 128^3 27.1 ->
// 24.6, 64 x 64 x 512 27.1 -> 24.3, 160^3 40.0 -> 36.0, 256^3 111.5 -> 108.3, masked
// 1024 x 1024 x 5 52.0 -> 49.0; FP64 120 x 98 x 62 29.0 -> 24.7, 128^3 47 -> 44.
// ---------------------------------------------------------------------------
struct PassSlot {
    int32_t theta;
    uint32_t pad;
    int64_t sweep;
};
static_assert(offsetof(PassSlot, theta) == offsetof(DevState, theta) && offsetof(PassSlot, sweep) == offsetof(DevState, sweep),
              "a pass reads either");

struct PassHead {
    const PassSlot* from;    // what the sweep (red: the one before) left, or the chain state
    PassSlot* to;            // red: what it leaves; else null
    const uint32_t* red;     // the counts of the sweep before
    const uint32_t* black;
    uint32_t nrec;           // of each: 0 where the pass takes the cone angle as it is
    int32_t fin;             // finalize flags
    double T, N;
};

// The head of a pass of a carried sweep: cone angle and sweep number, from vector
// loads, which hold up nothing before their use.  (Other passes take them by scalar
// loads at their start.  Through this head, whose table look-up waits behind the
// first planes' loads, they took 0.3 to 4 % longer: MI355X, us a sampled sweep, 464^3
// FP32 750.5 for 747.3, 2 x 2 x 100000 FP64 632 for 608, one sweep a call of 128^3 FP32
// 26.8 for 25.8, FP64 45.6 for 44.1.)  load() comes before the loads of the march's
// first planes, table() after them, ready() stands for the barrier that follows.
template <typename R, int C>
struct HeadLoads {
    static constexpr uint32_t NC = kCarryRecords / kThreads;
    uint32_t c[2 * NC];
    int32_t theta;
    uint32_t sweep;
    R c1, down;
    __device__ __forceinline__ void load(const PassHead& h)
    {
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(h.from, 1u);
        theta = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (uint32_t)offsetof(PassSlot, theta), 0u, 0);
        sweep = __builtin_amdgcn_raw_buffer_load_b32(rs, (uint32_t)offsetof(PassSlot, sweep), 0u, 0);
        if constexpr (C == 0) {
            const __amdgpu_buffer_rsrc_t r = row_rsrc(h.red, h.nrec), b = row_rsrc(h.black, h.nrec);
#pragma unroll
            for (uint32_t u = 0; u < NC; ++u) {
                const uint32_t v = (u * (uint32_t)kThreads + threadIdx.x) * 4u;
                c[2 * u] = c[2 * u + 1] = 0u;
                if (u >= NC / 2 && h.nrec <= (uint32_t)kCarryRecords / 2u) continue;
                c[2 * u] = __builtin_amdgcn_raw_buffer_load_b32(r, v, 0u, 0);
                c[2 * u + 1] = __builtin_amdgcn_raw_buffer_load_b32(b, v, 0u, 0);
            }
        }
    }
    __device__ __forceinline__ void table(const KArgs<R>& a, const PassHead& h)
    {
        const __amdgpu_buffer_rsrc_t r = row_rsrc(a.c1tab, 181u);
        if constexpr (C == 0) {
            const int32_t up = h.nrec ? min(theta + 1, 180) : theta, dn = h.nrec ? max(theta - 1, 1) : theta;
            c1 = Gm<R>::ld(r, (uint32_t)up * (uint32_t)sizeof(R), 0u);
            down = Gm<R>::ld(r, (uint32_t)dn * (uint32_t)sizeof(R), 0u);
        } else {
            c1 = Gm<R>::ld(r, (uint32_t)theta * (uint32_t)sizeof(R), 0u);
        }
    }
    __device__ __forceinline__ void ready(const PassHead& h, uint32_t* wtot)
    {
        if constexpr (C == 0) {
            uint32_t n = 0;
#pragma unroll
            for (uint32_t u = 0; u < 2 * NC; ++u) n += c[u];
            n = wave_sum(n);
            if ((threadIdx.x & 63u) == 0) wtot[threadIdx.x >> 6] = n;
        }
        __syncthreads();
        // the same on every lane: into scalar registers
        theta = read_lane(theta, 0);
        sweep = read_lane(sweep, 0);
        if (C == 0 && h.nrec) {
            long long accepted = 0;
            for (int w = 0; w < kThreads / 64; ++w) accepted += (long long)wtot[w];
            const bool more = 2.0 * (double)accepted > h.N;
            theta = more ? min(theta + 1, 180) : max(theta - 1, 1);
            ++sweep;
            c1 = more ? c1 : down;
        }
        c1 = read_lane(c1, 0);
    }
};

// ---------------------------------------------------------------------------
// The Metropolis update of one site (Table A1, Eq. 1, Eq. 2): cone proposal,
// energy change in the local field, acceptance P < exp(-dE/T).  Returns the
// final spin; OBS adds the site and its red x-partner to the observables.
// ---------------------------------------------------------------------------
template <typename R, bool OBS, typename A>
__device__ __forceinline__ V3<R> update_site(const Model<R>& m, const V3<R>& s, const V3<R>& nb,
                                             const V3<R>& partner, const Rand4& rn, R c1, R scale,
                                             uint32_t& nacc, A& acc)
{
    const V3<R> hl{m.J * nb.x + m.h.x, m.J * nb.y + m.h.y, m.J * nb.z + m.h.z};
    const V3<R> tr = cone_move(s, Prim<R>::u01(rn.r0), Prim<R>::u01(rn.r1), c1);
    SiteTerms<R> k;
    const R dE = delta_e(m, s, tr, hl, k);
    const bool ok = Prim<R>::u01(rn.r2) < Prim<R>::boltzmann(dE, scale);
    const V3<R> f = ok ? tr : s;
    nacc += ok ? 1u : 0u;
    if (OBS) {
        // acc is the FP64 Acc (FP64 spins) or the spin-precision partial sums
        const V3<R> fp{f.x + partner.x, f.y + partner.y, f.z + partner.z};
        acc.M[0] += fp.x;
        acc.M[1] += fp.y;
        acc.M[2] += fp.z;
        acc.ex += -m.J * dot(f, nb);
        if (m.Ku != R(0)) {
            const R sf = ok ? k.te : k.se, sp = dot(partner, m.e);
            acc.eu += -m.Ku * (sf * sf + sp * sp);
        }
        if (m.Kc != R(0)) acc.ec += m.Kc * ((ok ? k.ct : k.cs) + cubic_f(partner));
        if (m.h.x != R(0) || m.h.y != R(0) || m.h.z != R(0)) acc.ez += -dot(m.h, fp);
    }
    return f;
}

// ---------------------------------------------------------------------------
// Standard colour pass (Table A1, MonteCarlo_Red(Black)ParallelPass).
//
// A work-group owns up to 256*SPT in-plane sites of one colour and marches over
// z_chunk planes.  The other colour's plane z sits in LDS with the x and y
// neighbours of the owned sites, so each plane of each colour is fetched once
// per pass, plus a halo.  Two geometries (GEO):
//
// * a window of consecutive colour indices, [base - hx, base + Q + hx) with the
//   halo (GEO 1 or 2: halo sites per thread): every access is one run of lines;
// * where rows are longer than 256 sites of a colour (GEO 0), a tile of tx
//   columns of ty rows, with a row more above and below and for each row the
//   one site beyond its edge that an x neighbour can be (left or right, by the
//   row's parity in that plane).  A window of one row of 512 fetched two rows
//   beside it.
//
// Short rows keep the window: its halo comes from the caches, and the tiles'
// broken lines cost more (measured on MI355X, us per sampled sweep: tiles
// against windows in each one's best shape, masked 1024 x 1024 x 5 52 for 64, 1024
// x 512 x 15 67 for 86; 464^3 FP32 937 for 757, 256^3 FP64 284 for 262).
// Two marches share this layout and differ in how far ahead the loads run:
//
// * depth one (march1): step z issues the other colour's plane z+2 and the
//   own colour's plane z+1; the other colour's z-1, z, z+1 and z+2 values at
//   the owned columns stay in registers, rotating by renaming over a march
//   unrolled by four.  Best while the spins stay in the 256 MB last-level
//   cache, whose latency one plane of look-ahead covers.
// * depth two (march2): step z issues the other colour's plane z+3 and the
//   own colour's plane z+2, so two planes of loads are in flight while one
//   is computed; the same-index partner comes from the window and becomes
//   the z-1 value of the next step, and three register planes rotate over a
//   march unrolled by three.  Best for lattices that stream from HBM.
//
// OBS (black pass only) fuses the observables: the black site after its
// update plus its red x-partner (same colour index), and the exchange of the
// black site with its six final red neighbours, so every site and every bond
// is counted once.  With FP32 spins a thread sums these terms in FP32 over
// its z chunk (z_chunk x SPT sites) and converts the sums to FP64 once;
// everything above the thread is FP64.
// ---------------------------------------------------------------------------
template <int GEO> constexpr int kHaloSlots = GEO == 2 ? 2 : 1;

template <typename R, int SPT, int GEO>
struct PassCtx {
    static constexpr int NH = kHaloSlots<GEO>;
    uint32_t tx, P, nz, W, z0, zn;   // tx: LDS entries from row to row
    uint32_t voff[SPT];          // byte offset of each owned column in a plane
    uint32_t w[SPT];             // its LDS entry
    uint32_t wd[2][SPT];         // LDS entry of its second x-neighbour, by z parity
    uint32_t par[SPT];           // x parity of the column at z = z0
    bool act[SPT];
    uint32_t hvoff[NH], hw[NH];  // the halo sites this thread fetches and their LDS entries
    uint32_t hodd;               // GEO 0: the halo site of planes z0 + 1, z0 + 3, ... (hvoff: z0, z0 + 2, ...)
    bool hact[NH];
    // the halo site of slot i in planes of parity b
    __device__ __forceinline__ uint32_t halo(int i, uint32_t b) const { return GEO == 0 && b ? hodd : hvoff[i]; }
    unsigned char* lds[2];
    R c1, scale;
    uint32_t sweep;
    uint32_t zbound;
};

// The neighbour sum of a site, in the order x-, x+, y-, y+, z-, z+ (o0, the
// same-index partner, and xd are the x neighbours, p the site's x parity); with
// MASK, bonds cut by the site's mask (intergrain bonds) weigh zero.
template <typename R, bool MASK>
__device__ __forceinline__ V3<R> neighbour_sum(const V3<R>& o0, const V3<R>& xd, uint32_t p, const V3<R>& ym,
                                               const V3<R>& yp, const V3<R>& zm, const V3<R>& zp, uint32_t mb)
{
    if constexpr (MASK) {
        const V3<R> xm = p ? o0 : xd, xp = p ? xd : o0;
        const R w0 = (mb & 1u) ? R(1) : R(0), w1 = (mb & 2u) ? R(1) : R(0);
        const R w2 = (mb & 4u) ? R(1) : R(0), w3 = (mb & 8u) ? R(1) : R(0);
        const R w4 = (mb & 16u) ? R(1) : R(0), w5 = (mb & 32u) ? R(1) : R(0);
        return V3<R>{((((w0 * xm.x + w1 * xp.x) + w2 * ym.x) + w3 * yp.x) + w4 * zm.x) + w5 * zp.x,
                     ((((w0 * xm.y + w1 * xp.y) + w2 * ym.y) + w3 * yp.y) + w4 * zm.y) + w5 * zp.y,
                     ((((w0 * xm.z + w1 * xp.z) + w2 * ym.z) + w3 * yp.z) + w4 * zm.z) + w5 * zp.z};
    } else {
        // x- + x+ is the same sum in either order
        return V3<R>{((((o0.x + xd.x) + ym.x) + yp.x) + zm.x) + zp.x,
                     ((((o0.y + xd.y) + ym.y) + yp.y) + zm.y) + zp.y,
                     ((((o0.z + xd.z) + ym.z) + yp.z) + zm.z) + zp.z};
    }
}

// Depth-one march: one step, plane z = z0 + zi; the register planes om, o0,
// op, opp hold the other colour's z-1, z, z+1 and z+2 (in flight), sc and
// sn the own colour's z and z+1 (in flight), mc and mn their masks, hp and hpp
// the halo's z+1 and z+2 (in flight).
template <typename R, int C, bool OBS, int SPT, int GEO, int K, bool MASK, typename A>
__device__ __forceinline__ void step1(const KArgs<R>& a, const Arrays<R>& g, const PassCtx<R, SPT, GEO>& x, uint32_t zi,
                                      V3<R> (&om)[SPT], V3<R> (&o0)[SPT], V3<R> (&op)[SPT], V3<R> (&opp)[SPT],
                                      V3<R> (&sc)[SPT], V3<R> (&sn)[SPT], uint32_t (&mc)[SPT], uint32_t (&mn)[SPT],
                                      V3<R> (&hp)[kHaloSlots<GEO>], V3<R> (&hpp)[kHaloSlots<GEO>], uint32_t& nacc, A& acc)
{
    constexpr int O = 1 - C;
    constexpr int B = K & 1;
    const uint32_t z = x.z0 + zi;
    const bool more = zi + 1 < x.zn;
    auto plane_off = [&](uint32_t zz) -> uint32_t {
        return x.P * (uint32_t)sizeof(R) * (zz >= x.nz ? zz - x.nz : zz);
    };
    if (more) {
        // the look-ahead loads leave at a raised wave priority: the march is
        // bound by their latency, and the SIMD then issues them before other
        // waves' arithmetic (measured on MI355X: 256^3 FP32 pass 53.7 -> 53.0
        // us)
        __builtin_amdgcn_s_setprio(2);
        const uint32_t fpp = plane_off(z + 2), fn = plane_off(z + 1);
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            opp[j] = g.get(O, x.voff[j], fpp);
            sn[j] = g.get(C, x.voff[j], fn);
            if (MASK) mn[j] = a.mask[C][x.voff[j] / (uint32_t)sizeof(R) + x.P * (z + 1)];
        }
#pragma unroll
        for (int i = 0; i < x.NH; ++i)
            if (x.hact[i]) hpp[i] = g.get(O, x.halo(i, B), fpp);
        __builtin_amdgcn_s_setprio(0);
        // anti-periodic or open z: plane z + 2 = nz is plane 0 seen across
        // the boundary; it serves only as the z+1 neighbour of plane nz - 1.
        // The uniform branch is taken once per tile at most.
        if (__builtin_expect(x.zbound != 0 && z + 2u == x.nz, 0)) {
            __asm__ volatile("");
#pragma unroll
            for (int j = 0; j < SPT; ++j) opp[j] = across_z(opp[j], x.zbound);
        }
    }
    // the sites' indices are formed here: carried from step to step they cost 4 to 6
    // registers, and with them a wave per SIMD (a batch of 24 lattices of 48^3 to
    // 128^3 FP32 in (1, 4): 173 us a sweep for 162 on MI355X)
    uint32_t pz = x.P * z;
    asm("" : "+s"(pz));
    const unsigned char* L = x.lds[B];
    const uint32_t fz = plane_off(z);
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        if (!x.act[j]) continue;
        const uint32_t p = x.par[j] ^ (uint32_t)B;
        const V3<R> xd = LdsPlane<R>::get(L, x.W, x.wd[B][j]);
        const V3<R> ym = LdsPlane<R>::get(L, x.W, x.w[j] - x.tx);
        const V3<R> yp = LdsPlane<R>::get(L, x.W, x.w[j] + x.tx);
        const uint32_t k = x.voff[j] / (uint32_t)sizeof(R) + pz;
        const V3<R> nb = neighbour_sum<R, MASK>(o0[j], xd, p, ym, yp, om[j], op[j], MASK ? mc[j] : 0u);
        const Rand4 rn = philox(x.sweep, 2u * k + p, (uint32_t)C, a.inst, a.key0, a.key1);
        const V3<R> f = update_site<R, OBS>(a.m, sc[j], nb, o0[j], rn, x.c1, x.scale, nacc, acc);
        g.put(C, x.voff[j], fz, f);
    }
    if (more) {
        unsigned char* Ln = x.lds[B ^ 1];
#pragma unroll
        for (int j = 0; j < SPT; ++j) LdsPlane<R>::put(Ln, x.W, x.w[j], op[j]);
#pragma unroll
        for (int i = 0; i < x.NH; ++i)
            if (x.hact[i]) LdsPlane<R>::put(Ln, x.W, x.hw[i], hp[i]);
    }
    __syncthreads();
}

// table and ready: what is due after the loads of the first planes, and in place
// of the barrier behind their stores (the cone angle and the sweep number are
// read no earlier).
template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, typename Table, typename Ready>
__device__ __forceinline__ void march1(const KArgs<R>& a, const Arrays<R>& g, const PassCtx<R, SPT, GEO>& x, uint32_t& nacc,
                                       Acc& acc, Table table, Ready ready)
{
    constexpr int O = 1 - C;
    V3<R> rA[SPT], rB[SPT], rC[SPT], rD[SPT], s0[SPT], s1[SPT], h0[kHaloSlots<GEO>], h1[kHaloSlots<GEO>];
    uint32_t m0[SPT], m1[SPT];
    {
        auto plane_off = [&](int zz) -> uint32_t {
            const int w = zz < 0 ? zz + (int)a.nz : (zz >= (int)a.nz ? zz - (int)a.nz : zz);
            return a.P * (uint32_t)sizeof(R) * (uint32_t)w;
        };
        const uint32_t fm = plane_off((int)x.z0 - 1), f0 = plane_off((int)x.z0), fp = plane_off((int)x.z0 + 1);
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            rA[j] = g.get(O, x.voff[j], fm);
            rB[j] = g.get(O, x.voff[j], f0);
            rC[j] = g.get(O, x.voff[j], fp);
            s0[j] = g.get(C, x.voff[j], f0);
            if (MASK) m0[j] = a.mask[C][x.voff[j] / (uint32_t)sizeof(R) + a.P * x.z0];
        }
        table();
#pragma unroll
        for (int i = 0; i < x.NH; ++i)
            if (x.hact[i]) {
                LdsPlane<R>::put(x.lds[0], x.W, x.hw[i], g.get(O, x.halo(i, 0), f0));
                h0[i] = g.get(O, x.halo(i, 1), fp);
            }
#pragma unroll
        for (int j = 0; j < SPT; ++j) LdsPlane<R>::put(x.lds[0], x.W, x.w[j], rB[j]);
        // anti-periodic or open z: the z-1 plane of z0 = 0 and the z+1 plane
        // of z0 = nz - 1 lie across the boundary (both used only as z
        // neighbours)
        if (x.zbound != 0 && x.z0 == 0) {
#pragma unroll
            for (int j = 0; j < SPT; ++j) rA[j] = across_z(rA[j], x.zbound);
        }
        if (x.zbound != 0 && x.z0 + 1u == a.nz) {
#pragma unroll
            for (int j = 0; j < SPT; ++j) rC[j] = across_z(rC[j], x.zbound);
        }
    }
    ready();

    Part<R> part;
    auto& pa = site_acc<R>(acc, part);
    uint32_t zi = 0;
    for (; zi + 4 <= x.zn; zi += 4) {
        step1<R, C, OBS, SPT, GEO, 0, MASK>(a, g, x, zi + 0, rA, rB, rC, rD, s0, s1, m0, m1, h0, h1, nacc, pa);
        step1<R, C, OBS, SPT, GEO, 1, MASK>(a, g, x, zi + 1, rB, rC, rD, rA, s1, s0, m1, m0, h1, h0, nacc, pa);
        step1<R, C, OBS, SPT, GEO, 2, MASK>(a, g, x, zi + 2, rC, rD, rA, rB, s0, s1, m0, m1, h0, h1, nacc, pa);
        step1<R, C, OBS, SPT, GEO, 3, MASK>(a, g, x, zi + 3, rD, rA, rB, rC, s1, s0, m1, m0, h1, h0, nacc, pa);
    }
    if (zi < x.zn) step1<R, C, OBS, SPT, GEO, 0, MASK>(a, g, x, zi + 0, rA, rB, rC, rD, s0, s1, m0, m1, h0, h1, nacc, pa);
    if (zi + 1 < x.zn)
        step1<R, C, OBS, SPT, GEO, 1, MASK>(a, g, x, zi + 1, rB, rC, rD, rA, s1, s0, m1, m0, h1, h0, nacc, pa);
    if (zi + 2 < x.zn)
        step1<R, C, OBS, SPT, GEO, 2, MASK>(a, g, x, zi + 2, rC, rD, rA, rB, s0, s1, m0, m1, h0, h1, nacc, pa);
    if constexpr (OBS) flush_part(acc, pa);
}

// Depth-two march: one step, plane z = z0 + zi.  op: the other colour's plane
// z+1 (landed); on: the slot that receives plane z+3.  sc, sn: the own
// colour's plane z (landed) and the slot for plane z+2; hp, hn: the halo
// likewise; mc, mn: the masks likewise.  om holds plane z-1 on entry and
// plane z on exit.
//
// Every step issues its loads unconditionally, so that the number of
// memory operations between a load and its use is the same on every path
// (the compiler's wait counts are then those of the steady state); the
// planes are clamped to the last one the tile needs, so the loads of the
// last steps re-read planes just fetched.
template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, typename A>
__device__ __forceinline__ void step2(const KArgs<R>& a, const Arrays<R>& g, const PassCtx<R, SPT, GEO>& x, uint32_t zi,
                                      V3<R> (&om)[SPT], V3<R> (&op)[SPT], V3<R> (&on)[SPT], V3<R> (&sc)[SPT],
                                      V3<R> (&sn)[SPT], V3<R> (&hp)[kHaloSlots<GEO>], V3<R> (&hn)[kHaloSlots<GEO>],
                                      uint32_t (&mc)[SPT],
                                      uint32_t (&mn)[SPT], uint32_t& nacc, A& acc)
{
    constexpr int O = 1 - C;
    const uint32_t z = x.z0 + zi;
    const uint32_t B = zi & 1u;
    const uint32_t zend = x.z0 + x.zn;      // <= nz
    auto plane_off = [&](uint32_t zz) -> uint32_t {
        return x.P * (uint32_t)sizeof(R) * (zz >= x.nz ? zz - x.nz : zz);
    };
    // loads two planes ahead: the other colour's plane z+3 (the z+1
    // neighbour of plane z+2) and the own colour's plane z+2
    // (at the normal wave priority: raising it around these loads, as the
    // depth-one step does, measured 0.5-1.3 % slower at 384^3 and 464^3)
    const uint32_t z3 = min(z + 3u, zend), z2 = min(z + 2u, zend - 1u);
    const uint32_t f3 = plane_off(z3), f2 = plane_off(z2);
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        on[j] = g.get(O, x.voff[j], f3);
        sn[j] = g.get(C, x.voff[j], f2);
        if (MASK) mn[j] = a.mask[C][x.voff[j] / (uint32_t)sizeof(R) + x.P * z2];
    }
#pragma unroll
    for (int i = 0; i < x.NH; ++i) hn[i] = g.get(O, x.halo(i, B ^ 1u), f3);
    // anti-periodic or open z: plane nz is plane 0 seen across the boundary
    // (only ever the z+1 neighbour of plane nz - 1); a uniform branch taken
    // in the top tile only
    if (__builtin_expect(x.zbound != 0 && z3 == x.nz, 0)) {
        __asm__ volatile("");
#pragma unroll
        for (int j = 0; j < SPT; ++j) on[j] = across_z(on[j], x.zbound);
    }
    // plane z+1 (issued two steps ago) into the other LDS buffer; its
    // readers of the step before have passed the barrier
    {
        unsigned char* Ln = B ? x.lds[0] : x.lds[1];   // a select keeps the LDS addressing
#pragma unroll
        for (int j = 0; j < SPT; ++j) LdsPlane<R>::put(Ln, x.W, x.w[j], op[j]);
#pragma unroll
        for (int i = 0; i < x.NH; ++i)
            if (x.hact[i]) LdsPlane<R>::put(Ln, x.W, x.hw[i], hp[i]);
    }
    const unsigned char* L = B ? x.lds[1] : x.lds[0];
    const uint32_t fz = plane_off(z);
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        if (!x.act[j]) continue;
        const uint32_t p = x.par[j] ^ B;
        const V3<R> xd = LdsPlane<R>::get(L, x.W, B ? x.wd[1][j] : x.wd[0][j]);
        const V3<R> ym = LdsPlane<R>::get(L, x.W, x.w[j] - x.tx);
        const V3<R> yp = LdsPlane<R>::get(L, x.W, x.w[j] + x.tx);
        const V3<R> o0 = LdsPlane<R>::get(L, x.W, x.w[j]);
        const uint32_t k = x.voff[j] / (uint32_t)sizeof(R) + x.P * z;
        const V3<R> nb = neighbour_sum<R, MASK>(o0, xd, p, ym, yp, om[j], op[j], MASK ? mc[j] : 0u);
        const Rand4 rn = philox(x.sweep, 2u * k + p, (uint32_t)C, a.inst, a.key0, a.key1);
        const V3<R> f = update_site<R, OBS>(a.m, sc[j], nb, o0, rn, x.c1, x.scale, nacc, acc);
        g.put(C, x.voff[j], fz, f);
        om[j] = o0;
    }
    __syncthreads();
}

template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, typename Table, typename Ready>
__device__ __forceinline__ void march2(const KArgs<R>& a, const Arrays<R>& g, const PassCtx<R, SPT, GEO>& x, uint32_t& nacc,
                                       Acc& acc, Table table, Ready ready)
{
    constexpr int O = 1 - C;
    // register planes: the other colour's z-1 (om) and three rotating slots
    // (planes z+1, z+2, z+3 at step z), the own colour's and the halo's
    // three rotating slots, and the masks'
    V3<R> om[SPT], oA[SPT], oB[SPT], oC[SPT], sA[SPT], sB[SPT], sC[SPT], hA[kHaloSlots<GEO>], hB[kHaloSlots<GEO>], hC[kHaloSlots<GEO>];
    uint32_t mA[SPT], mB[SPT], mC[SPT];
    {
        auto plane_off = [&](int zz) -> uint32_t {
            const int w = zz < 0 ? zz + (int)a.nz : (zz >= (int)a.nz ? zz - (int)a.nz : zz);
            return a.P * (uint32_t)sizeof(R) * (uint32_t)w;
        };
        // planes z0-1 .. z0+2 of the other colour, z0 and z0+1 of the own
        // colour (clamped to the tile's last needed plane, as in the steps)
        const uint32_t zend = x.z0 + x.zn;
        const uint32_t pB = min(x.z0 + 2u, zend), sBz = min(x.z0 + 1u, zend - 1u);
        const uint32_t fm = plane_off((int)x.z0 - 1), f0 = plane_off((int)x.z0), f1 = plane_off((int)x.z0 + 1),
                       f2 = plane_off((int)pB), fs1 = plane_off((int)sBz);
        // plane z0 (written to LDS below) is loaded last: waiting for it
        // waits for every other prologue load, so no prologue load is still
        // in flight when the march starts and the waits inside the march are
        // set by the march alone
        V3<R> o0[SPT], h0[kHaloSlots<GEO>];
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            om[j] = g.get(O, x.voff[j], fm);
            oA[j] = g.get(O, x.voff[j], f1);
            oB[j] = g.get(O, x.voff[j], f2);
            sA[j] = g.get(C, x.voff[j], f0);
            sB[j] = g.get(C, x.voff[j], fs1);
            if (MASK) {
                mA[j] = a.mask[C][x.voff[j] / (uint32_t)sizeof(R) + a.P * x.z0];
                mB[j] = a.mask[C][x.voff[j] / (uint32_t)sizeof(R) + a.P * sBz];
            }
        }
#pragma unroll
        for (int i = 0; i < x.NH; ++i) {
            hA[i] = g.get(O, x.halo(i, 1), f1);
            hB[i] = g.get(O, x.halo(i, 0), f2);
        }
#pragma unroll
        for (int j = 0; j < SPT; ++j) o0[j] = g.get(O, x.voff[j], f0);
#pragma unroll
        for (int i = 0; i < x.NH; ++i) h0[i] = g.get(O, x.halo(i, 0), f0);
        table();
#pragma unroll
        for (int i = 0; i < x.NH; ++i)
            if (x.hact[i]) LdsPlane<R>::put(x.lds[0], x.W, x.hw[i], h0[i]);
#pragma unroll
        for (int j = 0; j < SPT; ++j) LdsPlane<R>::put(x.lds[0], x.W, x.w[j], o0[j]);
        // anti-periodic or open z: plane -1 (the z-1 neighbour of plane 0)
        // and plane nz (the z+1 neighbour of plane nz - 1) lie across the
        // boundary
        if (x.zbound != 0) {
#pragma unroll
            for (int j = 0; j < SPT; ++j) {
                if (x.z0 == 0) om[j] = across_z(om[j], x.zbound);
                if (x.z0 + 1u == a.nz) oA[j] = across_z(oA[j], x.zbound);
                if (pB == a.nz) oB[j] = across_z(oB[j], x.zbound);
            }
        }
    }
    ready();

    Part<R> part;
    auto& pa = site_acc<R>(acc, part);
    uint32_t zi = 0;
    for (; zi + 3 <= x.zn; zi += 3) {
        step2<R, C, OBS, SPT, GEO, MASK>(a, g, x, zi + 0, om, oA, oC, sA, sC, hA, hC, mA, mC, nacc, pa);
        step2<R, C, OBS, SPT, GEO, MASK>(a, g, x, zi + 1, om, oB, oA, sB, sA, hB, hA, mB, mA, nacc, pa);
        step2<R, C, OBS, SPT, GEO, MASK>(a, g, x, zi + 2, om, oC, oB, sC, sB, hC, hB, mC, mB, nacc, pa);
    }
    if (zi < x.zn) step2<R, C, OBS, SPT, GEO, MASK>(a, g, x, zi + 0, om, oA, oC, sA, sC, hA, hC, mA, mC, nacc, pa);
    if (zi + 1 < x.zn) step2<R, C, OBS, SPT, GEO, MASK>(a, g, x, zi + 1, om, oB, oA, sB, sA, hB, hA, mB, mA, nacc, pa);
    if constexpr (OBS) flush_part(acc, pa);

}

// One work-group of a colour pass: logical tile b (in-plane window or tile
// b % n, of z-slab b / n) of the lattice described by a, with the march of
// depth two when DEEP.  head: of a carried sweep, else null (the pass reads the
// chain state); wtot: a word per wave in shared memory with it.
template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, bool DEEP>
__device__ __forceinline__ void pass_tile(const KArgs<R>& a, const PassGeom& q, const uint32_t zc, const uint32_t b,
                                          const R scale, unsigned char* smem, const PassHead* head, uint32_t* wtot)
{
    const Arrays<R> g(a);
    HeadLoads<R, C> hl;
    if (head) hl.load(*head);
    const uint32_t hx = a.hx, ny = a.ny;
    PassCtx<R, SPT, GEO> x;
    x.P = a.P;
    x.nz = a.nz;
    x.tx = GEO == 0 ? q.tx : hx;
    x.W = GEO == 0 ? q.entries : kThreads * SPT + 2u * hx;
    const uint32_t t = threadIdx.x;
    const uint32_t zb = b / q.n, r = b - zb * q.n;
    x.z0 = zb * zc;
    x.zn = min(zc, a.nz - x.z0);
    x.lds[0] = smem;
    x.lds[1] = smem + (size_t)x.W * LdsPlane<R>::bytes_per_entry;
    if (!head) {
        x.c1 = a.c1tab[a.st->theta];
        x.sweep = (uint32_t)a.st->sweep;
    }
    x.scale = scale;
    x.zbound = a.zbound;
    if constexpr (GEO != 0) {
        constexpr uint32_t Q = kThreads * SPT;
        const uint32_t base = r * Q;
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const uint32_t k = base + t + (uint32_t)kThreads * j;
            x.act[j] = k < a.P;
            const uint32_t km = x.act[j] ? k : k % a.P;
            const uint32_t kx = km % hx, yy = km / hx;
            x.voff[j] = km * (uint32_t)sizeof(R);
            x.w[j] = hx + t + (uint32_t)kThreads * j;
            x.par[j] = (yy + x.z0 + (uint32_t)C) & 1u;
            // window entry of the x-neighbour that is not the same-index partner:
            // x+1 (wrapping inside the row) when the site's x is odd, else x-1
#pragma unroll
            for (int bpar = 0; bpar < 2; ++bpar) {
                const uint32_t p = x.par[j] ^ (uint32_t)bpar;
                const uint32_t w = x.w[j];
                x.wd[bpar][j] = p ? (kx == hx - 1 ? w + 1 - hx : w + 1) : (kx == 0 ? w + hx - 1 : w - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < x.NH; ++i) {
            const uint32_t slot = t + (uint32_t)kThreads * i;
            x.hact[i] = slot < 2u * hx;
            x.hw[i] = slot < hx ? slot : slot + Q;
            x.hvoff[i] = ((base + x.hw[i] + a.P - hx) % a.P) * (uint32_t)sizeof(R);
        }
        x.hodd = 0u;
    } else {
        const uint32_t by = r / q.ntx, bx = r - by * q.ntx;
        const uint32_t x0 = bx * q.tx, y0 = by * q.ty;
        const uint32_t tw = min(q.tx, hx - x0), th = min(q.ty, ny - y0);     // of this tile
        const uint32_t edge = (q.ty + 2u) * q.tx;                            // entries of the sites beyond the edges
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const uint32_t e = t + (uint32_t)kThreads * j;
            const uint32_t ly = e / q.tx, lx = e - ly * q.tx;
            x.act[j] = lx < tw && ly < th;
            const uint32_t cx = x.act[j] ? lx : 0u, cy = x.act[j] ? ly : 0u;
            x.voff[j] = (x0 + cx + hx * (y0 + cy)) * (uint32_t)sizeof(R);
            // a thread without a site writes its plane values to a spare entry
            const uint32_t w = (cy + 1u) * q.tx + cx;
            x.w[j] = x.act[j] ? w : q.entries - 1u;
            x.par[j] = (y0 + cy + x.z0 + (uint32_t)C) & 1u;
#pragma unroll
            for (int bpar = 0; bpar < 2; ++bpar) {
                const uint32_t p = x.par[j] ^ (uint32_t)bpar;
                x.wd[bpar][j] = p ? (cx == tw - 1 ? edge + cy : w + 1) : (cx == 0 ? edge + cy : w - 1);
            }
        }
        // halo slots: the row above, the row below, then the sites beyond the edges
        const bool top = t < q.tx, row = t < 2u * q.tx;
        const uint32_t lx = top ? t : t - q.tx, le = t - 2u * q.tx;
        x.hact[0] = row ? lx < tw : le < th;
        const uint32_t yy = top ? (y0 == 0 ? ny - 1 : y0 - 1) : (y0 + th == ny ? 0u : y0 + th);
        uint32_t h[2];
#pragma unroll
        for (uint32_t bpar = 0; bpar < 2; ++bpar) {
            // an odd site's neighbour lies right of the tile, an even one's left
            const uint32_t p = (y0 + le + x.z0 + (uint32_t)C + bpar) & 1u;
            const uint32_t xe = p ? (x0 + tw == hx ? 0u : x0 + tw) : (x0 == 0 ? hx - 1 : x0 - 1);
            const uint32_t site = row ? x0 + lx + hx * yy : xe + hx * (y0 + le);
            h[bpar] = x.hact[0] ? site * (uint32_t)sizeof(R) : 0u;
        }
        x.hvoff[0] = h[0];
        x.hodd = h[1];
        x.hw[0] = row ? (top ? lx : (th + 1u) * q.tx + lx) : edge + le;
    }

    uint32_t nacc = 0;
    Acc acc;
    const auto table = [&] {
        if (head) hl.table(a, *head);
    };
    const auto ready = [&] {
        if (!head) {
            __syncthreads();
            return;
        }
        hl.ready(*head, wtot);
        x.c1 = hl.c1;
        x.sweep = hl.sweep;
    };
    if constexpr (DEEP) march2<R, C, OBS, SPT, GEO, MASK>(a, g, x, nacc, acc, table, ready);
    else march1<R, C, OBS, SPT, GEO, MASK>(a, g, x, nacc, acc, table, ready);
    if (C == 0 && head && b == 0 && threadIdx.x == 0)
        *head->to = PassSlot{hl.theta, 0u, (int64_t)hl.sweep};
    // LDS is free after the last barrier of the march
    block_end<R, OBS, false>(a, C, b, nacc, acc, reinterpret_cast<double*>(smem));
}

// The depth-two FP32 variants with up to two sites per thread are held to
// 128 registers (four waves per SIMD), which they reach without spilling.
template <typename R, int SPT, bool DEEP>
constexpr int pass_waves_per_eu()
{
    return DEEP && sizeof(R) == 4 && SPT <= 2 ? 4 : 1;
}

template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, bool DEEP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(pass_waves_per_eu<R, SPT, DEEP>())))
void pass_kernel(const KArgs<R> a, const PassGeom q, const uint32_t zc, const uint32_t nblk, const R scale)
{
    extern __shared__ __align__(16) unsigned char smem[];
    pass_tile<R, C, OBS, SPT, GEO, MASK, DEEP>(a, q, zc, xcd_remap(blockIdx.x, nblk), scale, smem, nullptr, nullptr);
}

// A pass of a carried sweep.
template <typename R, int C, bool OBS, int SPT, int GEO, bool MASK, bool DEEP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(pass_waves_per_eu<R, SPT, DEEP>())))
void carried_pass_kernel(const KArgs<R> a, const PassGeom q, const uint32_t zc, const uint32_t nblk, const R scale,
                         const PassHead h)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t wtot[kThreads / 64];
    if (C == 0 && blockIdx.x == nblk) {
        // (the records lie before the red counts this launch writes)
        double* tot = reinterpret_cast<double*>(smem);
        fold_sweep<kThreads, kObsRows>(
            a.st, h.fin, h.T, h.N, tot, reinterpret_cast<unsigned long long*>(tot + kObsRows),
            [&](uint32_t e) { return fold_groups(a.part + (size_t)e * a.cnt_stride, nblk); },
            [&] { return fold_pass_counts(h.red, h.black, nblk); });
        return;
    }
    pass_tile<R, C, OBS, SPT, GEO, MASK, DEEP>(a, q, zc, xcd_remap(blockIdx.x, nblk), scale, smem, &h, wtot);
}

// Launch of one colour pass of one lattice; the kernel variant follows the
// launch shape (sites per thread), the geometry and the colour.  Each
// translation unit instantiates one family: the plain depth-one march in hmc_kernels.hip, the
// masked one in hmc_masked_kernels.hip, the depth-two march in
// hmc_deep_kernels.hip (so they compile in parallel).
template <bool MASK, bool DEEP>
struct PassLaunch {
    template <typename R, int C, bool OBS, int SPT, int GEO>
    static void go(const KArgs<R>& args, const DevLattice& d, int zc, double T, const SweepCarry& c, hipStream_t s)
    {
        const uint32_t nblk = (uint32_t)pass_blocks(d, SPT, zc);
        const PassGeom& q = pass_geom(d, SPT);
        const size_t lds = pass_lds_bytes(d, SPT);
        const R scale = Prim<R>::scale_for(T);
        if (!c.on) {
            pass_kernel<R, C, OBS, SPT, GEO, MASK, DEEP><<<nblk, kThreads, lds, s>>>(args, q, (uint32_t)zc, nblk, scale);
            return;
        }
        KArgs<R> a = args;
        PassSlot* slot = carry_slots(d);
        const bool head = C == 0 && c.sweep > 0;                 // finalizes the sweep before
        PassHead h{};
        h.from = reinterpret_cast<const PassSlot*>(d.st);
        if (head) h.from = slot + ((c.sweep - 1) & 1);
        else if (C == 1) h.from = slot + (c.sweep & 1);
        h.red = red_counts(d, c.sweep - 1);
        h.black = d.cnt + d.max_blocks;
        h.nrec = head ? nblk : 0u;
        h.fin = c.fin;
        h.T = T;
        h.N = (double)d.N;
        if (C == 0) {
            h.to = slot + (c.sweep & 1);
            a.cnt = red_counts(d, c.sweep);
        }
        const uint32_t grid = nblk + (head ? 1u : 0u);
        carried_pass_kernel<R, C, OBS, SPT, GEO, MASK, DEEP><<<grid, kThreads, lds, s>>>(a, q, (uint32_t)zc, nblk, scale, h);
    }

    template <typename R, int SPT, int GEO>
    static void by_colour(const KArgs<R>& a, const DevLattice& d, int colour, bool obs, int zc, double T,
                          const SweepCarry& c, hipStream_t s)
    {
        if (colour == 0) go<R, 0, false, SPT, GEO>(a, d, zc, T, c, s);
        else if (obs) go<R, 1, true, SPT, GEO>(a, d, zc, T, c, s);
        else go<R, 1, false, SPT, GEO>(a, d, zc, T, c, s);
    }

    template <typename R, int SPT>
    static void by_geometry(const KArgs<R>& a, const DevLattice& d, int colour, bool obs, int zc, double T,
                            const SweepCarry& c, hipStream_t s)
    {
        const int geo = geometry_of(d.hx);
        if (geo == 1) by_colour<R, SPT, 1>(a, d, colour, obs, zc, T, c, s);
        else if (geo == 2) by_colour<R, SPT, 2>(a, d, colour, obs, zc, T, c, s);
        else by_colour<R, SPT, 0>(a, d, colour, obs, zc, T, c, s);
    }

    template <typename R>
    static void by_shape(const DevLattice& d, int colour, bool obs, int spt, int zc, double T,
                         const SweepCarry& c, hipStream_t s)
    {
        const auto a = make_args<R>(d);
        if (spt == 1) by_geometry<R, 1>(a, d, colour, obs, zc, T, c, s);
        else if (spt == 2) by_geometry<R, 2>(a, d, colour, obs, zc, T, c, s);
        else by_geometry<R, 4>(a, d, colour, obs, zc, T, c, s);
    }

    static hipError_t run(const DevLattice& d, int colour, bool obs, int spt, int zc, double T, const SweepCarry& c,
                          hipStream_t s)
    {
        if (d.precision == 32) by_shape<float>(d, colour, obs, spt, zc, T, c, s);
        else by_shape<double>(d, colour, obs, spt, zc, T, c, s);
        return hipGetLastError();
    }
};

// ---------------------------------------------------------------------------
// Measurement of the current spins: M, the energies and the torque.  A thread
// takes one column of a slab of zc planes: for each of its colour indices k
// the black site k with its six red neighbours (every bond once) and the red
// site k.  The red planes z-1, z and z+1 of the column rotate through
// registers; the in-plane neighbours are loaded again, from cache.  Threads
// number the columns of all slabs through, so thin lattices leave none idle.
//
// The bytes ask for one read of the spins; what a one-site-per-thread launch
// spent its time on is the work-group sum of ten doubles, about as many
// instructions as the 64 sites of a wave.  A slab shares that sum between its
// planes (us per hmc_observables on MI355X against one site per thread: 256^3
// FP32 67 for 119, 464^3 332 for 685, 256^3 FP64 125 for 157).
// Every term is formed in the spin precision and added in FP64.
// ---------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void measure_column(const KArgs<R>& a, const uint32_t zc, const uint32_t f, Acc& acc)
{
    constexpr uint32_t rs = sizeof(R);
    const uint32_t hx = a.hx, ny = a.ny, nz = a.nz, P = a.P;
    const uint32_t slab = f / P, q = f - slab * P;
    const uint32_t z0 = slab * zc;
    if (z0 >= nz) return;
    const uint32_t zn = min(zc, nz - z0);
    const uint32_t y = q / hx, kx = q - y * hx;
    const Arrays<R> g(a);
    // distance to the x-neighbour that is not the same-index partner, by the
    // x parity of the black site, and to the y-neighbours (in sites)
    const int32_t d0 = kx == 0 ? (int32_t)hx - 1 : -1, d1 = kx == hx - 1 ? 1 - (int32_t)hx : 1;
    const int32_t dm = y == 0 ? (int32_t)(hx * (ny - 1)) : -(int32_t)hx;
    const int32_t dp = y == ny - 1 ? -(int32_t)(hx * (ny - 1)) : (int32_t)hx;
    uint32_t k = q + P * z0;
    V3<R> om = g.get(0, (z0 == 0 ? q + P * (nz - 1) : k - P) * rs, 0);
    V3<R> o0 = g.get(0, k * rs, 0);
    // what a step reads: the red plane above, the black site, the in-plane
    // neighbours and the mask
    struct Step {
        V3<R> op, blk, xd, ym, yp;
        uint32_t mb;
    };
    auto load = [&](uint32_t z, uint32_t i, Step& s) {
        s.op = g.get(0, (z == nz - 1 ? q : i + P) * rs, 0);
        s.blk = g.get(1, i * rs, 0);
        s.xd = g.get(0, (i + (uint32_t)(((y + z + 1u) & 1u) ? d1 : d0)) * rs, 0);
        s.ym = g.get(0, (i + (uint32_t)dm) * rs, 0);
        s.yp = g.get(0, (i + (uint32_t)dp) * rs, 0);
        s.mb = a.mask[1] ? a.mask[1][i] : 0x3Fu;
    };
    if (a.zbound && z0 == 0) om = across_z(om, a.zbound);
    Step cur;
    load(z0, k, cur);
    const auto add = [&](uint32_t z) {
        if (a.zbound && z == nz - 1) cur.op = across_z(cur.op, a.zbound);
        const uint32_t p = (y + z + 1u) & 1u;
        V3<R> xm = p ? o0 : cur.xd, xp = p ? cur.xd : o0, zm = om, zp = cur.op;
        if (a.mask[1]) {
            const V3<R> zero{R(0), R(0), R(0)};
            if (!(cur.mb & 1u)) xm = zero;
            if (!(cur.mb & 2u)) xp = zero;
            if (!(cur.mb & 4u)) cur.ym = zero;
            if (!(cur.mb & 8u)) cur.yp = zero;
            if (!(cur.mb & 16u)) zm = zero;
            if (!(cur.mb & 32u)) zp = zero;
        }
        const V3<R> nb{((((xm.x + xp.x) + cur.ym.x) + cur.yp.x) + zm.x) + zp.x,
                       ((((xm.y + xp.y) + cur.ym.y) + cur.yp.y) + zm.y) + zp.y,
                       ((((xm.z + xp.z) + cur.ym.z) + cur.yp.z) + zm.z) + zp.z};
        acc.ex += (double)(-a.m.J * dot(cur.blk, nb));
        add_site<R, true>(acc, a.m, cur.blk);
        add_site<R, true>(acc, a.m, o0);
        om = o0;
        o0 = cur.op;
    };
    // The next step's loads leave before this step's sums.  FP64: the last step
    // stands behind the loop.  FP32: it loads its own planes again, which is faster
    // where a thread has several (256^3 67.4 us for 71.7); a thread of one plane has
    // no loop.  (When every last step loaded again, lattices of one or two planes a
    // thread took 0.7 to 1.5 us longer: 64^3 FP64 33.4 us for 32.5, 72^3 34.3 for 33.6,
    // 64^3 FP32 32.1 for 31.7; 256^3 FP64 129 for 125.  With its loads behind a
    // branch in the loop the waits came early: 464^3 FP32 359 us for 330.)
    const uint32_t zl = z0 + zn - 1;
    if constexpr (sizeof(R) == 8) {
        for (uint32_t z = z0; z < zl; ++z) {
            Step next;
            k += P;
            load(z + 1u, k, next);
            add(z);
            cur = next;
        }
        add(zl);
    } else if (zn == 1u) {
        add(z0);
    } else {
        for (uint32_t z = z0; z <= zl; ++z) {
            Step next;
            load(min(z + 1u, zl), z < zl ? k + P : k, next);
            add(z);
            cur = next;
            k += P;
        }
    }
}

// The colour pass of a lattice with bond masks (hmc_masked_kernels.hip).
hipError_t launch_pass_masked(const DevLattice& d, int colour, bool obs, int spt, int zc, double T,
                              const SweepCarry& c, hipStream_t s);
// The colour pass with the depth-two march (hmc_deep_kernels.hip).
hipError_t launch_pass_deep(const DevLattice& d, int colour, bool obs, int spt, int zc, double T,
                            const SweepCarry& c, hipStream_t s);

}  // namespace hmc
