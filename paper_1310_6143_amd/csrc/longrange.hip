// Long-range step of libsllg for gfx950: predictor and corrector launches
// for simple-cubic lattices whose sites all have one and the same set of
// links, up to four cells away on each axis (exchange reaching hundreds of
// partners; uniform material, scalar exchange, periodic on every axis).
//
// Paper (Evans et al., arXiv:1310.6143), "The classical spin Hamiltonian":
// exchange reaching several lattice spacings; "Time Integration of the LLG
// Equation": the two launches keep every predictor before any corrector.
//
// What bounds it: the wide stencil form reads a table entry, its coupling
// and its spin for every link of every site through the L2 (10.5 vector
// instructions and two loads a link).  Here a workgroup copies the spins of
// an 8 x 8 x 4 cell tile and four cells around it into LDS once.  A lane
// holds a run of four sites along z: for each column (dx, dy) of links it
// reads the column's spins once and uses each for up to four sites, so a link
// costs three FMAs and a third of an LDS read.  The columns are ordered by their reach along z, so each loop
// over them has its run unrolled, and their couplings and offsets come from
// LDS (scalar loads, which drain with the LDS reads, took 29.4 us a step for
// 110,592 FP32 spins against 26.9 here; the wide form 70.6, and FP64 115.4
// against 37.9).  The four waves take a quarter of the columns each (a small
// system has too few sites to fill the chip otherwise) and add their parts
// in LDS in a fixed order; then every thread finishes one site.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_common.hpp"
#include "kernels.hpp"
#include "layout.hpp"
#include "site_step.hpp"

namespace sllg {
namespace {

using namespace dev;

constexpr int TX = 8, TY = 8, TZ = 4, H = kLongReach;
constexpr int BX = TX + 2 * H, BY = TY + 2 * H, BZ = TZ + 2 * H, BOX = BX * BY * BZ;
constexpr int BT = 256, WAVES = BT / 64;
static_assert(TX * TY == 64 && TX * TY * TZ == BT, "a lane per column of the tile, a thread per site at the end");

// The box, z fastest (a lane's run is consecutive).  FP32: 16 bytes a site;
// FP64: x, y in one array and z in another.
template <typename R>
struct LongBox;
template <>
struct LongBox<float> {
    typedef float Slot __attribute__((ext_vector_type(4)));
    Slot s[BOX];
    __device__ __forceinline__ V3<float> get(int q) const
    {
        const Slot v = s[q];
        return V3<float>{v.x, v.y, v.z};
    }
    __device__ __forceinline__ void put(int q, const V3<float>& v) { s[q] = Slot{v.x, v.y, v.z, 0.0f}; }
};
template <>
struct LongBox<double> {
    typedef double XY __attribute__((ext_vector_type(2)));
    XY xy[BOX];
    double z[BOX];
    __device__ __forceinline__ V3<double> get(int q) const
    {
        const XY v = xy[q];
        return V3<double>{v.x, v.y, z[q]};
    }
    __device__ __forceinline__ void put(int q, const V3<double>& v)
    {
        xy[q] = XY{v.x, v.y};
        z[q] = v.z;
    }
};

// Slot of box cell (x, y, z): planes of BX x BY, so that the lanes of a wave
// (8 x 8 cells of one plane) read whole rows of consecutive slots.
__device__ __forceinline__ int box_slot(int x, int y, int z) { return (z * BY + y) * BX + x; }

// Couplings of a column in LDS: 2 kLongReach + 1, padded to whole 16 bytes.
template <typename R>
constexpr int kJStride = sizeof(R) == 4 ? 12 : 10;

// The links of a column with |dz| <= HZ on the lane's TZ sites: q is the
// slot of the column's cell at the tile's first plane.
template <typename R, int HZ>
__device__ __forceinline__ void column(const LongBox<R>& box, int q, const R* J, V3<R> acc[TZ])
{
    R j[2 * HZ + 1];
#pragma unroll
    for (int k = 0; k <= 2 * HZ; ++k)
        j[k] = J[k];
#pragma unroll
    for (int u = -HZ; u < TZ + HZ; ++u) {
        const V3<R> v = box.get(q + u * (BX * BY));
#pragma unroll
        for (int t = 0; t < TZ; ++t) {
            const int dz = u - t;
            if (dz < -HZ || dz > HZ)
                continue;
            acc[t].x = fma(j[dz + HZ], v.x, acc[t].x);
            acc[t].y = fma(j[dz + HZ], v.y, acc[t].y);
            acc[t].z = fma(j[dz + HZ], v.z, acc[t].z);
        }
    }
}

// `count` columns of reach HZ from column c on; returns the column after.
template <typename R, int HZ>
__device__ __forceinline__ int columns(const LongBox<R>& box, int q0, const int32_t* off, const R* J, int c, int count,
                                       V3<R> acc[TZ])
{
#pragma unroll 2
    for (int e = c + count; c < e; ++c)
        column<R, HZ>(box, q0 + off[c], J + kJStride<R> * c, acc);
    return c;
}

__device__ __forceinline__ int wrap_near(int u, int n)
{
    u += u < 0 ? n : 0;
    u -= u >= n ? n : 0;
    u -= u >= n ? n : 0;
    return u;
}

// PHASE 0 the predictor of step k (S' into Sp; m and E terms of the state it
// reads), 1 the corrector, 2 the m and E sums of the state after the chunk
// (k < 0: the current state).  Items as in brick.hip.
template <typename R, int PHASE>
__global__ __launch_bounds__(BT) void k_long(const ReplicaDev<R>* __restrict__ reps,
                                             const FusedItem* __restrict__ items, const int* __restrict__ n_items,
                                             int k, int remap)
{
    // the box, and in the same memory once it has been read the waves' parts
    // of the sums (three FP32 or two FP64 workgroups fit a compute unit)
    __shared__ __attribute__((aligned(16))) char mem[sizeof(LongBox<R>)];
    static_assert(sizeof(R) * WAVES * 3 * BT <= sizeof(LongBox<R>), "the parts fit the box's memory");
    LongBox<R>& box = *reinterpret_cast<LongBox<R>*>(mem);
    R(*part)[3][BT] = reinterpret_cast<R(*)[3][BT]>(mem);
    __shared__ __attribute__((aligned(16))) R l_J[kLongColumns * kJStride<R>];
    __shared__ int32_t l_off[kLongColumns];
    __shared__ double red[4][WAVES];
    const int t = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int W = *n_items;
    bool first = true;
    int staged = -1;
    int32_t head[6];   // this wave's first column, then its columns of reach 4 .. 0
    for (TileIter it(W, remap); it.more(); it.next()) {
        const FusedItem w = items[it.t];
        const ReplicaDev<R>& r = reps[w.replica];
        const int32_t flags = r.flags;
        const int nsteps = r.nsteps;
        if (PHASE == 2 ? (!(flags & kRecord) || nsteps <= 0) : k >= nsteps)
            continue;   // uniform over the block
        if (!first)
            __syncthreads();   // every thread is done with the previous item's LDS
        first = false;
        if (w.z1 < 0) {
            if (PHASE == 0 && (flags & kRecord) && k >= 2)
                item_record<R, BT, false>(r, (k - 1) & 1, k - 2, red);
            continue;
        }
        const int mslot = PHASE == 2 ? (k < 0 ? 0 : nsteps) : k;
        const int par = (r.parity + mslot) & 1;
        const R* __restrict__ S = PHASE == 1 ? (const R*)r.Sp : (const R*)r.S[par];
        const int nx = r.f_nx, ny = r.f_ny, nz = r.f_nz;
        // a thread's box cells: one x and y row position, every plane pair
        {
            const int x = t & (BX - 1), y = t / BX;   // BX x BY cells are BT
            static_assert(BX * BY == BT && (BX & (BX - 1)) == 0, "a thread per cell of a box plane");
            const int col = wrap_near(w.x0 - H + x, nx) + nx * wrap_near(w.y0 - H + y, ny);
#pragma unroll
            for (int z = 0; z < BZ; ++z)
                box.put(box_slot(x, y, z), load3(S, col + (int64_t)nx * ny * wrap_near(w.z0 - H + z, nz)));
        }
        if (w.replica != staged) {
            const int nc = r.l_columns;
            for (int q = t; q < nc * (2 * H + 1); q += BT)
                l_J[kJStride<R> * (q / (2 * H + 1)) + q % (2 * H + 1)] = gload(r.l_J, q);
            if (t < nc)
                l_off[t] = gload(r.l_head, kLongHead + t);
#pragma unroll
            for (int q = 0; q < 6; ++q)
                head[q] = __builtin_amdgcn_readfirstlane(gload(r.l_head, 8 * wave + q));
            staged = w.replica;
        }
        // the site this thread finishes: lane's column, plane `wave`
        const int lx = lane & (TX - 1), ly = lane / TX;
        const int ux = w.x0 + lx, uy = w.y0 + ly, uz = w.z0 + wave;
        const bool own = ux < nx && uy < ny && uz < nz;
        const int site = wrap_near(ux, nx) + nx * (wrap_near(uy, ny) + ny * wrap_near(uz, nz));
        const MaterialDev<R> m = uniform_material(r);
        V3<R> s0{0, 0, 0};
        if (PHASE == 1 && own)
            s0 = load3_once((const R*)r.S[par], site);
        R gn[3] = {0, 0, 0};
        if (PHASE != 2 && m.sigma != (R)0 && own)
            thermal_normals(r.seed, r.step + (uint64_t)k, (uint32_t)site, gn);
        __syncthreads();   // the box is complete
        V3<R> acc[TZ];
#pragma unroll
        for (int j = 0; j < TZ; ++j)
            acc[j] = V3<R>{0, 0, 0};
        {
            // this wave's columns, by reach
            const int q0 = box_slot(lx + H, ly + H, H);
            int c = head[0];
            c = columns<R, 4>(box, q0, l_off, l_J, c, head[1], acc);
            c = columns<R, 3>(box, q0, l_off, l_J, c, head[2], acc);
            c = columns<R, 2>(box, q0, l_off, l_J, c, head[3], acc);
            c = columns<R, 1>(box, q0, l_off, l_J, c, head[4], acc);
            columns<R, 0>(box, q0, l_off, l_J, c, head[5], acc);
        }
        const V3<R> s = box.get(box_slot(lx + H, ly + H, wave + H));
        __syncthreads();   // every thread has read the box
#pragma unroll
        for (int j = 0; j < TZ; ++j) {
            part[wave][0][64 * j + lane] = acc[j].x;
            part[wave][1][64 * j + lane] = acc[j].y;
            part[wave][2][64 * j + lane] = acc[j].z;
        }
        __syncthreads();
        V3<R> sum{0, 0, 0};
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            sum.x += part[v][0][t];
            sum.y += part[v][1][t];
            sum.z += part[v][2][t];
        }
        const V3<R> e{m.axis[0], m.axis[1], m.axis[2]};
        const V3<R> Happ{r.H[0], r.H[1], r.H[2]};
        const V3<R> hex{m.mu_rel * sum.x, m.mu_rel * sum.y, m.mu_rel * sum.z};
        const R se = dot(s, e);
        if (PHASE != 2 && own) {
            V3<R> h{hex.x + m.ani * se * e.x + Happ.x, hex.y + m.ani * se * e.y + Happ.y,
                    hex.z + m.ani * se * e.z + Happ.z};
            h.x = fma(m.sigma, gn[0], h.x);
            h.y = fma(m.sigma, gn[1], h.y);
            h.z = fma(m.sigma, gn[2], h.z);
            const V3<R> ds = llg_step(s, h, r.gdt, r.alpha);
            if (PHASE == 0) {
                store3(r.Sp, site, normalised(V3<R>{s.x + ds.x, s.y + ds.y, s.z + ds.z}));
            } else {
                // S + dS dt / 2 from S and S' (k_correct in kernels.hip)
                const R c = (R)0.5 * recip(dot(s0, s));
                const V3<R> sn = normalised(V3<R>{(R)0.5 * s0.x + c * s.x + (R)0.5 * ds.x,
                                                  (R)0.5 * s0.y + c * s.y + (R)0.5 * ds.y,
                                                  (R)0.5 * s0.z + c * s.z + (R)0.5 * ds.z});
                store3(r.S[par ^ 1], site, sn);
                if (!spin_ok(sn))
                    flag_fault(r.fault);
            }
        }
        if (PHASE != 1 && (flags & kRecord) && (PHASE == 2 || k >= 1)) {
            const R u = (R)0.5 * dot(s, hex) + m.ku_mu * se * se + dot(s, Happ);
            const double v[4] = {own ? (double)(m.mu_frac * s.x) : 0.0, own ? (double)(m.mu_frac * s.y) : 0.0,
                                 own ? (double)(m.mu_frac * s.z) : 0.0, own ? (double)(m.mu_frac * u) : 0.0};
            double out[4];
            sum4_256<BT>(v, out, red);
            if (t == 0) {
                double* p = r.f_partials + 4 * ((int64_t)(mslot & 1) * r.f_items + w.idx);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    p[c] = out[c];
            }
        }
    }
}

}  // namespace

int long_slot_offset(int dx, int dy) { return dy * BX + dx; }

void long_cells(int cells[3])
{
    cells[0] = TX;
    cells[1] = TY;
    cells[2] = TZ;
}

template <typename R>
hipError_t launch_long(const ReplicaDev<R>* reps, const FusedItem* items, const int* n_items, int grid, int k,
                       int remap, bool measure, hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    if (measure) {
        hipLaunchKernelGGL((k_long<R, 2>), dim3(grid), dim3(BT), 0, st, reps, items, n_items, k, remap);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_long<R, 0>), dim3(grid), dim3(BT), 0, st, reps, items, n_items, k, remap);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((k_long<R, 1>), dim3(grid), dim3(BT), 0, st, reps, items, n_items, k, remap);
    return hipGetLastError();
}

template <typename R>
int long_resident_blocks(int device)
{
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0 ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void*)k_long<R, 0>, BT, 0) != hipSuccess)
        return 0;
    return cus * per;
}

template hipError_t launch_long<float>(const ReplicaDev<float>*, const FusedItem*, const int*, int, int, int, bool,
                                       hipStream_t);
template hipError_t launch_long<double>(const ReplicaDev<double>*, const FusedItem*, const int*, int, int, int, bool,
                                        hipStream_t);
template int long_resident_blocks<float>(int);
template int long_resident_blocks<double>(int);

}  // namespace sllg
