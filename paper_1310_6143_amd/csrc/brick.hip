// Brick step of libsllg for gfx950: one launch per Heun step on small and
// middle-sized crystals (simple cubic, bcc, bcc with second neighbours;
// uniform material, scalar exchange).
//
// Paper (Evans et al., arXiv:1310.6143), "Time Integration of the LLG
// Equation": every predictor before any corrector.  A workgroup owns a brick
// of TX x TY x TZ cells, copies the spins of the brick and of the sites
// around it that its steps reach into LDS, takes the predictor on the brick
// and on its neighbours (one site per thread, a single round), and after one
// barrier the corrector on the brick.  The predictor of a brick's neighbours
// is recomputed by every brick that touches them, so no workgroup needs
// another's results within a launch.
//
// What bounds it: below about 2^18 spins a launch is a chain of latencies
// (launch 1.6 us, table and spin reads, noise, two exchange sums), not
// bandwidth or arithmetic.  The two-launch step pays that chain twice, each
// with a table staging and two further reductions; here it is paid once, the
// noise is drawn while the spin reads are in flight, and the m and E sums
// run on the waves that have no corrector to do.  The plane-marching step
// (fused.hip) recomputes less per site but walks its planes in series.
// Measured per step (FP32, 300 K, records every step, two-launch step before):
// 4,096 simple-cubic spins 12.7 -> 5.1 us, 262,144 15.2 -> 9.0, 65,536 bcc
// spins 13.0 -> 5.3, 524,288 23.1 -> 17.0; FP64 16.5 -> 6.8, 19.7 -> 16.7,
// 16.0 -> 7.3 and 35.5 -> 28.8.
// The terms, their order and the formulas are those of the two-launch step
// (kernels.hip), so the spins are the same bits whichever of the two runs.
// For that a site's links come from a table by class (basis site, first,
// inner or last cell on each axis) that holds its row's order, not from the
// kind's constants (which took 4.5 us for the 4,096 spins: FP32 trajectories
// above room temperature part from a rounding difference by 1e-3 of a spin
// component within 2000 steps, so one set of roundings is kept).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "device_common.hpp"
#include "kernels.hpp"
#include "layout.hpp"
#include "site_step.hpp"

namespace sllg {
namespace {

using namespace dev;

// Brick shape of a kind: cells per axis, threads, and the cells the S box
// reaches beyond the brick (two links).  The predictor sites (brick first,
// in whole waves per basis site, then its neighbours in whole waves per
// basis site) fill the workgroup in one round: 256 + 256 sites for simple
// cubic 8 x 8 x 4, 256 + 194 for bcc 8 x 4 x 4, 256 + 354 with second
// neighbours.
template <int KIND>
struct Brick {
    static constexpr int NB = kind_basis(KIND);
    static constexpr int TX = 8, TY = KIND == kKindSc6 ? 8 : 4, TZ = 4;
    static constexpr int BT = KIND == kKindBcc14 ? 640 : 512;
    static constexpr int H = KIND == kKindBcc8 ? 1 : 2;   // bcc sites reach half a cell per link
    static constexpr int SX = TX + 2 * H, SY = TY + 2 * H, SZ = TZ + 2 * H, VOL = SX * SY * SZ;
    static constexpr int OWN = NB * TX * TY * TZ;
    static constexpr int PAIRS = brick_pairs(KIND);       // link words of a class: near, then far
    static constexpr int WORDS = (2 * PAIRS + 3) & ~3;    // in whole 16-byte loads
    static constexpr int LOADS = (NB * VOL + BT - 1) / BT;   // table rounds (pruned entries are invalid)
    static_assert(OWN == 256, "the record sums take 256 brick sites, four waves");
    static_assert(NB * VOL <= 4096, "slots fit the table entries");
};

// Table entry: slot in the S box (basis-major) << 16 | z << 10 | y << 5 | x of
// its cell within the box; bit 15 clear.  kNone: nothing to do.
constexpr uint32_t kNone = 0xFFFFFFFFu;

// x, y, z of a box slot.  FP32: 16 bytes per slot, read and written as one
// vector (as three words they may become 4-byte reads at a 16-byte stride, a
// fourfold bank conflict: 21.0 against 15.0 us per step on 221,184 bcc spins
// with second neighbours, links by constants).  FP64: x, y in one array and z in another.
template <typename R, int SLOTS>
struct Box;
template <int SLOTS>
struct Box<float, SLOTS> {
    typedef float Slot __attribute__((ext_vector_type(4)));
    Slot s[SLOTS];
    __device__ __forceinline__ V3<float> get(int q) const
    {
        const Slot v = s[q];
        return V3<float>{v.x, v.y, v.z};
    }
    __device__ __forceinline__ void put(int q, const V3<float>& v) { s[q] = Slot{v.x, v.y, v.z, 0.0f}; }
};
template <int SLOTS>
struct Box<double, SLOTS> {
    typedef double XY __attribute__((ext_vector_type(2)));
    XY xy[SLOTS];
    double z[SLOTS];
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

// Cell u of an axis of n >= kBrickMinEdge cells, u in [-2, n + 9].
__device__ __forceinline__ int wrap_near(int u, int n)
{
    u += u < 0 ? n : 0;
    u -= u >= n ? n : 0;
    u -= u >= n ? n : 0;
    return u;
}

// Exchange sum of the site at slot q from its class's link words: the near
// links in row order, the far ones in row order, then their sum, as the
// two-launch step adds them (links past a class's own are padding, J = 0).
template <typename R, int KIND, typename BoxT>
__device__ __forceinline__ V3<R> box_links(const BoxT& box, int q, const uint32_t words[Brick<KIND>::WORDS],
                                           int near, int far, const R kj[2])
{
    constexpr int P = Brick<KIND>::PAIRS;
    // every read of a part is issued before the first is used
    auto part = [&](const uint32_t* w, int pairs) {
        V3<R> v[2 * P], h{0, 0, 0};
        auto half = [&](int k) { return k & 1 ? (int)w[k / 2] >> 16 : (int)(int16_t)(w[k / 2] & 0xFFFFu); };
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (j < pairs) {
                v[2 * j] = box.get(q + (half(2 * j) >> 2));
                v[2 * j + 1] = box.get(q + (half(2 * j + 1) >> 2));
            }
#pragma unroll
        for (int j = 0; j < P; ++j)
            if (j < pairs)
#pragma unroll
                for (int k = 2 * j; k < 2 * j + 2; ++k) {
                    const int code = half(k) & 3;
                    const R J = code == 0 ? kj[0] : KIND == kKindBcc14 && code == 1 ? kj[1] : (R)0;
                    h.x = fma(J, v[k].x, h.x);
                    h.y = fma(J, v[k].y, h.y);
                    h.z = fma(J, v[k].z, h.z);
                }
        return h;
    };
    const V3<R> hn = part(words, near), hf = part(words + P, far);
    return V3<R>{hn.x + hf.x, hn.y + hf.y, hn.z + hf.z};
}

// Adds the thermal field sigma * g.
template <typename R>
__device__ __forceinline__ void add_thermal(const MaterialDev<R>& m, const R g[3], V3<R>& h)
{
    if (m.sigma != (R)0) {
        h.x += m.sigma * g[0];
        h.y += m.sigma * g[1];
        h.z += m.sigma * g[2];
    }
}

// Step k of every brick listed (MEASURE: the m and E sums of the state after
// the chunk's steps, or with k < 0 of the current state).  An item with
// z1 < 0 is a replica's record item: its workgroup adds the bricks' sums of
// the previous launch into the record two steps back, beside the bricks
// instead of before one of them.
template <typename R, int KIND, bool MEASURE>
__global__ __launch_bounds__(Brick<KIND>::BT) void k_brick(const ReplicaDev<R>* __restrict__ reps,
                                                           const FusedItem* __restrict__ items,
                                                           const int* __restrict__ n_items,
                                                           const uint32_t* __restrict__ table, int k, int remap)
{
    using G = Brick<KIND>;
    constexpr int BT = G::BT;
    __shared__ Box<R, G::NB * G::VOL> box_s, box_p;
    __shared__ R terms[4][G::OWN];
    __shared__ double red[4][BT / 64];
    const int t = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    // the thread's table entries: the same for every brick
    const uint32_t pe = gload(table, t);
    uint32_t le[G::LOADS];
#pragma unroll
    for (int j = 0; j < G::LOADS; ++j)
        le[j] = gload(table, (1 + j) * BT + t);
    const int W = *n_items;
    bool first = true;
    for (TileIter it(W, remap); it.more(); it.next()) {
        const FusedItem w = items[it.t];
        const ReplicaDev<R>& r = reps[w.replica];
        const int32_t flags = r.flags;
        const int nsteps = r.nsteps;
        if (MEASURE ? (!(flags & kRecord) || nsteps <= 0) : k >= nsteps)
            continue;   // uniform over the block
        if (!first)
            __syncthreads();   // every thread is done with the previous item's LDS
        first = false;
        if (w.z1 < 0) {
            if (!MEASURE && (flags & kRecord) && k >= 2)
                item_record<R, BT, false>(r, (k - 1) & 1, k - 2, red);
            continue;
        }
        const int mslot = MEASURE ? (k < 0 ? 0 : nsteps) : k;
        const int par = (r.parity + mslot) & 1;
        const R* __restrict__ S = r.S[par];
        const int nx = r.f_nx, ny = r.f_ny, nz = r.f_nz;
        const bool zper = r.f_zper != 0;
        // S of the box; sites beyond an open z surface are zero
#pragma unroll
        for (int j = 0; j < G::LOADS; ++j) {
            if (le[j] == kNone)
                continue;
            const int q = (int)(le[j] >> 16), b = G::NB == 1 ? 0 : (q >= G::VOL ? 1 : 0);
            const int x = wrap_near(w.x0 - G::H + (int)(le[j] & 31), nx);
            const int y = wrap_near(w.y0 - G::H + (int)((le[j] >> 5) & 31), ny);
            int z = w.z0 - G::H + (int)((le[j] >> 10) & 31);
            const bool exists = zper || (z >= 0 && z < nz);
            if (zper)
                z = wrap_near(z, nz);
            V3<R> v{0, 0, 0};
            if (exists)
                v = load3(S, b + (int64_t)G::NB * (x + nx * (y + ny * z)));
            box_s.put(q, v);
        }
        // the thread's predictor site, and its noise while the reads fly
        const bool has = pe != kNone;
        const int q = has ? (int)(pe >> 16) : G::VOL / 2, b = G::NB == 1 ? 0 : __builtin_amdgcn_readfirstlane(q >= G::VOL ? 1 : 0);
        const int ux = w.x0 - G::H + (int)(pe & 31), uy = w.y0 - G::H + (int)((pe >> 5) & 31);
        const int uz = w.z0 - G::H + (int)((pe >> 10) & 31);
        const bool exists = has && (zper || (uz >= 0 && uz < nz));
        const int zw = zper ? wrap_near(uz, nz) : uz;
        const uint32_t site = (uint32_t)b + (uint32_t)G::NB * (uint32_t)(wrap_near(ux, nx) + nx * (wrap_near(uy, ny) + ny * zw));
        const bool own = t < G::OWN && exists && ux < nx && uy < ny && uz < nz;
        const MaterialDev<R> m = uniform_material(r);
        const R kj[2] = {r.f_kj[0], r.f_kj[1]};
        const V3<R> e{m.axis[0], m.axis[1], m.axis[2]};
        const V3<R> Happ{r.H[0], r.H[1], r.H[2]};
        const bool rec = (flags & kRecord) && (MEASURE || k >= 1);
        // its links: those of its class (basis site, first, inner or last cell
        // of each axis)
        uint32_t words[G::WORDS];
        const int near = r.b_near, far = r.b_far;
        if (exists) {
            const int cls = b * 27 + edge_class(zw, nz) * 9 + edge_class(wrap_near(uy, ny), ny) * 3 +
                            edge_class(wrap_near(ux, nx), nx);
#pragma unroll
            for (int j = 0; j < G::WORDS; j += 4) {
                typedef uint32_t Word4 __attribute__((ext_vector_type(4)));
                const Word4 v = gload((const Word4*)r.b_links, cls * (G::WORDS / 4) + j / 4);
                words[j] = v.x;
                words[j + 1] = v.y;
                words[j + 2] = v.z;
                words[j + 3] = v.w;
            }
        }
        R gn[3] = {0, 0, 0};
        if (!MEASURE && m.sigma != (R)0 && exists)
            thermal_normals(r.seed, r.step + (uint64_t)k, site, gn);
        __syncthreads();   // S complete
        V3<R> s0{0, 0, 0}, spn{0, 0, 0};
        if (MEASURE ? own : exists) {
            s0 = box_s.get(q);
            const V3<R> sum = box_links<R, KIND>(box_s, q, words, near, far, kj);
            const V3<R> hex{m.mu_rel * sum.x, m.mu_rel * sum.y, m.mu_rel * sum.z};
            const R se = dot(s0, e);
            if (rec && own) {
                // in units of mu_ref: mu_s/mu_ref S and mu_s/mu_ref (-E_i/mu_s)
                const R u = (R)0.5 * dot(s0, hex) + m.ku_mu * se * se + dot(s0, Happ);
                terms[0][t] = m.mu_frac * s0.x;
                terms[1][t] = m.mu_frac * s0.y;
                terms[2][t] = m.mu_frac * s0.z;
                terms[3][t] = m.mu_frac * u;
            }
            if (!MEASURE) {
                V3<R> h{hex.x + m.ani * se * e.x + Happ.x, hex.y + m.ani * se * e.y + Happ.y,
                        hex.z + m.ani * se * e.z + Happ.z};
                add_thermal(m, gn, h);
                const V3<R> ds = llg_step(s0, h, r.gdt, r.alpha);
                spn = normalised(V3<R>{s0.x + ds.x, s0.y + ds.y, s0.z + ds.z});
            }
        }
        if (rec && t < G::OWN && !own)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                terms[c][t] = (R)0;
        if (!MEASURE && has)
            box_p.put(q, spn);
        __syncthreads();   // S' and the record terms complete
        if (t < G::OWN) {
            if (!MEASURE && own) {
                const V3<R> sum = box_links<R, KIND>(box_p, q, words, near, far, kj);
                const R se = dot(spn, e);
                V3<R> h{m.mu_rel * sum.x + m.ani * se * e.x + Happ.x, m.mu_rel * sum.y + m.ani * se * e.y + Happ.y,
                        m.mu_rel * sum.z + m.ani * se * e.z + Happ.z};
                add_thermal(m, gn, h);
                const V3<R> ds = llg_step(spn, h, r.gdt, r.alpha);
                // this sum's order is the one the two-launch corrector is compiled to
                const R c = (R)0.5 * recip(fma(s0.z, spn.z, fma(s0.x, spn.x, s0.y * spn.y)));
                const V3<R> half{(R)0.5 * s0.x + c * spn.x, (R)0.5 * s0.y + c * spn.y, (R)0.5 * s0.z + c * spn.z};
                const V3<R> sn = normalised(
                    V3<R>{half.x + (R)0.5 * ds.x, half.y + (R)0.5 * ds.y, half.z + (R)0.5 * ds.z});
                SLLG_GLOBAL R* dst = (SLLG_GLOBAL R*)r.S[par ^ 1] + 3 * (int64_t)site;
                dst[0] = sn.x;
                dst[1] = sn.y;
                dst[2] = sn.z;
                if (!spin_ok(sn))
                    flag_fault(r.fault);
            }
        } else if (rec && wave < G::OWN / 64 + 4) {
            // waves without a corrector: one record component each, the 256
            // brick sites added in a fixed order
            const int c = wave - G::OWN / 64;
            double v = (double)terms[c][lane];
#pragma unroll
            for (int j = 1; j < G::OWN / 64; ++j)
                v += (double)terms[c][lane + 64 * j];
            const double s = wave_sum(v);
            if (lane == 0)
                r.f_partials[4 * ((int64_t)(mslot & 1) * r.f_items + w.idx) + c] = s;
        }
    }
}

// Predictor and load tables of a kind: [BT] predictor entries, then LOADS x
// [BT] load entries.
template <int KIND>
std::vector<uint32_t> build_table()
{
    using G = Brick<KIND>;
    std::vector<char> pred(G::NB * G::VOL, 0), load(G::NB * G::VOL, 0);
    auto slot = [](int b, int x, int y, int z) { return b * G::VOL + ((z + G::H) * G::SY + y + G::H) * G::SX + x + G::H; };
    // sites within one link of the sites marked in `from`
    auto spread = [&](const std::vector<char>& from, std::vector<char>& to) {
        to = from;
        for (int b = 0; b < G::NB; ++b)
            for (int z = 0; z < G::SZ; ++z)
                for (int y = 0; y < G::SY; ++y)
                    for (int x = 0; x < G::SX; ++x) {
                        if (!from[(size_t)slot(b, x - G::H, y - G::H, z - G::H)])
                            continue;
                        for (int dz = -1; dz <= 1; ++dz)
                            for (int dy = -1; dy <= 1; ++dy)
                                for (int dx = -1; dx <= 1; ++dx)
                                    for (int bp = 0; bp < G::NB; ++bp) {
                                        int s = 0;
                                        if (kind_link(KIND, b, dz, dy, dx, bp, &s))
                                            to.at((size_t)slot(bp, x + dx - G::H, y + dy - G::H, z + dz - G::H)) = 1;
                                    }
                    }
    };
    std::vector<char> own(G::NB * G::VOL, 0);
    for (int b = 0; b < G::NB; ++b)
        for (int z = 0; z < G::TZ; ++z)
            for (int y = 0; y < G::TY; ++y)
                for (int x = 0; x < G::TX; ++x)
                    own[(size_t)slot(b, x, y, z)] = 1;
    spread(own, pred);
    spread(pred, load);
    std::vector<uint32_t> tab((size_t)(1 + G::LOADS) * G::BT, kNone);
    auto entry = [](int b, int x, int y, int z) {
        return (uint32_t)(b * G::VOL + (z * G::SY + y) * G::SX + x) << 16 | (uint32_t)z << 10 | (uint32_t)y << 5 | (uint32_t)x;
    };
    size_t at = 0, put = (size_t)G::BT;
    for (int ring = 0; ring < 2; ++ring)
        for (int b = 0; b < G::NB; ++b) {
            for (int z = 0; z < G::SZ; ++z)
                for (int y = 0; y < G::SY; ++y)
                    for (int x = 0; x < G::SX; ++x) {
                        const size_t q = (size_t)(b * G::VOL + (z * G::SY + y) * G::SX + x);
                        if (ring ? (pred[q] && !own[q]) : own[q])
                            tab.at(at++) = entry(b, x, y, z);
                    }
            at = (at + 63) / 64 * 64;   // the next basis site starts a wave
        }
    if (at > (size_t)G::BT)
        return {};
    // loads in memory order
    for (int z = 0; z < G::SZ; ++z)
        for (int y = 0; y < G::SY; ++y)
            for (int x = 0; x < G::SX; ++x)
                for (int b = 0; b < G::NB; ++b)
                    if (load[(size_t)(b * G::VOL + (z * G::SY + y) * G::SX + x)])
                        tab.at(put++) = entry(b, x, y, z);
    return tab;
}

}  // namespace

std::vector<uint32_t> brick_table(int kind)
{
    switch (kind) {
    case kKindSc6: return build_table<kKindSc6>();
    case kKindBcc8: return build_table<kKindBcc8>();
    case kKindBcc14: return build_table<kKindBcc14>();
    }
    return {};
}

BrickBox brick_box(int kind)
{
    switch (kind) {
    case kKindSc6: return {Brick<kKindSc6>::SX, Brick<kKindSc6>::SY, Brick<kKindSc6>::VOL, Brick<kKindSc6>::WORDS};
    case kKindBcc8: return {Brick<kKindBcc8>::SX, Brick<kKindBcc8>::SY, Brick<kKindBcc8>::VOL, Brick<kKindBcc8>::WORDS};
    case kKindBcc14:
        return {Brick<kKindBcc14>::SX, Brick<kKindBcc14>::SY, Brick<kKindBcc14>::VOL, Brick<kKindBcc14>::WORDS};
    }
    return {};
}

void brick_cells(int kind, int cells[3])
{
    cells[0] = 8;
    cells[1] = kind == kKindSc6 ? 8 : 4;
    cells[2] = 4;
}

template <typename R>
hipError_t launch_brick(const ReplicaDev<R>* reps, const FusedItem* items, const int* n_items, const uint32_t* table,
                        int grid, int k, int remap, bool measure, int kind, hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
#define SLLG_BRICK(K_)                                                                                              \
    if (kind == K_) {                                                                                               \
        if (measure)                                                                                                \
            hipLaunchKernelGGL((k_brick<R, K_, true>), dim3(grid), dim3(Brick<K_>::BT), 0, st, reps, items, n_items, \
                               table, k, remap);                                                                    \
        else                                                                                                        \
            hipLaunchKernelGGL((k_brick<R, K_, false>), dim3(grid), dim3(Brick<K_>::BT), 0, st, reps, items, n_items, \
                               table, k, remap);                                                                    \
        return hipGetLastError();                                                                                   \
    }
    SLLG_BRICK(kKindSc6)
    SLLG_BRICK(kKindBcc8)
    SLLG_BRICK(kKindBcc14)
#undef SLLG_BRICK
    return hipErrorInvalidValue;
}

template <typename R>
int brick_resident_blocks(int device, int kind)
{
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0)
        return 0;
    const void* f = kind == kKindSc6   ? (const void*)k_brick<R, kKindSc6, false>
                    : kind == kKindBcc8 ? (const void*)k_brick<R, kKindBcc8, false>
                                        : (const void*)k_brick<R, kKindBcc14, false>;
    const int bt = kind == kKindBcc14 ? Brick<kKindBcc14>::BT : Brick<kKindSc6>::BT;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, bt, 0) != hipSuccess)
        return 0;
    return cus * per;
}

#define SLLG_BRICK_INSTANTIATE(R)                                                                              \
    template hipError_t launch_brick<R>(const ReplicaDev<R>*, const FusedItem*, const int*, const uint32_t*, int, int, \
                                        int, bool, int, hipStream_t);                                          \
    template int brick_resident_blocks<R>(int, int);
SLLG_BRICK_INSTANTIATE(float)
SLLG_BRICK_INSTANTIATE(double)

}  // namespace sllg
