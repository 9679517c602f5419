// Host-side preparation of a spin system for the device: validation of the
// caller's CSR neighbour list and material arrays, conversion of the CSR to
// the SELL-64 layout the step kernels read, and the material table.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/sllg.h"
#include "layout.hpp"

namespace sllg {

// Internal failure carrying an ABI status; caught at the C boundary.
struct Failure {
    sllg_status code;
    std::string msg;
};

[[noreturn]] void fail(sllg_status code, const std::string& msg);

// Boltzmann constant (J/K), Table 1 of the paper.
constexpr double kBoltzmann = 1.3807e-23;
// Bohr magneton (J/T), Table 1 of the paper.
constexpr double kBohrMagneton = 9.2740e-24;

// Macrocell decomposition for the demagnetising field: cubic cells of edge
// cell_size on a grid that starts a thousandth of a cell below the smallest
// atom coordinate on each axis (atomic planes on a cell boundary go to the
// upper cell); cells are numbered in the order of (x, y, z) cell index.
struct HostDemag {
    bool on = false;
    double cell_size = 0.0, atom_volume = 0.0;
    int64_t every = 1;
    int64_t cells = 0;
    std::vector<double> pos;           // [3n] atom positions relative to the grid corner (m)
    std::vector<int32_t> cell_of;      // [n]
    std::vector<int32_t> start;        // [cells + 1]
    std::vector<int32_t> atoms;        // [n] sites sorted by cell, ascending within a cell
};

// Source chunks of the demagnetising-field update: enough workgroups
// (blocks of 256 cells x chunks, about 2048) to fill the chip, at most 32.
inline int demag_chunks(int64_t cells)
{
    const int64_t blocks = (cells + 255) / 256;
    const int64_t c = (2048 + blocks - 1) / (blocks > 0 ? blocks : 1);
    return (int)(c < 1 ? 1 : (c > 32 ? 32 : c));
}

// Validates and builds the decomposition (pos: 3n metres).
HostDemag build_demag(int64_t n, const double* pos, double cell_size, double atom_volume, int64_t every);

// A lattice declared cell by cell (sllg_set_lattice): site
// i = b + nb (x + nx (y + ny z)); every link joins cells at most one cell
// apart on each axis (across the boundary of a periodic axis).  The fused
// step keeps one link pattern per (plane, basis site).
struct FusedLink {
    int8_t dz, dy, dx;      // cell offset of the neighbour
    uint8_t bp;             // its basis site
    uint8_t type;           // interaction type
    bool operator<(const FusedLink& o) const
    {
        if (dz != o.dz) return dz < o.dz;
        if (dy != o.dy) return dy < o.dy;
        if (dx != o.dx) return dx < o.dx;
        if (bp != o.bp) return bp < o.bp;
        return type < o.type;
    }
    bool operator==(const FusedLink& o) const
    {
        return dz == o.dz && dy == o.dy && dx == o.dx && bp == o.bp && type == o.type;
    }
};

struct HostLattice {
    bool on = false;
    int nb = 0, nx = 0, ny = 0, nz = 0;
    bool per[3] = {false, false, false};
    bool fusable = false;                       // the fused step can run on this structure
    std::string why;                            // why not, when it cannot
    std::vector<std::vector<FusedLink>> pats;   // link patterns, each sorted (dz first)
    std::vector<uint8_t> pat_b;                 // basis site of each pattern
    std::vector<uint8_t> plane_pat;             // [nz * nb] pattern of each (plane, basis site);
                                                // empty when the pattern is the basis site itself
    int kind = 0;                               // FusedKind whose links every site has (kKindGeneric: none)
    int slot_type[2] = {0, 0};                  // interaction type of each of the kind's slots
};

// Sets the error text of the calls without a handle (sllg_last_error(NULL)).
void set_create_error(const std::string& msg);

// Whether the fused step is built for lattice L of n sites in a precision
// (bytes per real): FP32 any fusable lattice, FP64 the compiled kinds; the
// spins must be addressable with 31-bit byte offsets.
inline bool fused_precision_ok(const HostLattice& L, int64_t n, size_t real_bytes)
{
    return L.on && L.fusable && (real_bytes == 4 || L.kind != kKindGeneric) && n * 3 * (int64_t)real_bytes + 16 <= 0x7FFFFFFF;
}

// Neighbour structure in stencil or SELL-64 form.  Every row lists its
// near links (|col - row| <= halo_cap) first and the far ones after, each
// part in the caller's order; the step kernels sum the two parts separately
// (near ones from the LDS window), so both forms add the same terms in the
// same order.
struct HostStructure {
    int64_t n = 0;
    int64_t nnz = 0;
    int n_types = 0;
    int halo = 0;                      // window halo: max near |col - row|, rounded up to 4
    int tile_request = 0;              // sites per tile: 0 from n (tile_for), -1 the largest, else this
    std::vector<double> J;             // joules per link, per type
    // exchange tensors (set_exchange_tensors): 9 per type, row-major, joules
    bool tensor = false;
    std::vector<double> Jt;
    // reverse[t] bit u: some link of type t has its reverse link of type u
    // (recorded by the symmetry check; rev_known = false without it)
    bool rev_known = false;
    uint16_t reverse[kMaxTypes] = {};
    std::vector<uint32_t> nb;          // packed entries, 64 rows per slice, column-major
    std::vector<int64_t> slice_off;    // [n_slices + 1]
    std::vector<uint32_t> deg;         // [n] near << 16 | degree
    bool long_rows = false;            // SELL rows longer than kLongRow links
    // stencil form, filled when every row matches one of few patterns
    bool stencil = false;
    std::vector<uint8_t> pat_id;       // [n]
    std::vector<int32_t> pat_tab;      // packed (col - row) << 4 | type
    std::vector<uint16_t> pat_start;   // [n_patterns + 1]
    std::vector<uint16_t> pat_far;     // [n_patterns] first far entry of each pattern
    bool no_far = false;               // no pattern has a far link (no padding then)
    // wide stencil form, filled when the patterns exceed the LDS tables
    // (kMaxPatterns, kMaxPatternEntries) but not kWideMaxPatterns /
    // kWideMaxEntries: the table stays in global memory
    bool wide = false;
    int w_len = 0;                     // entries of the longest pattern (a multiple of kWideBatch)
    std::vector<uint16_t> w_pid;       // [n] pattern of each site
    std::vector<int32_t> w_tab;        // [w_len][patterns] packed (col - row) << 5 | type: the near links,
                                       // padded to kWideBatch, then the far ones, padded (type kMaxTypes)
    std::vector<uint16_t> w_near;      // [patterns] near entries of each pattern with their padding
    // macrocell demagnetising field (set_demag)
    HostDemag demag;
    // Monte Carlo colour classes (build_colours): sites sorted by colour
    std::vector<int32_t> colour_sites;
    std::vector<int64_t> colour_start;   // [n_colours + 1]
    // lattice declaration and fused-step patterns (set_lattice)
    HostLattice lat;
    // brick step: link words per site class (ReplicaDev::b_links) and the
    // pairs in use; empty when the lattice or its rows do not allow it
    std::vector<uint32_t> brick_words;
    int brick_near = 0, brick_far = 0;
    // long-range step: the simple-cubic lattice found in the wide form's rows
    // (kind kKindLong) and its columns of links; off when there is none
    HostLattice far;
    struct LongColumn {
        int dx = 0, dy = 0, reach = 0;
        int type[2 * kLongReach + 1];   // by dz + kLongReach; -1: no link
    };
    std::vector<LongColumn> columns;
};

// Fills s.far and s.columns when the wide form's rows are those of a
// simple-cubic lattice, site i = x + nx (y + ny z), periodic on every axis
// with at least 2 kLongReach + 1 cells, whose sites all have the same links
// (cell offsets and types) at most kLongReach cells away on each axis.
// Every pattern and every site's pattern is checked.
void detect_long(HostStructure& s);

// Largest lattice the brick tables are made for (sites); from kFusedMinSpins
// on the fused step is the default.
constexpr int64_t kBrickMaxSites = int64_t(1) << 20;

// Whether the brick step is faster than the two-launch step on a lattice of n
// spins of one of its kinds, below the fused step's size.  What counts is the
// bricks, not the spins: on thin films, rods and lattices that cut them they
// are partly empty, and a brick costs nearly as much.  Measured us per step,
// brick and two-launch, 300 K with records:
//  - second neighbours: two bricks fill a compute unit's LDS in FP32 and one
//    does in FP64, so beyond one brick per unit a launch takes half as long
//    again: FP32 9.0 and 11.5 with 256 bricks (65,536 spins), 13.6 and 11.9
//    with 405 (93,312), 25.6 and 12.4 with 950 (5 x 5 x 1900 cells); FP64 12.7
//    and 14.9, 20.2 and 15.6, 37.5 and 16.9.
//  - nearest neighbours: the launch's share of a brick, and of the two-launch
//    step's sites, are lines through the measurements.  FP32: simple cubic
//    9.7 and 13.2 (64^3), 24.9 and 29.0 (96^3), 33.8 and 30.9 (101^3), 62.7
//    and 31.0 (5 x 5 x 40000), 67 and 30.0 (1000 x 1000 x 1), 6.9 and 10.7
//    (256 x 256 x 1); bcc 19.7 and 20.3 (64^3), 36.1 and 32.3 (80^3), 49 and
//    19.2 (512 x 512 x 1).  FP64: 18.3 and 19.9, 50.4 and 50.6, 63 and 61.7,
//    137 and 60.1, 137 and 58.0, 10.6 and 13.7; 32.9 and 34.2, 61.4 and 64.2,
//    69.8 and 33.0.  A film of one layer costs about 5/8 of a full brick.
bool brick_pays(const HostLattice& L, int64_t n, size_t real_bytes);

// Whether the long-range step is faster than the wide two-launch step on a
// structure that detect_long accepted.  It copies 12 box spins a site and
// walks the columns whatever the links, the wide form reads every link of
// every site; and like the bricks its tiles can be partly empty.  The four
// lines are fits through 15 sets of 12 to 388 links on 729 to 884,736 spins
// (us per step; within a tenth, on average, of the measurements), the long
// one raised by a twenty-fifth so that a close call goes to the two-launch
// step.  Measured, long-range and two-launch, FP32: 12 links 14.6 and 11.6
// (24^3), 68 and 36 (96^3); 24 links 16.8 and 16.0 (48^3), 45.6 and 31.9
// (80^3); 56 links 16.9 and 20.4 (48^3), 75 and 67 (96^3); 146 links 17.4 and
// 33.1 (16^3), 90 and 154 (96^3), 71 and 48 (9 x 9 x 3000); 388 links 27.3 and
// 72.1 (48^3).  FP64: 12 links 13.0 and 16.7 (16^3), 87 and 67 (96^3); 24
// links 20.0 and 21.8 (48^3), 91 and 83 (96^3); 146 links 125 and 281 (96^3),
// 104 and 65 (9 x 9 x 3000).
bool long_pays(const HostStructure& s, size_t real_bytes);

// Whether the brick step can run on the structure in a precision (bytes per
// real).  Its tables (set_lattice) exist for a compiled kind with at least kBrickMinEdge cells per periodic axis in which every
// site of a class lists its links in the same order.
inline bool brick_ok(const HostStructure& s, size_t real_bytes)
{
    return (!s.brick_words.empty() || s.far.on) && s.n * 3 * (int64_t)real_bytes + 16 <= 0x7FFFFFFF;
}

// Declares the structure's sites as a lattice of nb sites per cell on
// cells[0] x cells[1] x cells[2] cells (periodic[a] != 0: periodic axis) and
// derives the fused step's link patterns.  Throws Failure(SLLG_E_ARG) when
// the counts do not match or a link joins cells more than one cell apart;
// otherwise sets s.lat (fusable false, with the reason, when the fused step
// cannot take the structure: open x or y, patterns that change within a
// plane, more than 2 sites per cell, too many patterns).
void set_lattice(HostStructure& s, int nb, const int cells[3], const int periodic[3]);

// Sites per tile of this structure at a precision (see tile_request).
int tile_of(const HostStructure& s, size_t real_bytes);

// Validates and converts.  Throws Failure(SLLG_E_ARG) on malformed input.
// allow_stencil = false keeps the SELL form even when patterns would fit
// (LDS stencil or wide stencil).
// halo_cap (a multiple of 4) bounds the offsets read from the LDS window.
HostStructure build_structure(int64_t n, const int64_t* row_ptr, const int32_t* col,
                              const uint8_t* ntype, const double* J, int n_types,
                              bool check_symmetry, int halo_cap, bool allow_stencil = true);

// Exchange tensors for the types of s (n_types must match).  With the
// symmetry check's record, every link of type t whose reverse has type u
// needs Jt[u] = Jt[t]^T, so the energy -S_i^T J_ij S_j is the same read
// from either end.  Jt = NULL returns to the scalar table.
void set_exchange_tensors(HostStructure& s, const double* Jt, int n_types);

// Greedy colouring of the neighbour graph for Monte Carlo: the sites are
// visited in ascending order, or (lattice_order, on a declared lattice)
// grouped by basis site and by the parity of the cell's x + y + z, each
// taking the smallest colour no earlier-visited neighbour has (so no link
// joins two sites of one colour); fills colour_sites / colour_start.
void build_colours(HostStructure& s, bool lattice_order);

// Materials: distinct (mu_s, k_u, k_c) triples, per-site ids when there is
// more than one, per-site easy axes when they differ.
struct HostMaterials {
    int64_t n = 0;
    std::vector<double> mat_mu;        // J/T per material
    std::vector<double> mat_ku;        // J per material
    std::vector<double> mat_kc;        // J per material (cubic anisotropy)
    bool cubic = false;                // some k_c != 0
    double axis[3] = {0, 0, 1};        // uniform easy axis (when !per_site_axis)
    std::vector<uint8_t> matid;        // [n] when per_site_material
    std::vector<double> axis_site;     // [3n] when per_site_axis
    bool per_site_material = false;
    bool per_site_axis = false;
    double mu_ref = 0.0;               // reference moment for the field units
    double mu_total = 0.0;             // sum over sites of mu_s
};

// Per demagnetising macrocell: magnetic centre of mass sum mu x / sum mu (3
// per cell, relative to the grid corner) and the self-field factor
// mu0 / (3 V), V = atoms * atom_volume.
void demag_cells(const HostDemag& dm, const HostMaterials& m, std::vector<double>& centre,
                 std::vector<double>& self);

// k_c: cubic anisotropy, n values when kc_per_site, else one (NULL: none).
HostMaterials build_materials(int64_t n, const double* mu_s, const double* k_u,
                              const double* easy_axis, int per_site, const double* k_c = nullptr,
                              int kc_per_site = 0);

// Validate spins (3n doubles; throws on zero or non-finite length) and
// normalise them, or with normalise = false copy them unchanged (a restored
// checkpoint continues bit for bit).
std::vector<double> normalised_spins(int64_t n, const double* S, bool normalise = true);

// Integration parameters of one replica.
struct Dynamics {
    double alpha = -1.0, gamma = -1.0, dt = -1.0;
    double temperature = 0.0;
    double H[3] = {0.0, 0.0, 0.0};
    uint64_t seed = 0;
    uint64_t step = 0;
};

void check_dynamics(const Dynamics& d);

// Device material table for the current dynamics (thermal width depends on
// lambda, T, gamma and dt).
template <typename R>
std::vector<MaterialDev<R>> material_table(const HostMaterials& m, const Dynamics& d);

// Fill the parameter part of a replica record (J table, gamma dt, field, ...).
template <typename R>
void fill_parameters(ReplicaDev<R>& rec, const HostStructure& s, const HostMaterials& m,
                     const Dynamics& d);

// Whether a replica can take the fused and brick steps as far as its
// interactions go: one material, scalar exchange, no cubic anisotropy or
// demagnetising field.
inline bool plain_interactions(const HostStructure& s, const HostMaterials& m)
{
    return !m.per_site_material && !m.per_site_axis && !s.tensor && !m.cubic && !s.demag.on;
}

// Thermal averages from per-block sums acc[b][5] = sums of (|m|, m_x, m_y,
// m_z, E) over block_len samples each: out = { <|m|>, se, <m_x>, <m_y>,
// <m_z>, <E>, se(E), n_blocks }, se = std of the block means / sqrt(n_blocks).
void averages_from_block_sums(const double* acc, int n_blocks, int64_t block_len, double out[8]);

}  // namespace sllg
