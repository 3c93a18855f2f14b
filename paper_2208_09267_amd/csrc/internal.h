// internal.h -- solver state shared by the host API (api.hip) and the kernel
// launchers (kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <string>

namespace vanse {

enum Mode { MODE_F64 = 0, MODE_F32S = 1, MODE_F16S = 2, MODE_FX16S = 3 };

// Launch-time view of one lattice: sizes and the population plane stride
// (elements between direction planes of the SoA population array).
struct Geometry {
    int nx, ny, nz;
    int nxy;
    int ncells;
    long long stride;
};

// Division by a launch-invariant divisor d (see fdiv in cell.h).
struct FastDiv {
    unsigned m;  // < 2^32 for every d >= 1
    unsigned s;
};

inline FastDiv make_fastdiv(unsigned d)
{
    unsigned l = 0;
    while ((1ull << l) < d) ++l;  // ceil(log2 d)
    FastDiv f;
    f.s = 31 + l;
    f.m = (unsigned)(((1ull << f.s) + d - 1) / d);
    return f;
}

// Everything one step of one solve needs, passed by value to the kernel.
struct StepArgs {
    Geometry geo;
    void *f;             // populations, SoA [Q][stride], storage type of the mode
    const void *pert;    // phi perturbation, double (FP64) or float (reduced)
    double eps_mean;     // phi = eps_mean + m * pert
    double shift;        // 16-bit modes: the unit c of the stored f_i / (c w_i) - 1
    double m;            // modulation m(n) of the current step
    double omega;        // 1 / tau
    double fcoef;        // 1 - omega / 2 (Guo forcing prefactor)
    double F[3];         // constant external force density
    double Fk[3];        // the same in the step kernels' units (16-bit modes: F / c)
    double fscale;       // per-cell force to the step kernels' units (16-bit modes: 1 / c)
    const void *force;   // optional per-cell force density, SoA [d][stride] (R), or null
    double wq;           // quadrature weight varpi_{i != 0}
    double n2;           // 2 * (number of quadrature axes)
    int qmask;           // quadrature axes bitmask
    // launch shape
    int row;             // 1: tiled (tile divides the lattice), 0: FLAT
    int flags;           // 1: nontemporal loads+stores, 2: XCD remap, 8: nontemporal stores
    unsigned block;      // threads per block
    unsigned nblocks;    // grid size
    unsigned tx, txlog;  // tiled: cells of one x-row segment per block (2^txlog, >= 64)
    unsigned ty;         // tiled: rows per block
    unsigned nseg;       // tiled: segments per x-row (nx / tx)
    unsigned nyb;        // tiled: row blocks per z-plane (ny / ty)
    FastDiv fd_nx, fd_ny, fd_seg, fd_nyb;
    // two-step launch (march.h): n -> n + 2 from f into f2
    void *f2;            // destination populations (natural order at n + 2)
    double m2;           // modulation m(n + 1) of the second step
    unsigned fty;        // full x-rows per tile
    unsigned fsz;        // z-planes per tile segment
    unsigned fnyb;       // tiles per z-segment (ny / fty; x-split tiles: times fnxb)
    FastDiv fd_fnyb;
    unsigned ftx;        // x-split general tiles: interior columns per tile (>= nx: full rows)
    unsigned fnxb;       //   and tiles per x-row
    FastDiv fd_fnxb;
    void *trash;         // 8-byte device slot for discarded stores
};

// One solve inside a batched launch (device-resident table).
struct BatchMember {
    StepArgs a;            // geometry, pointers and physics of the solve
    unsigned block_begin;  // first block of the solve in the batched grid
    unsigned nblocks;
};

struct Solver {
    int lattice = 0, mode = 0, d = 0, q = 0;
    Geometry geo{};
    double tau = 0.0;
    double eps_mean = 1.0, period = 0.0;
    double shift = 1.0;          // 16-bit modes: unit c of the encoding, set by vanse_init
    int qmask = 0;
    double F[3] = {0.0, 0.0, 0.0};
    bool porosity_set = false, initialized = false, unstable = false;
    // bumped by every setter of the step's physics (phi, forces), so that a
    // batch knows when its copy of the step parameters is stale
    unsigned long long gen = 0;
    int64_t t = 0;
    int tile_x = 256;            // step kernel tile: x-row segment per block
    int tile_y = 1;              //   and rows per block
    int flags = 0;               // step-kernel variant flags (StepArgs::flags)
    int user_flags = 0;          // those of vanse_set_tuning (the autotuner adds its own to them)
    bool allow_row = true;       // use the tiled launch when the tile divides the lattice
    void *f = nullptr;           // populations (current time level)
    size_t f_bytes = 0;
    int fused_rows = 0;          // two-step launch: x-rows per tile (0 = off)
    int fused_planes = 0;        //   and z-planes per segment
    int box = 0;                 // D2Q9: box kind of launches of several steps (0 = off)
    void *f_alt = nullptr;       // second population array of these launches
    void *pert = nullptr;        // phi perturbation (double or float)
    size_t pert_bytes = 0;
    void *force = nullptr;       // per-cell force density (double or float), optional
    size_t force_bytes = 0;
    bool force_on = false;
    double *scratch = nullptr;   // reduction partials + results
    size_t scratch_bytes = 0;
    hipStream_t stream = nullptr;
    std::string err;
};

constexpr int kReduceBlocks = 1024;   // fixed grid of the reduction kernels
constexpr int kReduceThreads = 256;
// scratch (doubles): reduction partials [7 * kReduceBlocks], and from
// kTrashSlot on a slot that discarded kernel stores may write
constexpr int kTrashSlot = 7 * kReduceBlocks + 32;

double modulation(int64_t n, double period);
StepArgs step_args(const Solver &s, int64_t n);

// Kernel launchers (kernels.hip).  Each returns the hipError_t of the launch.
hipError_t launch_step(const Solver &s, const StepArgs &a, int parity);
constexpr int kFusedThreads = 512;    // threads per block the tile rules count with
// general tiles of batches whose members are all narrow (nx <= 96, D3Q19,
// reduced storage): blocks of 768 threads, the tile and its two outer rows in
// one pass
constexpr int kGenThreads768 = 768;
constexpr int kFusedMaxLds = 160 * 1024;
// Tile shapes vanse_set_fused takes when nx is a multiple of 64 and the rows
// divide ny: ipt interior and hpt halo-plane cells per thread of a 512-thread
// block (wide: nx = 256 with 4 rows, which D3Q27 takes too).
constexpr bool fused_compiled(int lattice, int mode, int ipt, int hpt, bool wide)
{
    if (lattice == 0 || ipt < 1 || hpt < ipt) return false;
    if (lattice == 2)
        return mode != MODE_F64 && (ipt == 1 ? hpt <= 3 : (ipt == 2 && (hpt <= 2 || (wide && hpt == 3))));
    if (mode == MODE_F64) return ipt == 1 && hpt <= 2;
    return ipt <= 2 && hpt <= ipt + 2;
}
// The same for any nx and a shorter last tile.
constexpr bool fused_compiled_gen(int lattice, int mode, int ipt, int hpt)
{
    if (lattice == 0 || ipt < 1 || hpt < ipt) return false;
    if (lattice == 2) return mode != MODE_F64 && ipt == 1 && hpt <= 2;
    if (mode == MODE_F64) return ipt == 1 && hpt == 1;
    return ipt == 1 ? hpt <= 3 : (ipt == 2 && hpt == 2);
}
// Whether vanse_set_fused takes tiles of `rows` full x-rows in segments of any
// length.
bool fused_shape(int lattice, int mode, const Geometry &g, int rows);
// LDS of one 512-thread block by that rule, and of a full-row member of an
// x-split batch: the population slab and the ring of 5 perturbation planes of
// rows + 4 x-rows.
size_t fused_lds_bytes(int q, int mode, int nx, int rows);
// Tile of the marching two-step kernel (march.h): threads per block, passes
// over the interior and over the region with the two outer rows, pert values
// a thread loads per plane.
struct MarchTile {
    int nt = 0, ipt = 0, hpt = 0, ppt = 0;
};
// Whether the kernel's 32-bit offsets reach a z-plane of this size.
bool march_plane(int mode, const Geometry &g);
// The compiled tile of `rows` full x-rows in blocks of nt threads (0: the
// block size chosen for that tile); false if there is none or its LDS does
// not fit.
bool march_tile(int lattice, int mode, const Geometry &g, int rows, int nt, MarchTile *out);
// The smallest compiled tile whose passes cover those of t (a batch's members
// share one kernel); false if there is none.
bool march_cover(int lattice, int mode, MarchTile *t);
// Most x-rows of a tile in blocks of nt threads whose interior takes one pass
// (0: none), evened out over ny.
int march_rows(int lattice, int mode, const Geometry &g, int nt);
// Largest block size of the lattice's and storage's tiles.
int march_threads(int lattice, int mode);
// Raise a kernel's LDS limit when a block needs more than 64 KiB, once per
// device.
hipError_t raise_lds(const void *fn, size_t lds, std::atomic<unsigned long long> &raised);
size_t march_lds_bytes(int lattice, int mode, int nx, int rows, const MarchTile &t);
// Two-step launch of one solve: tiles of a.fty x-rows and a.fsz planes.
hipError_t launch_march(const Solver &s, const StepArgs &a);
hipError_t launch_batch_march(int lattice, int mode, const MarchTile &t, unsigned nblocks, size_t lds,
                              const BatchMember *members, const unsigned *owner, const double *mtab,
                              int j, int count, int swap, hipStream_t st);
// Several steps of D2Q9 on boxes of cells in LDS (box.hip).
constexpr int kBoxMaxSteps = 8;
struct BoxSteps {
    int k;                     // steps of this launch (even)
    unsigned nbx;              // boxes per row of boxes
    FastDiv fd_x;
    double m[kBoxMaxSteps];    // modulations m(n) .. m(n + k - 1)
};
// Most steps of a launch of box `kind` (1, 2, ..); 0: no such box.
int box_steps(int lattice, int kind);
// k steps (even, at most box_steps) from a.f at an even level into a.f2; m: the
// modulation of each.
hipError_t launch_box(const Solver &s, const StepArgs &a, int kind, const double *m, int k);
hipError_t launch_init(const Solver &s, const double *rho0, const double *u0);
// Results of a reduction that the host waits for: pinned host memory that the
// last kernel writes, and then the flag with the call's ticket.  (A copy to
// pageable memory and a stream synchronisation cost a call 20 us more.)
struct HostSlot {
    double v[8];
    unsigned long long flag;
    unsigned long long pad[7];
};
struct HostResult {
    HostSlot *slot = nullptr;      // host address
    HostSlot *dev = nullptr;       // the same on the device
    unsigned long long ticket = 0;
};
// sum over cells of rho0 phi(x, 0) (the initial M0; rho0 NULL: 1), FP64, in
// the fixed order of the reductions, into out.v[0]; uses the solver's
// reduction scratch.
hipError_t launch_init_mass(const Solver &s, const double *rho0, const HostResult &out);
// remap: each XCD takes one contiguous range of the blocks.
hipError_t launch_batch_step(int lattice, int mode, bool nt, unsigned nblocks, unsigned block,
                             const BatchMember *members, const unsigned *owner,
                             const double *mtab, const long long *t0, int j, int count, bool remap,
                             hipStream_t st);
// Rows of a solve's general tile in the batched two-step launch with blocks
// of `threads` (kFusedThreads or kGenThreads768) threads (0: none).
int batch_fused_rows(const Solver &s, int threads = kFusedThreads);
// The tile of a D3Q19 solve in a batched two-step launch with x-split
// members: full rows (*cols = nx) when nx <= split_above or nx <= 62 (false
// if they do not fit), else segments of at most 62 columns, one wave per
// row; *rows rows.
bool batch_xt_tile(const Solver &s, int split_above, int *cols, int *rows);
// LDS of one block of an x-split tile (cols < nx): slab and a ring of 5
// perturbation planes of (rows + 4) x (cols + 4) values.
size_t fused_lds_bytes_xt(int q, int mode, int cols, int rows);
// Rows of the tile that a batched two-step launch uses when every member has
// this nx and a multiple of the rows in y (0: none for this lattice, mode and
// size).
int batch_uniform_rows(int lattice, int mode, int nx, int ny);
// x-split tiles of a D3Q19 batch (batch_xt_tile).
hipError_t launch_batch_fused(int mode, unsigned nblocks, size_t lds, const BatchMember *members,
                              const unsigned *owner, const double *mtab, int j, int count,
                              int swap, hipStream_t st);
hipError_t launch_moments(const Solver &s, int parity, double m, double *rho, double *p,
                          double *u);
hipError_t launch_populations(const Solver &s, int parity, double *f);
hipError_t launch_diagnostics(const Solver &s, int parity, double m, const HostResult &out);
// Allocation-free diagnostics over caller-owned natural-order FP64 inputs
// (plane stride g.stride == g.ncells); partials in a fixed per-device array.
hipError_t launch_diagnostics_noalloc(int lattice, const Geometry &g, const double *f,
                                      const double *phi, double wq, double n2, int qmask,
                                      const double F[3], const double *force, double *out,
                                      hipStream_t st);
size_t noalloc_scratch_bytes();
// `comps` fields of n FP64 values each into the solver's R (double or float)
// fields `dst`, dst_stride elements apart.
hipError_t launch_take(int mode, const double *src, void *dst, long long n, int comps,
                       long long dst_stride, hipStream_t st);
// min, max and non-finite count of n FP64 values into out.v[0 .. 2], through
// partials[3 * kReduceBlocks]
hipError_t launch_range(const double *src, long long n, double *partials, const HostResult &out,
                        hipStream_t st);
hipError_t launch_copy_probe(void *dst, const void *src, int64_t bytes, hipStream_t st);

}  // namespace vanse
