// kernels.hip -- gfx950 kernels of the consistent VANSE lattice Boltzmann
// step (arXiv:2208.09267, Section "Lattice Boltzmann scheme for VANSE").
//
// Data layout in HBM: one population array per solve, SoA f[i][cell] with a
// plane stride padded to 128 elements, cells x fastest.  It is updated in
// place with the AA pattern (Bailey et al., 2009):
//   even time level n: cell x reads slot i of x and writes its post-collision
//                      value for direction i into slot opp(i) of x;
//   odd time level n:  cell x reads slot opp(i) of x - xi_i and writes into
//                      slot i of x + xi_i.
// Each slot is read and written by the same thread within a step, so one
// copy of f suffices and every step moves Q loads + Q stores per cell.
// After an odd step the layout is natural again.
//
// One thread updates one cell; a wave covers 64 consecutive cells of the
// flattened index, so every direction plane is read and written with
// coalesced (at most one line misaligned) 64-wide accesses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "cell.h"

namespace vanse {

// ---------------------------------------------------------------------------
// One fused time step of one cell (the hot path): Q population loads, the
// phi stencil, the collision and Q stores.  (x, y, z) is the cell; its
// periodic neighbour rows are the element offsets Yo (y-1, y, y+1) and Zo
// (z-1, z, z+1).  Every access is a row base (wave-uniform under ROW
// tiling) plus a 32-bit lane offset of x-1, x or x+1.
// NT: 0 plain accesses, 1 nontemporal loads and stores, 2 nontemporal stores.
template <class L, int MODE, int PARITY, int NT>
__device__ __forceinline__ void cell_step(const StepArgs &a, int x, int y, int z)
{
    using St = Storage<MODE>;
    using T = typename St::T;
    using R = typename St::R;
    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz;
    const int X[3] = {(x == 0 ? nx : x) - 1, x, (x + 1 == nx) ? 0 : x + 1};
    const int Yo[3] = {((y == 0 ? ny : y) - 1) * nx, y * nx, ((y + 1 == ny) ? 0 : y + 1) * nx};
    const int Zo[3] = {((z == 0 ? nz : z) - 1) * a.geo.nxy, z * a.geo.nxy,
                       ((z + 1 == nz) ? 0 : z + 1) * a.geo.nxy};

    auto load = [&](const T *plane, int dx, int dy, int dz) -> T {
        return ld<T, NT == 1>(plane + (Zo[dz + 1] + Yo[dy + 1]),
                         (unsigned)X[dx + 1] * (unsigned)sizeof(T));
    };
    auto store = [&](T *plane, int dx, int dy, int dz, T val) {
        st<T, NT != 0>(plane + (Zo[dz + 1] + Yo[dy + 1]), (unsigned)X[dx + 1] * (unsigned)sizeof(T),
                  val);
    };

    T *__restrict__ f = static_cast<T *>(a.f);
    const long long S = a.geo.stride;
    R v[L::Q];
    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (PARITY == 0)
            v[i] = St::decode(load(f + i * S, 0, 0, 0));
        else
            v[i] = St::decode(load(f + opp<L>(i) * S, -L::cx[i], -L::cy[i], -L::cz[i]));
    });

    const R *__restrict__ pert = static_cast<const R *>(a.pert);
    const R em = R(a.eps_mean), mm = R(a.m);
    R e[7];
    e[0] = phi_of(em, mm, ld<R, false>(pert + (Zo[1] + Yo[1]), (unsigned)X[1] * sizeof(R)));
    e[1] = phi_of(em, mm, ld<R, false>(pert + (Zo[1] + Yo[1]), (unsigned)X[2] * sizeof(R)));
    e[2] = phi_of(em, mm, ld<R, false>(pert + (Zo[1] + Yo[1]), (unsigned)X[0] * sizeof(R)));
    e[3] = phi_of(em, mm, ld<R, false>(pert + (Zo[1] + Yo[2]), (unsigned)X[1] * sizeof(R)));
    e[4] = phi_of(em, mm, ld<R, false>(pert + (Zo[1] + Yo[0]), (unsigned)X[1] * sizeof(R)));
    e[5] = e[6] = R(0);
    if constexpr (L::D == 3) {
        e[5] = phi_of(em, mm, ld<R, false>(pert + (Zo[2] + Yo[1]), (unsigned)X[1] * sizeof(R)));
        e[6] = phi_of(em, mm, ld<R, false>(pert + (Zo[0] + Yo[1]), (unsigned)X[1] * sizeof(R)));
    }
    R I, gx, gy, gz;
    eps_combine<L, R>(e, R(a.wq), R(a.n2), a.qmask, I, gx, gy, gz);

    R Fex = R(a.Fk[0]), Fey = R(a.Fk[1]), Fez = R(a.Fk[2]);
    if (a.force) {  // per-cell force density, SoA [d][stride] (wave-uniform branch)
        const R *__restrict__ fc = static_cast<const R *>(a.force);
        const unsigned off = (unsigned)X[1] * (unsigned)sizeof(R);
        Fex = add_force<St>(Fex, ld<R, false>(fc + (Zo[1] + Yo[1]), off), a.fscale);
        Fey = add_force<St>(Fey, ld<R, false>(fc + a.geo.stride + (Zo[1] + Yo[1]), off), a.fscale);
        if constexpr (L::D == 3)
            Fez = add_force<St>(Fez, ld<R, false>(fc + 2 * a.geo.stride + (Zo[1] + Yo[1]), off),
                                a.fscale);
    }
    collide<L, MODE, R>(v, I, gx, gy, gz, R(a.omega), R(a.fcoef), Fex, Fey, Fez);

    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (PARITY == 0)
            store(f + opp<L>(i) * S, 0, 0, 0, St::encode(v[i]));
        else
            store(f + i * S, L::cx[i], L::cy[i], L::cz[i], St::encode(v[i]));
    });
}

// One time step of one solve.
// Tiled launch (the tile divides the lattice): a block covers tx consecutive
// cells of each of ty consecutive x-rows of one z-plane; every wave lies
// inside one row, so the y/z neighbour rows are wave-uniform (scalar
// registers), and the phi rows a block re-reads (y +- 1 inside the block)
// come from the CU's caches.  FLAT launch (any size): the lattice is flattened
// and divided with launch-invariant multipliers.
// XCD remap (flags & 2): the hardware deals blocks round-robin over the 8
// XCDs; the remap gives each XCD one contiguous range of blocks.
// Blocks of up to 1024 threads, except D3Q27 (27 populations per thread in
// registers), whose blocks are capped at 256 threads so that the compiler
// may hold them without spilling.
template <class L>
constexpr int max_block() { return L::Q > 19 ? 256 : 1024; }

template <class L, int MODE, int PARITY, bool ROW, int NT>
__global__ void __launch_bounds__(max_block<L>()) step_kernel(StepArgs a)
{
    unsigned b = blockIdx.x;
    if (a.flags & 2) {
        const unsigned q = a.nblocks >> 3, r = a.nblocks & 7, xcd = b & 7, idx = b >> 3;
        b = (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
    }
    if constexpr (ROW) {
        const unsigned rb = fdiv(b, a.fd_seg);
        const unsigned seg = b - rb * a.nseg;
        const unsigned zb = fdiv(rb, a.fd_nyb);
        const unsigned yb = rb - zb * a.nyb;
        // tx is a multiple of 64: all lanes of a wave share the row
        const unsigned ty = __builtin_amdgcn_readfirstlane(threadIdx.x >> a.txlog);
        const int x = (int)(seg * a.tx + (threadIdx.x & (a.tx - 1)));
        const int y = (int)(yb * a.ty + ty);
        cell_step<L, MODE, PARITY, NT>(a, x, y, (int)zb);
    } else {
        const unsigned c = b * a.block + threadIdx.x;
        if (c >= (unsigned)a.geo.ncells) return;
        const unsigned yz = fdiv(c, a.fd_nx);
        const int x = (int)(c - yz * a.geo.nx);
        const int z = (int)fdiv(yz, a.fd_ny);
        const int y = (int)yz - z * a.geo.ny;
        cell_step<L, MODE, PARITY, NT>(a, x, y, z);
    }
}

// One time step of many independent solves in one launch.  Block b belongs
// to solve owner[b]; that solve's blocks are a contiguous range starting at
// members[s].block_begin and tile its flattened lattice.  Each solve has its
// own time level (parity t0[s] + j) and modulation mtab[j][s].  The per-cell
// arithmetic is cell_step, so every solve evolves exactly as it would alone.
template <class L, int MODE, bool NT>
__global__ void __launch_bounds__(256) batch_step_kernel(const BatchMember *__restrict__ members,
                                                         const unsigned *__restrict__ owner,
                                                         const double *__restrict__ mtab,
                                                         const long long *__restrict__ t0,
                                                         int j, int count, bool remap)
{
    const unsigned b = remap ? xcd_contiguous(blockIdx.x, gridDim.x) : blockIdx.x;
    const unsigned s = owner[b];
    StepArgs a = members[s].a;
    a.m = mtab[(long long)j * count + s];
    const unsigned c = (b - members[s].block_begin) * a.block + threadIdx.x;
    if (c >= (unsigned)a.geo.ncells) return;
    const unsigned yz = fdiv(c, a.fd_nx);
    const int x = (int)(c - yz * a.geo.nx);
    const int z = (int)fdiv(yz, a.fd_ny);
    const int y = (int)yz - z * a.geo.ny;
    if ((t0[s] + j) & 1)
        cell_step<L, MODE, 1, NT ? 1 : 0>(a, x, y, z);
    else
        cell_step<L, MODE, 0, NT ? 1 : 0>(a, x, y, z);
}

// ---------------------------------------------------------------------------
// Two time steps in one launch (temporal blocking) with tiles that split the
// x-rows: the batched launch of D3Q19 members whose full x-rows do not fit a
// block (march.h has the tiles of full rows, and the scheme).
//
// A block owns the interior tile of fty rows of a segment of ftx columns and
// marches in z over the planes p = z0-1 .. z1:
//   1. step n on the tile's rows and columns of plane p with one halo row and
//      column on each side (recomputed by the neighbouring tiles too);
//   2. each post-collision value f*_i(x) is pushed into an LDS slab at its
//      destination x + xi_i (slab [Q][tile], values leaving the tile are
//      dropped);
//   3. each interior cell reads back the values streaming into it; those with
//      xi_z = -1 complete plane p - 1, those with xi_z = 0 and +1 wait in
//      registers for planes p and p + 1;
//   4. step n + 1 on interior plane p - 1, results pushed to x + xi_i of a.f2.
// The perturbation pert (phi = eps_mean + m pert) of the tile with two rows
// and columns on each side is staged in an LDS ring of 5 planes (p-2 .. p+2).
// Each halo cell's populations of plane p + 1 are loaded as soon as its values
// of plane p have been read, and the pert rows of plane p + 3 before step 4 of
// plane p.
// Tiles are numbered x-fastest, then y, in a z-segment (the last of each axis
// shorter).  Rows of at most 64 cells (ftx + 2 <= 64) each go to one wave,
// lane = column, so IPT and HPT count rows per wave: at most 8 IPT interior
// rows, and 8 HPT rows with the two outer ones.  A member whose ftx covers its
// whole row (ftx >= nx) has no halo columns (x wraps inside the row) and deals
// its cells to the threads in order.  Accesses use 32-bit element offsets: every
// array's byte size is below 2^32, and nx >= 8 when ftx < nx.
template <class L, int MODE, int IPT, int HPT>
__device__ __forceinline__ void split2_tile(const StepArgs &a, unsigned b)
{
    static_assert(L::D == 3, "two-step launch: 3-D lattices only");
    using St = Storage<MODE>;
    using T = typename St::T;
    using R = typename St::R;
    constexpr int Q = L::Q;
    constexpr int NT = kFusedThreads;
    constexpr int RING = 5;                 // pert planes p-2 .. p+2
    // pert values per thread and plane: (rows + 4)(cols + 4) <=
    // (HPT NT/64 + 2) 66 <= 2 HPT NT
    constexpr int PPT = 2 * HPT;
    extern __shared__ __align__(16) unsigned char fused_lds[];

    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz, nxy = a.geo.nxy;
    const long long S = a.geo.stride;
    const unsigned bz = fdiv(b, a.fd_fnyb);
    const unsigned tb = b - bz * a.fnyb;  // tile within its z-segment
    const unsigned yb = fdiv(tb, a.fd_fnxb);
    const int x0 = (int)(tb - yb * a.fnxb) * (int)a.ftx;  // first interior column
    const int y0 = (int)yb * (int)a.fty;
    const int TY = min((int)a.fty, ny - y0);
    // x-split: interior columns TX, halo row width HW = TX + 2, ring row width
    // RW = TX + 4; otherwise all three are nx (full rows, x wraps in the row)
    const bool xs = (int)a.ftx < nx;
    const int TX = xs ? min((int)a.ftx, nx - x0) : nx;
    const int HW = xs ? TX + 2 : nx;
    const int RW = xs ? TX + 4 : nx;
    const int NI = TX * TY;          // interior cells of one plane of the tile
    const int HC = HW * (TY + 2);    // cells of one plane with the two outer rows
    const int PR = TY + 4;           // pert rows per plane: y0-2 .. y0+TY+1
    const int PC = PR * RW;
    T *__restrict__ slab = reinterpret_cast<T *>(fused_lds);
    R *__restrict__ ring =
        reinterpret_cast<R *>(fused_lds + ((size_t)Q * NI * sizeof(T) + 15) / 16 * 16);
    const int z0 = (int)bz * (int)a.fsz;
    const int z1 = min(z0 + (int)a.fsz, nz);
    const T *__restrict__ src = static_cast<const T *>(a.f);
    T *__restrict__ dst = static_cast<T *>(a.f2);
    const R *__restrict__ pert = static_cast<const R *>(a.pert);
    const R *__restrict__ fc = static_cast<const R *>(a.force);
    const R em = R(a.eps_mean);
    const int tid = threadIdx.x;

    // periodic index for v in [-n, 2n): neighbours and the halo of one tile
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    // periodic plane index for any v >= -3 (the prologue and the prefetch
    // reach 2 planes below and 3 above the segment, also when nz < 3)
    auto zmod = [&](int v) { return (v + 3 * nz) % nz; };
    // rows of halo, ring and interior cell indices: row widths HW, RW, TX
    // (x-split tiles: divisors of this tile, found once; otherwise nx)
    FastDiv fd_hw = a.fd_nx, fd_rw = a.fd_nx, fd_tx = a.fd_nx;
    if (xs) {
        fd_hw = make_fastdiv_dev((unsigned)HW);
        fd_rw = make_fastdiv_dev((unsigned)RW);
        fd_tx = make_fastdiv_dev((unsigned)TX);
    }
    auto hrow = [&](int idx) { return (int)fdiv((unsigned)idx, fd_hw); };
    auto rrow = [&](int idx) { return (int)fdiv((unsigned)idx, fd_rw); };
    auto irow = [&](int idx) { return (int)fdiv((unsigned)idx, fd_tx); };
    // global column of halo column hx (x-split: x0 - 1 + hx, wrapped) and of
    // ring column c (x0 - 2 + c, wrapped); full rows: the column itself
    auto halo_x = [&](int hx) { return xs ? wrap(x0 - 1 + hx, nx) : hx; };
    auto ring_x = [&](int c) { return xs ? wrap(x0 - 2 + c, nx) : c; };
    // Cells of the tile handled by a thread.  Full rows: tile cells numbered
    // row by row, thread tid takes cell tid + pass * NT.  x-split tiles (HW <=
    // 64): one wave per row segment, lane = column, wave w takes row w + pass
    // * NW, so a wave's loads, LDS accesses and stores stay within one row
    // segment; lanes past the segment (and rows past the tile, which only
    // whole waves reach) repeat its last cell and are masked.
    constexpr int NW = NT / 64;
    const int lane = tid & 63, wv = tid >> 6;
    // halo cell of pass h: row hr (0 .. TY+1), column hx (0 .. HW-1), valid
    auto halo_cell = [&](int h, int &hr, int &hx, bool &valid) {
        if (xs) {
            const int r = wv + h * NW;
            valid = lane < HW && r < TY + 2;
            hr = min(r, TY + 1);
            hx = min(lane, HW - 1);
        } else {
            const int idx = min(tid + h * NT, HC - 1);
            valid = tid + h * NT < HC;
            hr = hrow(idx);
            hx = idx - hr * HW;
        }
    };
    // interior cell of pass k: row r (0 .. TY-1), column cx (0 .. TX-1), and
    // whether this thread owns it
    auto interior_cell = [&](int k, int &r, int &cx, bool &owned) {
        if (xs) {
            const int rr = wv + k * NW;
            owned = lane < TX && rr < TY;
            r = min(rr, TY - 1);
            cx = min(lane, TX - 1);
        } else {
            const int cell = min(tid + k * NT, NI - 1);
            owned = tid + k * NT < NI;
            r = irow(cell);
            cx = cell - r * TX;
        }
    };
    // element offset -> byte offset (32-bit, checked on the host)
    auto boff = [](int elem, unsigned size) { return (unsigned)elem * size; };
    // Ring slot s holds the pert rows of one plane at ring + s * PC; plane q
    // lives in slot (q - z0 + 2) mod 5.  The loop keeps the slots of planes
    // p-2 .. p+2 in wave-uniform registers and rotates them per plane.
    // phi stencil, external + per-cell force and collision of one cell at
    // (x, y, z) (r its ring row, c its ring
    // column: x itself for full rows, where the x-neighbours wrap in the row;
    // rm, r0, rp the ring planes of z - 1, z, z + 1) on the decoded values v,
    // at modulation mm
    auto update = [&](R (&v)[Q], int x, int y, int r, int c, const R *rm, const R *r0,
                      const R *rp, int z, R mm) {
        const int cm = xs ? c - 1 : (c == 0 ? nx : c) - 1;
        const int cp = xs ? c + 1 : ((c + 1 == nx) ? 0 : c + 1);
        const R *row = r0 + r * RW;
        R e[7];
        e[0] = phi_of(em, mm, row[c]);
        e[1] = phi_of(em, mm, row[cp]);
        e[2] = phi_of(em, mm, row[cm]);
        e[3] = phi_of(em, mm, row[RW + c]);
        e[4] = phi_of(em, mm, row[c - RW]);
        e[5] = phi_of(em, mm, rp[r * RW + c]);
        e[6] = phi_of(em, mm, rm[r * RW + c]);
        R I, gx, gy, gz;
        eps_combine<L, R>(e, R(a.wq), R(a.n2), a.qmask, I, gx, gy, gz);
        R Fex = R(a.Fk[0]), Fey = R(a.Fk[1]), Fez = R(a.Fk[2]);
        if (fc) {
            const unsigned o = boff(z * nxy + y * nx + x, sizeof(R));
            Fex = add_force<St>(Fex, ld<R, false>(fc, o), a.fscale);
            Fey = add_force<St>(Fey, ld<R, false>(fc + S, o), a.fscale);
            Fez = add_force<St>(Fez, ld<R, false>(fc + 2 * S, o), a.fscale);
        }
        collide<L, MODE, R>(v, I, gx, gy, gz, R(a.omega), R(a.fcoef), Fex, Fey, Fez);
    };
    // natural-order populations of halo cell h (of the fty + 2 rows) of plane p
    auto load_cell = [&](T (&raw_h)[Q], int h, int p) {
        const int pz = zmod(p);
        int hr, hx;
        bool valid;
        halo_cell(h, hr, hx, valid);
        const int x = halo_x(hx);
        const int y = wrap(y0 + hr - 1, ny);
        const unsigned o = boff(pz * nxy + y * nx + x, sizeof(T));
        static_for<0, Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            raw_h[i] = ld<T, false>(src + i * S, o);
        });
    };
    // pert of the PR ring rows of plane q: into registers, then into the ring
    auto load_pert = [&](R (&ph)[PPT], int q) {
        const int qz = zmod(q);
        static_for<0, PPT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int idx = min(tid + j * NT, PC - 1);
            const int r = rrow(idx);
            const int x = ring_x(idx - r * RW);
            const int y = ((y0 + r - 2) % ny + ny) % ny;
            ph[j] = ld<R, false>(pert, boff(qz * nxy + y * nx + x, sizeof(R)));
        });
    };
    auto store_pert = [&](const R (&ph)[PPT], int s) {
        static_for<0, PPT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int idx = min(tid + j * NT, PC - 1);
            ring[s * PC + idx] = ph[j];  // repeats write the same value
        });
    };

    // Every iteration issues the same memory operations in the same order
    // (pert loads, population loads, Q * IPT stores), so the hardware wait
    // counts stay exact across the loop: threads past the end of the tile
    // repeat its last cell, and stores that must not land (those repeats, and
    // the two leading iterations that complete no plane) go to a trash slot.
    R up_prev[IPT][Q] = {};  // xi_z = +1 values for plane p - 1 (read at p - 2)
    R up_next[IPT][Q] = {};  // xi_z = +1 values for plane p (read at p - 1)
    R mid[IPT][Q] = {};      // xi_z = 0 values for plane p - 1 (read at p - 1)
    T raw[HPT][Q] = {};
    R ph[PPT] = {};
    T *__restrict__ trash = static_cast<T *>(a.trash);
    for (int q = z0 - 2; q <= z0; ++q) {
        load_pert(ph, q);
        store_pert(ph, q - (z0 - 2));
    }
    load_pert(ph, z0 + 1);
    static_for<0, HPT>([&](auto hc) { load_cell(raw[decltype(hc)::value], decltype(hc)::value, z0 - 1); });
    static_for<0, IPT * Q>([&](auto) { st<T, false>(trash, 0u, T(0)); });

    int s0 = 1;  // ring slot of plane p
    for (int p = z0 - 1; p <= z1; ++p) {
        const int pz = wrap(p, nz);
        const int sp1 = s0 == RING - 1 ? 0 : s0 + 1, sp2 = sp1 == RING - 1 ? 0 : sp1 + 1;
        const int sm1 = s0 == 0 ? RING - 1 : s0 - 1, sm2 = sm1 == 0 ? RING - 1 : sm1 - 1;
        const R *ring_m2 = ring + sm2 * PC, *ring_m1 = ring + sm1 * PC;
        const R *ring_0 = ring + s0 * PC, *ring_p1 = ring + sp1 * PC;
        __syncthreads();  // the slab and the ring slot of plane p - 3 are free
        store_pert(ph, sp2);
        static_for<0, HPT>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            int hr, hx;   // halo row and column (full rows: hx = x)
            bool valid;
            halo_cell(h, hr, hx, valid);
            const int x = halo_x(hx);
            R v[Q];
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                v[i] = St::decode(raw[h][i]);
            });
            // the slot is free: its cell of plane p + 1 loads while this block
            // computes the rest of plane p
            load_cell(raw[h], h, p + 1);
            // a wave whose lanes all lie past the last halo cell only repeats
            // that cell (another wave computes it): it keeps the loads, so
            // every wave issues the same memory operations, and skips the
            // collision and the pushes
            const bool wave_on = xs ? wv + h * NW < TY + 2 : (tid & ~63) + h * NT < HC;
            if (wave_on) {
                update(v, x, wrap(y0 + hr - 1, ny), hr + 1, xs ? hx + 1 : x, ring_m1, ring_0,
                       ring_p1, pz, R(a.m));
                // destination rows hr - 1 + cy of the slab and columns x + cx
                // (full rows: wrapped in the row; x-split: hx - 1 + cx, kept
                // inside the tile)
                const int Ro[3] = {(hr - 2) * TX, (hr - 1) * TX, hr * TX};
                const int Xd[3] = {xs ? hx - 2 : (x == 0 ? nx : x) - 1, xs ? hx - 1 : x,
                                   xs ? hx : ((x + 1 == nx) ? 0 : x + 1)};
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const int r = hr - 1 + L::cy[i];
                    if ((unsigned)r < (unsigned)TY && valid && (unsigned)Xd[L::cx[i] + 1] < (unsigned)TX)
                        slab[i * NI + Ro[L::cy[i] + 1] + Xd[L::cx[i] + 1]] = St::encode(v[i]);
                });
            }
        });
        __syncthreads();  // slab of plane p and ring plane p + 2 complete
        load_pert(ph, p + 3);
        // interior plane p - 1 is completed from p = z0 + 1 on; before that the
        // work is done on plane z0 (in range) and its results are discarded
        // (the ring slots it reads may not hold data yet)
        const int z = max(p - 1, z0);
        static_for<0, IPT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            bool own;
            int r, cx;    // interior row and column (full rows: cx = x)
            interior_cell(k, r, cx, own);
            own = own && p > z0;
            const int cell = r * TX + cx;  // slab cell
            R t[Q];
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                t[i] = St::decode(slab[i * NI + cell]);
            });
            const int x = x0 + cx;
            const int y = y0 + r;
            R w[Q];
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if constexpr (L::cz[i] == 1) w[i] = up_prev[k][i];
                else if constexpr (L::cz[i] == 0) w[i] = mid[k][i];
                else w[i] = t[i];
            });
            update(w, x, y, r + 2, xs ? cx + 2 : x, ring_m2, ring_m1, ring_0, z, R(a.m2));
            // push to x + xi_i: wrapped rows and columns of a.f2
            const int Yo[3] = {((y == 0 ? ny : y) - 1) * nx, y * nx,
                               ((y + 1 == ny) ? 0 : y + 1) * nx};
            const int Zo[3] = {((z == 0 ? nz : z) - 1) * nxy, z * nxy,
                               ((z + 1 == nz) ? 0 : z + 1) * nxy};
            const unsigned Xo[3] = {(unsigned)((x == 0 ? nx : x) - 1) * (unsigned)sizeof(T),
                                    (unsigned)x * (unsigned)sizeof(T),
                                    (unsigned)((x + 1 == nx) ? 0 : x + 1) * (unsigned)sizeof(T)};
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const unsigned o =
                    boff(Zo[L::cz[i] + 1] + Yo[L::cy[i] + 1], sizeof(T)) + Xo[L::cx[i] + 1];
                st<T, false>(own ? dst + i * S : trash, own ? o : 0u, St::encode(w[i]));
            });
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if constexpr (L::cz[i] == 1) {
                    up_prev[k][i] = up_next[k][i];
                    up_next[k][i] = t[i];
                } else if constexpr (L::cz[i] == 0) {
                    mid[k][i] = t[i];
                }
            });
        });
        s0 = sp1;
    }
}


// Two-step launch of many solves with x-split tiles: block b belongs to solve
// owner[b] (after the XCD-contiguous order), whose tiles are a contiguous
// range from members[s].block_begin.  Steps j and j + 1 of the chunk
// (modulations mtab[j][s], mtab[j + 1][s]); swap: the solve's current
// populations are in its second array (odd launch of a chunk).
template <class L, int MODE, int IPT, int HPT>
__global__ void __launch_bounds__(kFusedThreads, 1)
    batch_split2_kernel(const BatchMember *__restrict__ members, const unsigned *__restrict__ owner,
                        const double *__restrict__ mtab, int j, int count, int swap)
{
    const unsigned b = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned s = owner[b];
    StepArgs a = members[s].a;
    a.m = mtab[(long long)j * count + s];
    a.m2 = mtab[(long long)(j + 1) * count + s];
    if (swap) {
        void *t = a.f;
        a.f = a.f2;
        a.f2 = t;
    }
    split2_tile<L, MODE, IPT, HPT>(a, b - members[s].block_begin);
}

// ---------------------------------------------------------------------------
// FP64 view of one cell at time level n (parity = n & 1): populations in
// natural order and the macroscopic quantities of eqs. density, velocity and
// pressForce.  Used off the hot path (moments, diagnostics, export).
template <class L, int MODE>
__device__ __forceinline__ void load_natural(const StepArgs &a, const Cell &k, int parity,
                                             double (&fo)[L::Q])
{
    using T = typename Storage<MODE>::T;
    const T *__restrict__ f = static_cast<const T *>(a.f);
    const long long S = a.geo.stride;
    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        T raw;
        if (parity == 0)
            raw = f[i * S + k.c];
        else
            raw = f[opp<L>(i) * S + k.at(-L::cx[i], -L::cy[i], -L::cz[i])];
        fo[i] = to_f64<L, MODE, i>(raw, a.shift);
    });
}

template <class L, int MODE>
__device__ __forceinline__ void macro_f64(const StepArgs &a, const Cell &k, int parity,
                                          double &M0, double (&j)[3], double &rho, double &p,
                                          double (&F)[3], double (&u)[3])
{
    using R = typename Storage<MODE>::R;
    R Ir, gxr, gyr, gzr;
    eps_ops<L, R>(static_cast<const R *>(a.pert), R(a.eps_mean), R(a.m), R(a.wq), R(a.n2),
                  a.qmask, k, Ir, gxr, gyr, gzr);
    const double I = Ir, g[3] = {double(gxr), double(gyr), double(gzr)};
    double fo[L::Q];
    load_natural<L, MODE>(a, k, parity, fo);
    M0 = 0.0;
    j[0] = j[1] = j[2] = 0.0;
    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        M0 = M0 + fo[i];
        j[0] = j[0] + double(L::cx[i]) * fo[i];
        j[1] = j[1] + double(L::cy[i]) * fo[i];
        j[2] = j[2] + double(L::cz[i]) * fo[i];
    });
    rho = M0 / I;
    p = rho / 3.0;
    double Fc[3] = {0.0, 0.0, 0.0};
    if (a.force) {
        const R *fc = static_cast<const R *>(a.force);
        for (int d = 0; d < L::D; ++d) Fc[d] = double(fc[d * a.geo.stride + k.c]);
    }
    for (int d = 0; d < 3; ++d) {
        if (d < L::D) {
            F[d] = p * g[d] + (a.F[d] + Fc[d]);
            u[d] = (j[d] + 0.5 * F[d]) / M0;
        } else {
            F[d] = 0.0;
            u[d] = 0.0;
        }
    }
}

template <class L, int MODE>
__global__ void __launch_bounds__(256) moments_kernel(StepArgs a, int parity,
                                                      double *__restrict__ rho_out,
                                                      double *__restrict__ p_out,
                                                      double *__restrict__ u_out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.geo.ncells) return;
    const Cell k = locate(a, c);
    double M0, j[3], rho, p, F[3], u[3];
    macro_f64<L, MODE>(a, k, parity, M0, j, rho, p, F, u);
    if (rho_out) rho_out[c] = rho;
    if (p_out) p_out[c] = p;
    if (u_out)
        for (int d = 0; d < L::D; ++d) u_out[(long long)d * a.geo.ncells + c] = u[d];
}

template <class L, int MODE>
__global__ void __launch_bounds__(256) populations_kernel(StepArgs a, int parity,
                                                          double *__restrict__ out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.geo.ncells) return;
    const Cell k = locate(a, c);
    double fo[L::Q];
    load_natural<L, MODE>(a, k, parity, fo);
    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        out[(long long)i * a.geo.ncells + c] = fo[i];
    });
}

// Initial state (eq. equilibrium): f_i = f_i^eq(M0 = rho0 phi(x, 0), u0),
// written in natural order (time level 0 is even).
template <class L, int MODE>
__global__ void __launch_bounds__(256) init_kernel(StepArgs a, const double *__restrict__ rho0,
                                                   const double *__restrict__ u0)
{
    using T = typename Storage<MODE>::T;
    using R = typename Storage<MODE>::R;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.geo.ncells) return;
    const R e = R(a.eps_mean) + R(a.m) * static_cast<const R *>(a.pert)[c];
    const double M0 = (rho0 ? rho0[c] : 1.0) * double(e);
    double u[3] = {0.0, 0.0, 0.0};
    if (u0)
        for (int d = 0; d < L::D; ++d) u[d] = u0[(long long)d * a.geo.ncells + c];
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    T *__restrict__ f = static_cast<T *>(a.f);
    static_for<0, L::Q>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const double cu = L::cx[i] * u[0] + L::cy[i] * u[1] + L::cz[i] * u[2];
        const double feq = L::w[i] * M0 * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
        if constexpr (!Storage<MODE>::shifted)
            f[i * a.geo.stride + c] = feq;
        else if constexpr (!Storage<MODE>::scaled)
            f[i * a.geo.stride + c] = Storage<MODE>::encode(R(feq - L::w[i]));
        else
            f[i * a.geo.stride + c] =
                Storage<MODE>::encode(R((feq / (a.shift * L::w[i]) - 1.0) / Storage<MODE>::unit));
    });
}

// ---------------------------------------------------------------------------
// Deterministic FP64 reductions: a fixed grid of kReduceBlocks blocks, each
// accumulating a fixed strided subset of cells, a wave64 shuffle tree and a
// fixed-order combination of the waves; then one block combines the block
// partials in a fixed order.
template <int NV>
__device__ __forceinline__ void block_reduce(double (&acc)[NV], double *__restrict__ out)
{
    __shared__ double lds[kReduceThreads / 64][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int v = 0; v < NV; ++v) {
        double x = acc[v];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
        if (lane == 0) lds[wave][v] = x;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double s = 0.0;
        for (int w = 0; w < kReduceThreads / 64; ++w) s += lds[w][threadIdx.x];
        out[threadIdx.x] = s;
    }
}

template <class L, int MODE>
__global__ void __launch_bounds__(kReduceThreads) diag_kernel(StepArgs a, int parity,
                                                              double *__restrict__ partials)
{
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    // two cells at a time, added in order: the second's loads are in flight
    // while the first is summed (past the end: the last cell again, not added)
    const int n = a.geo.ncells, stride = gridDim.x * kReduceThreads;
    for (int c = blockIdx.x * kReduceThreads + threadIdx.x; c < n; c += 2 * stride) {
        double M0[2], j[2][3], rho, p, F[2][3], u[3];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const Cell k = locate(a, t == 0 ? c : min(c, n - 1 - stride) + stride);
            macro_f64<L, MODE>(a, k, parity, M0[t], j[t], rho, p, F[t], u);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t == 1 && c >= n - stride) break;
            acc[0] += M0[t];
            for (int d = 0; d < 3; ++d) {
                acc[1 + d] += j[t][d];
                acc[4 + d] += F[t][d];
            }
        }
        if (c >= n - 2 * stride) break;  // c + 2 stride would pass the end (and 2^31)
    }
    block_reduce<7>(acc, partials + 7 * blockIdx.x);
}

// sum over cells of rho0 phi(x, 0), phi formed in R as init_kernel forms it
// (the mean initial M0 is the unit of the 16-bit encodings)
template <class R>
__global__ void __launch_bounds__(kReduceThreads) init_mass_kernel(StepArgs a,
                                                                   const double *__restrict__ rho0,
                                                                   double *__restrict__ partials)
{
    double acc[1] = {0.0};
    for (int c = blockIdx.x * kReduceThreads + threadIdx.x; c < a.geo.ncells;
         c += gridDim.x * kReduceThreads) {
        const R e = R(a.eps_mean) + R(a.m) * static_cast<const R *>(a.pert)[c];
        acc[0] += (rho0 ? rho0[c] : 1.0) * double(e);
    }
    block_reduce<1>(acc, partials + blockIdx.x);
}

// The results in `out` (pinned host memory) are complete: raise the flag the
// host polls.  Called by the whole block.
__device__ __forceinline__ void raise_flag(unsigned long long *flag, unsigned long long ticket)
{
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(flag, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// flag: NULL when out is device memory that nobody polls
template <int NV>
__global__ void __launch_bounds__(kReduceThreads) finalize_kernel(const double *__restrict__ partials,
                                                                  int nblocks,
                                                                  double *__restrict__ out,
                                                                  unsigned long long *flag,
                                                                  unsigned long long ticket)
{
    double acc[NV];
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kReduceThreads)
        for (int v = 0; v < NV; ++v) acc[v] += partials[NV * b + v];
    block_reduce<NV>(acc, out);
    if (flag) raise_flag(flag, ticket);
}

// min and max over a block, and the sum of bad: thread 0 has them.
__device__ __forceinline__ void block_range(double &lo, double &hi, double &bad)
{
    __shared__ double s[3][kReduceThreads / 64];
    for (int off = 32; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_down(lo, off, 64));
        hi = fmax(hi, __shfl_down(hi, off, 64));
        bad += __shfl_down(bad, off, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s[0][wave] = lo;
        s[1][wave] = hi;
        s[2][wave] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kReduceThreads / 64; ++w) {
            lo = fmin(lo, s[0][w]);
            hi = fmax(hi, s[1][w]);
            bad += s[2][w];
        }
}

// min, max and non-finite count of n FP64 values (a caller's input array,
// checked before the library takes it over).
__global__ void __launch_bounds__(kReduceThreads) range_kernel(const double *__restrict__ src,
                                                               long long n,
                                                               double *__restrict__ partials)
{
    double lo = 1e300, hi = -1e300, bad = 0.0;
    for (long long c = (long long)blockIdx.x * kReduceThreads + threadIdx.x; c < n;
         c += (long long)gridDim.x * kReduceThreads) {
        const double v = src[c];
        if (!isfinite(v)) {
            bad += 1.0;
        } else {
            lo = fmin(lo, v);
            hi = fmax(hi, v);
        }
    }
    block_range(lo, hi, bad);
    if (threadIdx.x == 0) {
        partials[3 * blockIdx.x + 0] = lo;
        partials[3 * blockIdx.x + 1] = hi;
        partials[3 * blockIdx.x + 2] = bad;
    }
}

__global__ void __launch_bounds__(kReduceThreads) range_final_kernel(const double *__restrict__ partials,
                                                                     int nblocks,
                                                                     double *__restrict__ out,
                                                                     unsigned long long *flag,
                                                                     unsigned long long ticket)
{
    double lo = 1e300, hi = -1e300, bad = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kReduceThreads) {
        lo = fmin(lo, partials[3 * b]);
        hi = fmax(hi, partials[3 * b + 1]);
        bad += partials[3 * b + 2];
    }
    block_range(lo, hi, bad);
    if (threadIdx.x == 0) {
        out[0] = lo;
        out[1] = hi;
        out[2] = bad;
    }
    raise_flag(flag, ticket);
}

// A caller's fields (blockIdx.y: the component) into the solver's own.
template <class R>
__global__ void __launch_bounds__(256) take_kernel(const double *__restrict__ src, R *__restrict__ dst,
                                                   long long n, long long dst_stride)
{
    const long long c = (long long)blockIdx.x * 256 + threadIdx.x;
    if (c < n) dst[blockIdx.y * dst_stride + c] = R(src[blockIdx.y * n + c]);
}

// Streaming copy, one 16-byte vector per thread: the best-performing plain
// copy shape on gfx950 (bandwidth calibration of the measurements).
__global__ void __launch_bounds__(256) copy_kernel(const float4 *__restrict__ src,
                                                   float4 *__restrict__ dst, long long n)
{
    const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[k] = src[k];
}

// ---------------------------------------------------------------------------
// Host-side launchers.
static inline unsigned blocks_for(long long n, int threads)
{
    return (unsigned)((n + threads - 1) / threads);
}

template <class Fn>
static hipError_t dispatch(int lattice, int mode, Fn &&fn)
{
    auto by_mode = [&](auto lat) {
        if (mode == MODE_F64) return fn(lat, std::integral_constant<int, MODE_F64>{});
        if (mode == MODE_F32S) return fn(lat, std::integral_constant<int, MODE_F32S>{});
        if (mode == MODE_F16S) return fn(lat, std::integral_constant<int, MODE_F16S>{});
        return fn(lat, std::integral_constant<int, MODE_FX16S>{});
    };
    if (lattice == 0) return by_mode(D2Q9{});
    if (lattice == 1) return by_mode(D3Q19{});
    return by_mode(D3Q27{});
}

hipError_t launch_step(const Solver &s, const StepArgs &a, int parity)
{
    const int nt = (a.flags & 1) ? 1 : ((a.flags & 8) ? 2 : 0);
    return dispatch(s.lattice, s.mode, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        auto go = [&](auto row_c, auto nt_c) {
            constexpr bool ROW = decltype(row_c)::value;
            constexpr int NT = decltype(nt_c)::value;
            if (parity == 0)
                step_kernel<L, M, 0, ROW, NT><<<a.nblocks, a.block, 0, s.stream>>>(a);
            else
                step_kernel<L, M, 1, ROW, NT><<<a.nblocks, a.block, 0, s.stream>>>(a);
        };
        auto by_nt = [&](auto row_c) {
            if (nt == 1)
                go(row_c, std::integral_constant<int, 1>{});
            else if (nt == 2)
                go(row_c, std::integral_constant<int, 2>{});
            else
                go(row_c, std::integral_constant<int, 0>{});
        };
        if (a.row)
            by_nt(std::true_type{});
        else
            by_nt(std::false_type{});
        return hipGetLastError();
    });
}

hipError_t raise_lds(const void *fn, size_t lds, std::atomic<unsigned long long> &raised)
{
    if (lds <= 65536) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (raised.load() & bit) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kFusedMaxLds);
    if (e == hipSuccess) raised.fetch_or(bit);
    return e;
}

size_t fused_lds_bytes(int q, int mode, int nx, int rows)
{
    const size_t elem = mode == MODE_F64 ? 8 : (mode == MODE_F32S ? 4 : 2);
    const size_t slab = ((size_t)q * nx * rows * elem + 15) / 16 * 16;
    const size_t ring = (size_t)5 * (rows + 4) * nx * (mode == MODE_F64 ? 8 : 4);
    return slab + ring;
}

// The general rule of vanse_set_fused (every tile it takes is one of
// march_tile's): up to two interior and four halo-plane cells per thread of a
// 512-thread block, by lattice and storage, and 160 KiB for a slab of every
// population and 5 perturbation planes.  That is the budget of x-split tiles
// (split2_tile), and more than a marching tile needs; it stays the rule, so that
// calls are accepted and refused alike, whatever kernel runs them.
bool fused_shape(int lattice, int mode, const Geometry &g, int rows)
{
    const int nx = g.nx;
    if (rows < 1 || rows > g.ny) return false;
    const long long ni = (long long)nx * rows, hc = ni + 2ll * nx;
    const long long i = (ni + kFusedThreads - 1) / kFusedThreads;
    const long long h = (hc + kFusedThreads - 1) / kFusedThreads;
    if (i > 4 || h > 8) return false;
    if (nx % 64 != 0 || g.ny % rows != 0) {
        if ((long long)g.ncells * 8 >= (1ll << 32)) return false;
        if (!fused_compiled_gen(lattice, mode, (int)i, (int)h)) return false;
    } else if (!fused_compiled(lattice, mode, (int)i, (int)h, nx == 256 && rows == 4)) {
        return false;
    }
    const int q = lattice == 0 ? 9 : (lattice == 1 ? 19 : 27);
    return fused_lds_bytes(q, mode, nx, rows) <= (size_t)kFusedMaxLds;
}

int batch_fused_rows(const Solver &s, int threads)
{
    if (s.d != 3 || (long long)s.geo.ncells * 8 >= (1ll << 32)) return 0;
    const int nx = s.geo.nx;
    int rows;
    if (threads == kGenThreads768) {
        if (s.lattice != 1 || s.mode == MODE_F64) return 0;
        rows = kGenThreads768 / nx - 2;                 // 1 interior, 1 halo cell per thread
    } else if (s.mode == MODE_F64) {
        if (s.lattice != 1) return 0;
        rows = 512 / nx - 2;                            // 1 interior, 1 halo cell per thread
    } else {
        rows = std::min(512 / nx, 1024 / nx - 2);       // 1 interior, 2 halo cells per thread
    }
    rows = std::min(rows, s.geo.ny);
    return rows >= 1 ? rows : 0;
}

int batch_uniform_rows(int lattice, int mode, int nx, int ny)
{
    int rows = 0;
    if (lattice == 1 && nx == 256) rows = mode == MODE_F64 ? 2 : 4;
    else if (lattice == 1 && nx == 128) rows = 4;
    else if (lattice == 2 && nx == 256 && mode != MODE_F64) rows = 4;
    if (rows == 4 && nx == 256 && ny % 4 != 0) rows = mode == MODE_F64 ? 0 : 2;
    return (rows > 0 && ny % rows == 0) ? rows : 0;
}

size_t fused_lds_bytes_xt(int q, int mode, int cols, int rows)
{
    const size_t elem = mode == MODE_F64 ? 8 : (mode == MODE_F32S ? 4 : 2);
    const size_t slab = ((size_t)q * cols * rows * elem + 15) / 16 * 16;
    const size_t ring = (size_t)5 * (rows + 4) * (cols + 4) * (mode == MODE_F64 ? 8 : 4);
    return slab + ring;
}

// Rows and columns of a D3Q19 solve's tile in a batched launch with x-split
// members, whose kernel has one interior and one halo cell (FP64) or two and
// two (reduced storage) per thread: full rows where they fit (*cols = nx,
// as many rows as the cells per thread allow), unless split_above < nx;
// otherwise the fewest segments of at most 62 columns (a halo column on each
// side makes a row of at most 64: one wave per row) and as many rows as
// 8 waves hold (FP64 6, reduced 14).
bool batch_xt_tile(const Solver &s, int split_above, int *cols, int *rows)
{
    if (s.lattice != 1 || s.d != 3 || (long long)s.geo.ncells * 8 >= (1ll << 32)) return false;
    const int nx = s.geo.nx, ny = s.geo.ny;
    const int per = s.mode == MODE_F64 ? 1 : 2;        // interior and halo cells per thread
    const int full = std::min(per * kFusedThreads / nx - 2, ny);
    if (nx <= split_above || nx <= 62) {
        if (full < 1) return false;
        *cols = nx;
        *rows = full;
        return true;
    }
    const int k = (nx + 61) / 62;
    const int c = (nx + k - 1) / k;
    const int nw = kFusedThreads / 64;
    const int r = std::min(per * nw - 2, ny);
    if (fused_lds_bytes_xt(s.q, s.mode, c, r) > (size_t)kFusedMaxLds) return false;
    *cols = c;
    *rows = r;
    return true;
}

hipError_t launch_batch_fused(int mode, unsigned nblocks, size_t lds, const BatchMember *members,
                              const unsigned *owner, const double *mtab, int j, int count,
                              int swap, hipStream_t st)
{
    if (lds > (size_t)kFusedMaxLds) return hipErrorInvalidValue;
    return dispatch(1, mode, [&](auto lat, auto m) -> hipError_t {
        using L = decltype(lat);
        constexpr int M = decltype(m)::value;
        if constexpr (std::is_same<L, D3Q19>::value) {
            // one interior and one halo row per wave in FP64, two and two in
            // the reduced modes
            constexpr int PER = M == MODE_F64 ? 1 : 2;
            auto *fn = &batch_split2_kernel<L, M, PER, PER>;
            static std::atomic<unsigned long long> raised{0};
            const hipError_t rc = raise_lds(reinterpret_cast<const void *>(fn), lds, raised);
            if (rc != hipSuccess) return rc;
            fn<<<nblocks, kFusedThreads, lds, st>>>(members, owner, mtab, j, count, swap);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    });
}

hipError_t launch_batch_step(int lattice, int mode, bool nt, unsigned nblocks, unsigned block,
                             const BatchMember *members, const unsigned *owner,
                             const double *mtab, const long long *t0, int j, int count, bool remap,
                             hipStream_t st)
{
    return dispatch(lattice, mode, [&](auto lat, auto m) {
        using L = decltype(lat);
        constexpr int M = decltype(m)::value;
        if (nt)
            batch_step_kernel<L, M, true><<<nblocks, block, 0, st>>>(members, owner, mtab, t0, j,
                                                                    count, remap);
        else
            batch_step_kernel<L, M, false><<<nblocks, block, 0, st>>>(members, owner, mtab, t0,
                                                                     j, count, remap);
        return hipGetLastError();
    });
}

hipError_t launch_init(const Solver &s, const double *rho0, const double *u0)
{
    StepArgs a = step_args(s, 0);
    const unsigned nb = blocks_for(a.geo.ncells, 256);
    return dispatch(s.lattice, s.mode, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        init_kernel<L, M><<<nb, 256, 0, s.stream>>>(a, rho0, u0);
        return hipGetLastError();
    });
}

hipError_t launch_init_mass(const Solver &s, const double *rho0, const HostResult &out)
{
    StepArgs a = step_args(s, 0);
    double *partials = s.scratch;
    if (s.mode == MODE_F64)
        init_mass_kernel<double><<<kReduceBlocks, kReduceThreads, 0, s.stream>>>(a, rho0, partials);
    else
        init_mass_kernel<float><<<kReduceBlocks, kReduceThreads, 0, s.stream>>>(a, rho0, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    finalize_kernel<1><<<1, kReduceThreads, 0, s.stream>>>(partials, kReduceBlocks, out.dev->v,
                                                           &out.dev->flag, out.ticket);
    return hipGetLastError();
}

hipError_t launch_moments(const Solver &s, int parity, double m, double *rho, double *p,
                          double *u)
{
    StepArgs a = step_args(s, s.t);
    a.m = m;
    const unsigned nb = blocks_for(a.geo.ncells, 256);
    return dispatch(s.lattice, s.mode, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        moments_kernel<L, M><<<nb, 256, 0, s.stream>>>(a, parity, rho, p, u);
        return hipGetLastError();
    });
}

hipError_t launch_populations(const Solver &s, int parity, double *f)
{
    StepArgs a = step_args(s, s.t);
    const unsigned nb = blocks_for(a.geo.ncells, 256);
    return dispatch(s.lattice, s.mode, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        populations_kernel<L, M><<<nb, 256, 0, s.stream>>>(a, parity, f);
        return hipGetLastError();
    });
}

hipError_t launch_diagnostics(const Solver &s, int parity, double m, const HostResult &out)
{
    StepArgs a = step_args(s, s.t);
    a.m = m;
    double *partials = s.scratch;
    hipError_t e = dispatch(s.lattice, s.mode, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        diag_kernel<L, M><<<kReduceBlocks, kReduceThreads, 0, s.stream>>>(a, parity, partials);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    finalize_kernel<7><<<1, kReduceThreads, 0, s.stream>>>(partials, kReduceBlocks, out.dev->v,
                                                           &out.dev->flag, out.ticket);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Reduction scratch of the allocation-free diagnostics: a fixed device array
// (one copy per GPU, held until the process ends) for the block partials and
// the combined sums.  Host code never passes the array's name to a kernel
// (in host code it is a stand-in, not a device address): the device address
// comes from hipGetSymbolAddress, taken once per device and kept below.
constexpr int kNoAllocScratchDoubles = 7 * kReduceBlocks + 64;
static __device__ __align__(256) double g_noalloc_scratch[kNoAllocScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
double *g_noalloc_ptr[kMaxDevices] = {};
}  // namespace

// Device address of this GPU's copy of the scratch array, looked up on the
// first call made with that device current.
static hipError_t noalloc_scratch(double **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    if (!g_noalloc_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_noalloc_scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_noalloc_ptr[dev] = static_cast<double *>(ptr);
    }
    *out = g_noalloc_ptr[dev];
    return hipSuccess;
}

size_t noalloc_scratch_bytes() { return sizeof(double) * kNoAllocScratchDoubles; }

// The sums of launch_diagnostics over caller-owned FP64 inputs in natural
// order (f [Q][ncells], phi [ncells], force [d][ncells] or null): the same
// diag_kernel and finalize_kernel, with phi = 0 + 1 * phi and plane stride
// ncells, partials in the fixed scratch array.  Nothing is allocated.
hipError_t launch_diagnostics_noalloc(int lattice, const Geometry &g, const double *f,
                                      const double *phi, double wq, double n2, int qmask,
                                      const double F[3], const double *force, double *out,
                                      hipStream_t st)
{
    double *partials = nullptr;
    hipError_t e = noalloc_scratch(&partials);
    if (e != hipSuccess) return e;
    StepArgs a{};
    a.geo = g;
    a.fd_nx = make_fastdiv((unsigned)g.nx);
    a.fd_ny = make_fastdiv((unsigned)g.ny);
    a.f = const_cast<double *>(f);
    a.pert = phi;
    a.eps_mean = 0.0;
    a.shift = 1.0;
    a.m = 1.0;
    a.omega = 1.0;
    a.fcoef = 0.5;
    for (int d = 0; d < 3; ++d) a.F[d] = a.Fk[d] = F[d];
    a.fscale = 1.0;
    a.force = force;
    a.wq = wq;
    a.n2 = n2;
    a.qmask = qmask;
    e = dispatch(lattice, MODE_F64, [&](auto lat, auto mode) {
        using L = decltype(lat);
        constexpr int M = decltype(mode)::value;
        if constexpr (M == MODE_F64)
            diag_kernel<L, M><<<kReduceBlocks, kReduceThreads, 0, st>>>(a, 0, partials);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    finalize_kernel<7><<<1, kReduceThreads, 0, st>>>(partials, kReduceBlocks, out, nullptr, 0);
    return hipGetLastError();
}

hipError_t launch_take(int mode, const double *src, void *dst, long long n, int comps,
                       long long dst_stride, hipStream_t st)
{
    const dim3 grid(blocks_for(n, 256), (unsigned)comps);
    if (mode == MODE_F64)
        take_kernel<double><<<grid, 256, 0, st>>>(src, static_cast<double *>(dst), n, dst_stride);
    else
        take_kernel<float><<<grid, 256, 0, st>>>(src, static_cast<float *>(dst), n, dst_stride);
    return hipGetLastError();
}

hipError_t launch_range(const double *src, long long n, double *partials, const HostResult &out,
                        hipStream_t st)
{
    // 8 values a thread, so that small fields leave few partials to combine
    const int nb = (int)std::min<long long>(kReduceBlocks, (n + 8 * kReduceThreads - 1) / (8 * kReduceThreads));
    range_kernel<<<nb, kReduceThreads, 0, st>>>(src, n, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    range_final_kernel<<<1, kReduceThreads, 0, st>>>(partials, nb, out.dev->v, &out.dev->flag, out.ticket);
    return hipGetLastError();
}

hipError_t launch_copy_probe(void *dst, const void *src, int64_t bytes, hipStream_t st)
{
    const long long n = bytes / 16;
    if (n == 0) return hipSuccess;
    if ((n + 255) / 256 > 0x7fffffffLL) return hipErrorInvalidValue;
    copy_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(static_cast<const float4 *>(src),
                                                             static_cast<float4 *>(dst), n);
    return hipGetLastError();
}

}  // namespace vanse
