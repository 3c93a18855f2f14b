// march.h -- two time steps in one launch (temporal blocking) on a tile of
// full x-rows that marches in z, 3-D lattices; device code.
//
// Input: f at an even time level n in natural order (a.f).  Output: f at
// n + 2 in natural order in a second array (a.f2).  A block owns the interior
// tile of TY full x-rows (y0 .. y0+TY-1) of the z-planes z0 .. z1-1 and
// marches in z over the planes p = z0-1 .. z1:
//   1. step n on the rows y0-1 .. y0+TY of plane p (the two outer rows are
//      recomputed by the neighbouring tiles too): natural loads, the phi
//      stencil at m(n), collision -- the arithmetic of the even AA step;
//   2. each post-collision value f*_i(x) whose direction leaves the (x, y)
//      column goes to an LDS slab at its destination x + xi_i (values leaving
//      the tile rows are dropped: the neighbouring tile computes them); the
//      three directions along z stay with the thread, which owns the same
//      column in both steps;
//   3. each interior cell takes the values streaming into it; those with
//      xi_z = -1 complete plane p - 1, those with xi_z = 0 and +1 wait in
//      registers for planes p and p + 1;
//   4. step n + 1 on interior plane p - 1 (phi stencil at m(n+1)), results
//      pushed to x + xi_i of a.f2.
// The cell arithmetic is that of the single-step kernel (phi_of, eps_combine,
// collide) and the intermediate values pass through the storage encoding as
// they would through HBM, so one launch is bitwise equal to two single steps.
//
// What bounds it (counters of the launches the autotuner picks, D3Q19 256^3):
// FP32, 2 rows x 128 planes, moves 2.78 GB a launch (1.06 times what it needs)
// at 5.4 TB/s, the rate of 2 Q strided streams, with its vector ALUs busy 66% of
// the time; FP64, 2 x 128, reads its outer rows twice (6.86 GB, 1.31 times) at
// 6.5 TB/s and waits for loads at 2 waves per SIMD, ALUs 36%; the 16-bit modes,
// 4 x 64, are bound by their vector instructions.  So everything that does not change from
// plane to plane is kept per lane -- a cell's byte offset in its plane, its
// place in the slab (and from it in the phi ring), its destination rows -- and a
// plane costs scalar additions per direction and a few vector ones: 277 vector
// instructions per FP32 collision, of which the collision proper is 212, where
// per-plane index arithmetic had 350 (any width) or 277 (width and rows as
// compile-time constants, which this kernel does without).  With one set of
// load registers and a ring of 4 planes FP32 fits 1024-thread blocks at any
// width, or two 512-thread ones per CU, and D3Q27 fits in FP64.  Measured in
// GLUPS, before and after: D3Q19 256^3 FP32 60.2 -> 64.0, FP64 27.5 -> 31.2,
// FX16 78.7 -> 91.2; 128^3 FP32 49.6 -> 58.7, FP64 26.8 -> 27.9; 187 x 141 x 93
// FP64 16.5 (single steps) -> 24.2; D3Q27 256^3 FP64 11.8 (single steps) -> 20.7;
// ten batched solves of edges 37-173 FP32 43.8 -> 54.4.
#pragma once

#include "cell.h"

namespace vanse {

// slots of the phi ring: planes p-1, p, p+1 and the one being filled
constexpr int kMarchRing = 4;

// directions that leave the (x, y) column, and the place of direction i among
// them in the slab
template <class L>
constexpr int march_moving()
{
    int n = 0;
    for (int i = 0; i < L::Q; ++i) n += (L::cx[i] != 0 || L::cy[i] != 0) ? 1 : 0;
    return n;
}
template <class L>
constexpr int march_slot(int i)
{
    int n = 0;
    for (int k = 0; k < i; ++k) n += (L::cx[k] != 0 || L::cy[k] != 0) ? 1 : 0;
    return n;
}
template <class L>
constexpr bool march_moves(int i)
{
    return L::cx[i] != 0 || L::cy[i] != 0;
}

// The value, hidden from the optimiser at this point: what is derived from it
// is computed again per plane (one vector instruction) rather than kept in
// registers across the march.
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Accesses through buffer descriptors: the base of a direction's plane stays
// in scalar registers and a lane carries one 32-bit byte offset (plain
// pointers were added up per lane in 64 bits).  A lane whose offset is at or
// past the buffer's size reads zero and writes nothing (the hardware's bounds
// check), so a tile's unused lanes are masked once, in their offsets, and
// every wave issues the same number of memory operations.
constexpr unsigned kMarchNoStore = 0x80000000u;

template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_buffer(const T *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), 0, (int)bytes, 0x00020000);
}

template <class T>
__device__ __forceinline__ T buffer_load(__amdgpu_buffer_rsrc_t rsrc, unsigned off)
{
    T v;
    if constexpr (sizeof(T) == 8) {
        const auto d = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0);
        __builtin_memcpy(&v, &d, 8);
    } else if constexpr (sizeof(T) == 4) {
        const unsigned d = __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0);
        __builtin_memcpy(&v, &d, 4);
    } else {
        v = __builtin_amdgcn_raw_buffer_load_b16(rsrc, off, 0, 0);
    }
    return v;
}

template <class T>
__device__ __forceinline__ void buffer_store(T v, __amdgpu_buffer_rsrc_t rsrc, unsigned off)
{
    if constexpr (sizeof(T) == 8) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        u2 d;
        __builtin_memcpy(&d, &v, 8);
        __builtin_amdgcn_raw_buffer_store_b64(d, rsrc, off, 0, 0);
    } else if constexpr (sizeof(T) == 4) {
        unsigned d;
        __builtin_memcpy(&d, &v, 4);
        __builtin_amdgcn_raw_buffer_store_b32(d, rsrc, off, 0, 0);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(v, rsrc, off, 0, 0);
    }
}

// One tile (number b, y-fastest) of a two-step launch from a.f to a.f2 at
// modulations a.m, a.m2.  The region's cells -- first the NI = nx TY interior
// ones, row by row, then the two outer rows -- are dealt to the NT threads in
// order: cell h NT + tid for pass h < HPT, so an interior cell of pass k < IPT
// is computed by the same thread in both steps.  PPT: pert values a thread
// loads per plane.
//
// TWO: two sets of registers for the populations in flight, so that no value
// changes its register: with one, the compiler moves the next loads into place
// where the passes join (19 moves a pass) and waits for them there.  Two are
// faster where the registers hold them (D3Q19 FP16 with four phi values a
// thread is 2 VGPRs short and spills 12 bytes a lane) -- FX16 256^3 94.4 -> 96.9 GLUPS, FP16
// 102.3 -> 105.7, FP64 128^3 27.6 -> 28.6, one-pass tiles (FP32 64^3, two rows
// of 8 planes) 22.7 -> 23.7 -- but FP32 with two passes in 128 VGPRs spills
// (128^3 60.3 -> 44.1, 64 batched solves 59.3 -> 55.8), and D3Q27 lost 2-3% in
// FP32 and FP64.  A set per pass, loading a whole plane ahead, spilled too, or was no
// faster (FP64 256^3 29.5 against 31.2).
template <class L, int MODE, int IPT, int HPT, int PPT, int NT>
__device__ __forceinline__ void march2_tile(const StepArgs &a, unsigned b)
{
    static_assert(L::D == 3, "two-step launch: 3-D lattices only");
    static_assert(HPT >= IPT, "the region holds the interior");
    using St = Storage<MODE>;
    using T = typename St::T;
    using R = typename St::R;
    constexpr int Q = L::Q;
    constexpr int SP = IPT * NT;            // slab cells per direction
    constexpr bool TWO = HPT == 1 || sizeof(T) == 2 || (sizeof(T) == 8 && Q == 19);
    extern __shared__ __align__(16) unsigned char march_lds[];

    const int nx = a.geo.nx, ny = a.geo.ny, nz = a.geo.nz, nxy = a.geo.nxy;
    const long long S = a.geo.stride;
    const unsigned bz = fdiv(b, a.fd_fnyb);
    const int y0 = (int)(b - bz * a.fnyb) * (int)a.fty;
    const int TY = min((int)a.fty, ny - y0);
    const int NI = nx * TY;          // interior cells of one plane of the tile
    const int RC = NI + 2 * nx;      // with the two outer rows
    const int PC = NI + 4 * nx;      // pert values per plane: rows y0-2 .. y0+TY+1
    const unsigned plane_bytes = (unsigned)nxy * (unsigned)sizeof(T);
    const unsigned PB = (unsigned)PC * (unsigned)sizeof(R);
    unsigned char *slab = march_lds;
    unsigned char *ring = march_lds + (size_t)march_moving<L>() * SP * sizeof(T);
    const int z0 = (int)bz * (int)a.fsz;
    const int z1 = min(z0 + (int)a.fsz, nz);
    const T *__restrict__ src = static_cast<const T *>(a.f);
    T *__restrict__ dst = static_cast<T *>(a.f2);
    const R *__restrict__ pert = static_cast<const R *>(a.pert);
    const R *__restrict__ fc = static_cast<const R *>(a.force);
    const R em = R(a.eps_mean);
    const int tid = threadIdx.x;
    const int wbase = __builtin_amdgcn_readfirstlane(tid & ~63);

    // periodic index for v in [-n, 2n)
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };

    // What a lane keeps of its cells.  Pass h: byte offset of the cell in its
    // population plane, its byte place in a slab plane (rows -1 and TY:
    // outside, written through the row predicates only), the distances to its
    // periodic x-neighbours x-1, x+1 (in bytes of T; PACK: in cells, 16 bits
    // each, nx < 2^15), and whether its values moving by -1, 0, +1 rows land
    // in the tile.
    unsigned off[HPT];
    constexpr bool PACK = sizeof(T) == 2;  // the 16-bit modes need the registers
    int sp[HPT], xd[HPT], xe[PACK ? 1 : HPT];
    bool dn[HPT], in[HPT], up[HPT];
    // interior pass k: place of the cell in the slab (lanes without one: 0)
    // and the byte offsets of its destination rows y-1, y, y+1
    unsigned sr[IPT], so[IPT][3];
    static_for<0, HPT>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        const int idx = min(tid + h * NT, RC - 1);
        int r, x;
        if (idx < NI) {
            r = (int)fdiv((unsigned)idx, a.fd_nx);
            x = idx - r * nx;
        } else {
            const int e = idx - NI;
            r = e < nx ? -1 : TY;
            x = e < nx ? e : e - nx;
        }
        const int y = wrap(y0 + r, ny);
        off[h] = (unsigned)(y * nx + x) * (unsigned)sizeof(T);
        sp[h] = (r * nx + x) * (int)sizeof(T);
        const int dm = x == 0 ? nx - 1 : -1, dp = x + 1 == nx ? 1 - nx : 1;
        if constexpr (PACK) {
            xd[h] = (dm & 0xffff) | (int)((unsigned)dp << 16);
        } else {
            xd[h] = dm * (int)sizeof(T);
            xe[h] = dp * (int)sizeof(T);
        }
        dn[h] = (unsigned)(r - 1) < (unsigned)TY;
        in[h] = (unsigned)r < (unsigned)TY;
        up[h] = (unsigned)(r + 1) < (unsigned)TY;
        if constexpr (h < IPT) {
            const bool own = tid + h * NT < NI;
            sr[h] = own ? (unsigned)sp[h] : 0u;
            const int ys[3] = {y == 0 ? ny - 1 : y - 1, y, y + 1 == ny ? 0 : y + 1};
            for (int d = 0; d < 3; ++d)
                so[h][d] = own ? (unsigned)(ys[d] * nx + x) * (unsigned)sizeof(T) : kMarchNoStore;
        }
    });
    // pert value j of the thread: its byte offset in a pert plane (its place
    // in a ring plane is the value's number)
    unsigned po[PPT];
    static_for<0, PPT>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int idx = min(tid + j * NT, PC - 1);
        const int r = (int)fdiv((unsigned)idx, a.fd_nx);
        const int y = ((y0 + r - 2) % ny + ny) % ny;
        po[j] = (unsigned)(y * nx + (idx - r * nx)) * (unsigned)sizeof(R);
    });

    auto load_pert = [&](R (&ph)[PPT], int qz) {
        const __amdgpu_buffer_rsrc_t plane =
            plane_buffer(pert + (long long)qz * nxy, (unsigned)nxy * (unsigned)sizeof(R));
        static_for<0, PPT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            ph[j] = buffer_load<R>(plane, po[j]);
        });
    };
    auto store_pert = [&](const R (&ph)[PPT], unsigned slot) {
        static_for<0, PPT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const unsigned idx = (unsigned)min(tid + j * NT, PC - 1);
            // repeats write the same value
            *reinterpret_cast<R *>(ring + slot + idx * (unsigned)sizeof(R)) = ph[j];
        });
    };
    auto ring_at = [&](unsigned byte) { return *reinterpret_cast<const R *>(ring + byte); };
    // natural-order populations of a cell (byte offset o) of plane pz
    auto load_cell = [&](T (&raw)[Q], int pz, unsigned o) {
        const T *plane = src + (long long)pz * nxy;
        static_for<0, Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            raw[i] = buffer_load<T>(plane_buffer(plane + i * S, plane_bytes), o);
        });
    };
    auto x_neighbours = [&](int h, int &dm, int &dp) {
        if constexpr (PACK) {
            const int v = fresh(xd[h]);
            dm = (int)(short)v * (int)sizeof(T);
            dp = (v >> 16) * (int)sizeof(T);
        } else {
            dm = xd[h];
            dp = xe[h];
        }
    };
    // bytes of T -> bytes of R
    auto rb = [](int v) { return v / (int)sizeof(T) * (int)sizeof(R); };
    // byte of a cell's centre in a ring plane (ring row 2 is tile row 0)
    const unsigned row = (unsigned)nx * (unsigned)sizeof(R);
    auto ring_of = [&](int h) { return (unsigned)rb(fresh(sp[h])) + 2u * row; };
    // phi stencil, external + per-cell force and collision of a cell of plane
    // z: centre at byte k of the ring, x-neighbours dm, dp bytes (of R) away,
    // z-neighbours e5, e6
    auto update = [&](R (&v)[Q], unsigned k, int dm, int dp, R e5, R e6, R &ctr, int z, unsigned o,
                      R mm) {
        R e[7];
        ctr = ring_at(k);
        e[0] = phi_of(em, mm, ctr);
        e[1] = phi_of(em, mm, ring_at(k + dp));
        e[2] = phi_of(em, mm, ring_at(k + dm));
        e[3] = phi_of(em, mm, ring_at(k + row));
        e[4] = phi_of(em, mm, ring_at(k - row));
        e[5] = phi_of(em, mm, e5);
        e[6] = phi_of(em, mm, e6);
        R I, gx, gy, gz;
        eps_combine<L, R>(e, R(a.wq), R(a.n2), a.qmask, I, gx, gy, gz);
        R Fex = R(a.Fk[0]), Fey = R(a.Fk[1]), Fez = R(a.Fk[2]);
        if (fc) {
            const R *plane = fc + (long long)z * nxy;
            const unsigned fo = o / (unsigned)sizeof(T) * (unsigned)sizeof(R);
            Fex = add_force<St>(Fex, ld<R, false>(plane, fo), a.fscale);
            Fey = add_force<St>(Fey, ld<R, false>(plane + S, fo), a.fscale);
            Fez = add_force<St>(Fez, ld<R, false>(plane + 2 * S, fo), a.fscale);
        }
        collide<L, MODE, R, true>(v, I, gx, gy, gz, R(a.omega), R(a.fcoef), Fex, Fey, Fez);
    };

    R up_prev[IPT][Q] = {};  // xi_z = +1 values for plane p - 1 (read at p - 2)
    R up_next[IPT][Q] = {};  // xi_z = +1 values for plane p (read at p - 1)
    R mid[IPT][Q] = {};      // xi_z = 0 values for plane p - 1 (read at p - 1)
    R zc[IPT] = {};          // pert of the cell at plane p - 2
    T col[IPT][Q] = {};      // this plane's values of the directions along z
    T raw[Q] = {};
    R ph[PPT] = {};

    // plane q lives in ring slot (q - z0 + 2) mod 4; pz: plane p, periodic
    int pz = ((z0 - 1) % nz + nz) % nz;
    auto znext = [&](int v) { return v + 1 == nz ? 0 : v + 1; };
    auto zprev = [&](int v) { return v == 0 ? nz - 1 : v - 1; };
    load_pert(ph, zprev(pz));
    store_pert(ph, 0u);
    load_pert(ph, pz);
    store_pert(ph, PB);
    load_pert(ph, znext(pz));
    store_pert(ph, 2u * PB);
    load_pert(ph, znext(znext(pz)));
    load_cell(raw, pz, off[0]);

    int slot = 1;  // ring slot of plane p
    // one plane; FULL: plane p - 1 is complete and takes step n + 1
    auto plane = [&](auto fullc) {
        constexpr bool FULL = decltype(fullc)::value;
        const unsigned s0 = (unsigned)slot * PB;
        const unsigned sp1 = (unsigned)((slot + 1) & 3) * PB;
        const unsigned sp2 = (unsigned)((slot + 2) & 3) * PB;
        const unsigned sm1 = (unsigned)((slot + 3) & 3) * PB;
        const int pz1 = znext(pz);
        __syncthreads();  // the slab and the ring slot of plane p - 2 are free
        store_pert(ph, sp2);
        // step n of pass h on the decoded values v
        auto first = [&](auto hc, R (&v)[Q]) {
            constexpr int h = decltype(hc)::value;
            R ctr;
            int dm, dp;
            x_neighbours(h, dm, dp);
            const unsigned c = ring_of(h);
            update(v, s0 + c, rb(dm), rb(dp), ring_at(sp1 + c), ring_at(sm1 + c), ctr, pz,
                   off[h], R(a.m));
            if constexpr (h < IPT)
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (!march_moves<L>(i)) col[h][i] = St::encode(v[i]);
                });
            auto push = [&](auto cyc) {
                constexpr int CY = decltype(cyc)::value;
                const int to = fresh(sp[h]) + CY * nx * (int)sizeof(T);
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (march_moves<L>(i) && L::cy[i] == CY) {
                        const int d = to + (L::cx[i] == 1 ? dp : (L::cx[i] == -1 ? dm : 0));
                        *reinterpret_cast<T *>(slab + march_slot<L>(i) * SP * sizeof(T) + d) =
                            St::encode(v[i]);
                    }
                });
            };
            if (in[h]) push(std::integral_constant<int, 0>{});
            if (up[h]) push(std::integral_constant<int, 1>{});
            if (dn[h]) push(std::integral_constant<int, -1>{});
        };
        auto decode = [&](R (&v)[Q], const T (&r)[Q]) {
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                v[i] = St::decode(r[i]);
            });
        };
        // a wave's passes form a prefix
        auto wave_on = [&](int h) { return wbase + h * NT < RC; };
        if constexpr (TWO) {
            // Pass h works in place on one of two buffers while the other one
            // loads the wave's next pass; the first then loads pass 0 of the
            // next plane as soon as no later pass needs it.
            T other[Q];
            auto pass = [&](auto hc) {
                constexpr int h = decltype(hc)::value;
                if constexpr (h + 1 < HPT)
                    if (wave_on(h + 1)) load_cell(h % 2 ? raw : other, pz, off[h + 1]);
                R v[Q];
                decode(v, h % 2 ? other : raw);
                first(hc, v);
            };
            if (wave_on(0)) pass(std::integral_constant<int, 0>{});
            if constexpr (HPT <= 2) load_cell(raw, pz1, off[0]);
            static_for<1, HPT>([&](auto hc) {
                if (wave_on(decltype(hc)::value)) pass(hc);
            });
            if constexpr (HPT > 2) load_cell(raw, pz1, off[0]);
        } else {
            // each pass loads for the wave's next one, the last for pass 0 of
            // the next plane
            auto pass = [&](auto self, auto hc) -> void {
                constexpr int h = decltype(hc)::value;
                R v[Q];
                decode(v, raw);
                if constexpr (h + 1 < HPT) {
                    const bool more = wave_on(h + 1);
                    load_cell(raw, more ? pz : pz1, more ? off[h + 1] : off[0]);
                    if (wave_on(h)) first(hc, v);
                    if (more) self(self, std::integral_constant<int, h + 1>{});
                } else {
                    load_cell(raw, pz1, off[0]);
                    if (wave_on(h)) first(hc, v);
                }
            };
            pass(pass, std::integral_constant<int, 0>{});
        }
        __syncthreads();  // slab of plane p and ring plane p + 2 complete
        load_pert(ph, znext(znext(pz1)));
        const int z = zprev(pz);  // plane p - 1
        static_for<0, IPT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            R t[Q];
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if constexpr (march_moves<L>(i))
                    t[i] = St::decode(*reinterpret_cast<const T *>(
                        slab + march_slot<L>(i) * SP * sizeof(T) + sr[k]));
                else
                    t[i] = St::decode(col[k][i]);
            });
            if constexpr (FULL) {
                R w[Q];
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if constexpr (L::cz[i] == 1) w[i] = up_prev[k][i];
                    else if constexpr (L::cz[i] == 0) w[i] = mid[k][i];
                    else w[i] = t[i];
                });
                int dm, dp;
                x_neighbours(k, dm, dp);
                if (wbase + k * NT < NI) {  // the wave has an interior cell
                    R ctr;
                    const unsigned c = ring_of(k);
                    update(w, sm1 + c, rb(dm), rb(dp), ring_at(s0 + c), zc[k], ctr, z, off[k], R(a.m2));
                    zc[k] = ctr;
                }
                const int zs[3] = {zprev(z), z, pz};
                dm = fresh(dm);
                dp = fresh(dp);
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    T *base = dst + i * S + (long long)zs[L::cz[i] + 1] * nxy;
                    unsigned o = so[k][L::cy[i] + 1];
                    if constexpr (L::cx[i] == 1) o += dp;
                    if constexpr (L::cx[i] == -1) o += dm;
                    buffer_store<T>(St::encode(w[i]), plane_buffer(base, plane_bytes), o);
                });
            } else {
                zc[k] = ring_at(sm1 + ring_of(k));
            }
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
        pz = pz1;
        slot = (slot + 1) & 3;
    };
    for (int p = z0 - 1; p <= z0; ++p) plane(std::false_type{});
    for (int p = z0 + 1; p <= z1; ++p) plane(std::true_type{});
}

}  // namespace vanse
