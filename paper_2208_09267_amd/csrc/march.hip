// march.hip -- launches of the two-step tile kernel (march.h): one solve, and
// the tiles of many solves in one grid.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "march.h"

namespace vanse {

// Two-step launch of one solve.
template <class L, int MODE, int IPT, int HPT, int PPT, int NT, int WAVES>
__global__ void __launch_bounds__(NT, WAVES) fused2_kernel(StepArgs a)
{
    march2_tile<L, MODE, IPT, HPT, PPT, NT>(a, xcd_contiguous(blockIdx.x, gridDim.x));
}

// Two-step launch of many solves: block b belongs to solve owner[b] (after the
// XCD-contiguous order), whose tiles are a contiguous range from
// members[s].block_begin.  Steps j and j + 1 of the chunk (modulations
// mtab[j][s], mtab[j + 1][s]); swap: the solve's current populations are in
// its second array (odd launch of a chunk).
template <class L, int MODE, int IPT, int HPT, int PPT, int NT, int WAVES>
__global__ void __launch_bounds__(NT, WAVES)
    batch_fused2_kernel(const BatchMember *__restrict__ members, const unsigned *__restrict__ owner,
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
    march2_tile<L, MODE, IPT, HPT, PPT, NT>(a, b - members[s].block_begin);
}

namespace {

size_t r_bytes(int mode) { return mode == MODE_F64 ? 8 : 4; }
size_t t_bytes(int mode) { return mode == MODE_F64 ? 8 : (mode == MODE_F32S ? 4 : 2); }

// The compiled tiles.  fn(lat, mode, ipt, hpt, ppt, nt, waves) as compile-time
// constants, for the first that covers t's passes.
template <class Fn>
bool march_shapes(int lattice, int mode, const MarchTile &t, Fn &&fn)
{
    bool found = false;
    auto go = [&](auto lat, auto m, auto ic, auto hc, auto pc, auto nc, auto wc) {
        if (found || t.nt != decltype(nc)::value || t.ipt > decltype(ic)::value ||
            t.hpt > decltype(hc)::value || t.ppt > decltype(pc)::value)
            return;
        found = true;
        fn(lat, m, ic, hc, pc, nc, wc);
    };
#define VANSE_MARCH(i, h, p, n, w)                                                               \
    go(lat, m, std::integral_constant<int, i>{}, std::integral_constant<int, h>{},              \
       std::integral_constant<int, p>{}, std::integral_constant<int, n>{},                      \
       std::integral_constant<int, w>{})
    auto by_mode = [&](auto lat, auto m) {
        using L = decltype(lat);
        constexpr int M = decltype(m)::value;
        if constexpr (std::is_same<L, D3Q19>::value && M != MODE_F64) {
            // 128 VGPRs: 4 waves per SIMD, so two 512-thread blocks share a CU
            VANSE_MARCH(1, 1, 2, 512, 4);
            VANSE_MARCH(1, 2, 2, 512, 4);
            VANSE_MARCH(1, 2, 4, 512, 4);
            VANSE_MARCH(1, 1, 2, 768, 3);
            VANSE_MARCH(1, 1, 2, 1024, 4);
            VANSE_MARCH(1, 2, 2, 1024, 4);
            VANSE_MARCH(1, 2, 3, 1024, 4);
            VANSE_MARCH(1, 2, 4, 1024, 4);
        } else {
            // FP64 values and D3Q27's 27 of them need up to 256 VGPRs
            VANSE_MARCH(1, 1, 2, 512, 2);
            VANSE_MARCH(1, 2, 2, 512, 2);
            VANSE_MARCH(1, 2, 4, 512, 2);
            if constexpr (std::is_same<L, D3Q27>::value && M != MODE_F64) {
                VANSE_MARCH(1, 3, 5, 512, 2);
                VANSE_MARCH(2, 2, 4, 512, 2);
                VANSE_MARCH(2, 3, 4, 512, 2);
            }
        }
    };
#undef VANSE_MARCH
    auto by_lattice = [&](auto lat) {
        if (mode == MODE_F64) by_mode(lat, std::integral_constant<int, MODE_F64>{});
        else if (mode == MODE_F32S) by_mode(lat, std::integral_constant<int, MODE_F32S>{});
        else if (mode == MODE_F16S) by_mode(lat, std::integral_constant<int, MODE_F16S>{});
        else by_mode(lat, std::integral_constant<int, MODE_FX16S>{});
    };
    if (lattice == 1) by_lattice(D3Q19{});
    else if (lattice == 2) by_lattice(D3Q27{});
    return found;
}

}  // namespace

size_t march_lds_bytes(int lattice, int mode, int nx, int rows, const MarchTile &t)
{
    const int moving = lattice == 1 ? march_moving<D3Q19>() : march_moving<D3Q27>();
    return (size_t)moving * t.ipt * t.nt * t_bytes(mode) +
           (size_t)kMarchRing * (rows + 4) * nx * r_bytes(mode);
}

bool march_cover(int lattice, int mode, MarchTile *t)
{
    return march_shapes(lattice, mode, *t, [&](auto, auto, auto i, auto h, auto p, auto, auto) {
        t->ipt = decltype(i)::value;
        t->hpt = decltype(h)::value;
        t->ppt = decltype(p)::value;
    });
}

int march_threads(int lattice, int mode) { return lattice == 1 && mode != MODE_F64 ? 1024 : 512; }

// Byte offsets in a plane of populations or perturbation values, and one row
// beyond, stay below kMarchNoStore.
bool march_plane(int mode, const Geometry &g)
{
    return ((long long)g.nxy + 2ll * g.nx) * (long long)std::max(t_bytes(mode), r_bytes(mode)) < (1ll << 31);
}

bool march_tile(int lattice, int mode, const Geometry &g, int rows, int nt, MarchTile *out)
{
    if (lattice == 0 || rows < 1 || rows > g.ny || !march_plane(mode, g)) return false;
    if (nt == 0) {
        // two 512-thread blocks per CU where the tile fits them (D3Q19 FP32
        // 128 x 4 at 128^3: 58.7 GLUPS against 50.2 with 1024 threads), else
        // the largest block
        return march_tile(lattice, mode, g, rows, 512, out) ||
               (march_threads(lattice, mode) > 512 &&
                march_tile(lattice, mode, g, rows, march_threads(lattice, mode), out));
    }
    const long long ni = (long long)g.nx * rows;
    if (ni > 2 * nt) return false;
    MarchTile t;
    t.nt = nt;
    t.ipt = (int)((ni + nt - 1) / nt);
    t.hpt = (int)((ni + 2ll * g.nx + nt - 1) / nt);
    t.ppt = (int)((ni + 4ll * g.nx + nt - 1) / nt);
    if (!march_cover(lattice, mode, &t)) return false;
    if (march_lds_bytes(lattice, mode, g.nx, rows, t) > (size_t)kFusedMaxLds) return false;
    if (out) *out = t;
    return true;
}

int march_rows(int lattice, int mode, const Geometry &g, int nt)
{
    MarchTile t;
    for (int rows = std::min(nt / g.nx, g.ny); rows >= 1; --rows)
        if (march_tile(lattice, mode, g, rows, nt, &t) && t.ipt == 1) {
            const int tiles = (g.ny + rows - 1) / rows;
            return (g.ny + tiles - 1) / tiles;
        }
    return 0;
}

hipError_t launch_march(const Solver &s, const StepArgs &a)
{
    MarchTile t;
    if (!march_tile(s.lattice, s.mode, a.geo, (int)a.fty, 0, &t)) return hipErrorInvalidValue;
    const size_t lds = march_lds_bytes(s.lattice, s.mode, a.geo.nx, (int)a.fty, t);
    const unsigned nzb = (unsigned)((a.geo.nz + (int)a.fsz - 1) / (int)a.fsz);
    hipError_t rc = hipErrorInvalidValue;
    march_shapes(s.lattice, s.mode, t, [&](auto lat, auto m, auto i, auto h, auto p, auto n, auto w) {
        // march_tile's choices (nt = 0): 768 threads are for batches
        if constexpr (decltype(n)::value != kGenThreads768) {
            auto *fn = &fused2_kernel<decltype(lat), decltype(m)::value, decltype(i)::value,
                                      decltype(h)::value, decltype(p)::value, decltype(n)::value,
                                      decltype(w)::value>;
            static std::atomic<unsigned long long> raised{0};
            if ((rc = raise_lds(reinterpret_cast<const void *>(fn), lds, raised)) != hipSuccess) return;
            fn<<<a.fnyb * nzb, decltype(n)::value, lds, s.stream>>>(a);
            rc = hipGetLastError();
        }
    });
    return rc;
}

hipError_t launch_batch_march(int lattice, int mode, const MarchTile &t, unsigned nblocks, size_t lds,
                              const BatchMember *members, const unsigned *owner, const double *mtab,
                              int j, int count, int swap, hipStream_t st)
{
    if (lds > (size_t)kFusedMaxLds) return hipErrorInvalidValue;
    hipError_t rc = hipErrorInvalidValue;
    march_shapes(lattice, mode, t, [&](auto lat, auto m, auto i, auto h, auto p, auto n, auto w) {
        auto *fn = &batch_fused2_kernel<decltype(lat), decltype(m)::value, decltype(i)::value,
                                        decltype(h)::value, decltype(p)::value, decltype(n)::value,
                                        decltype(w)::value>;
        static std::atomic<unsigned long long> raised{0};
        if ((rc = raise_lds(reinterpret_cast<const void *>(fn), lds, raised)) != hipSuccess) return;
        fn<<<nblocks, decltype(n)::value, lds, st>>>(members, owner, mtab, j, count, swap);
        rc = hipGetLastError();
    });
    return rc;
}

}  // namespace vanse
