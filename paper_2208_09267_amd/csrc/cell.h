// cell.h -- device code shared by the kernels: population storage, the
// volume-fraction stencil and the collision of one cell.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "internal.h"
#include "lattice.h"

namespace vanse {

// ---------------------------------------------------------------------------
// Compile-time loop: f(std::integral_constant<int, I>) for I = 0 .. N-1, so
// lattice constants indexed by I stay constant expressions.
template <int I, int N, class Fn>
__device__ __forceinline__ void static_for(Fn &&fn)
{
    if constexpr (I < N) {
        fn(std::integral_constant<int, I>{});
        static_for<I + 1, N>(fn);
    }
}

// a*x + b*y + c*z for compile-time a, b, c in {-1, 0, 1}; zero terms vanish
// and the first nonzero term starts the sum (no 0 + x to evaluate).
template <int B, int C, class R>
__device__ __forceinline__ R add_terms(R s, R y, R z)
{
    if constexpr (B == 1) s = s + y;
    if constexpr (B == -1) s = s - y;
    if constexpr (C == 1) s = s + z;
    if constexpr (C == -1) s = s - z;
    return s;
}
template <int A, int B, int C, class R>
__device__ __forceinline__ R dot3(R x, R y, R z)
{
    if constexpr (A != 0) return add_terms<B, C>(A == 1 ? x : -x, y, z);
    else if constexpr (B != 0) return add_terms<0, C>(B == 1 ? y : -y, y, z);
    else if constexpr (C != 0) return C == 1 ? z : -z;
    else return R(0);
}

// Storage of one population: T is the raw element type in HBM, R the
// arithmetic type, and `shifted` / `scaled` / `unit_c` say what the stored
// value v_i is:
//   FP64        v_i = f_i                     (T = double)
//   FP32 shift  v_i = f_i - w_i               (T = float)
//   FP16 shift  v_i = f_i / (c w_i) - 1       (T = binary16 bits, decoded to float)
//   FX16 shift  v_i = f_i / (c w_i) - 1       (T = int16 bits: 2^15 v_i rounded to
//                                              nearest, saturated at +-32767)
// c is the solve's mean M0 at initialisation (StepArgs::shift): sum_i f_i is
// conserved, so v_i stays of the size of the relative deviations of M0 and u
// from their means, which the 16-bit codes resolve best near 0 (FP16: 11
// significant bits) or uniformly over 0 < f_i < 2 c w_i (FX16: rounding
// error at most 2^-16 c w_i).  The 16-bit modes step in units of c: their
// M0 is sum f / c, and the forces enter divided by c (StepArgs::Fk, fscale);
// u is the same in any unit of mass.
template <int MODE> struct Storage;
template <> struct Storage<MODE_F64> {
    using T = double;
    using R = double;
    static constexpr bool shifted = false, scaled = false, unit_c = false;
    static constexpr double unit = 1.0;   // decoded values are in units of `unit`
    static __device__ __forceinline__ R decode(T v) { return v; }
    static __device__ __forceinline__ T encode(R v) { return v; }
};
template <> struct Storage<MODE_F32S> {
    using T = float;
    using R = float;
    static constexpr bool shifted = true, scaled = false, unit_c = false;
    static constexpr double unit = 1.0;
    static __device__ __forceinline__ R decode(T v) { return v; }
    static __device__ __forceinline__ T encode(R v) { return v; }
};
template <> struct Storage<MODE_F16S> {
    using T = unsigned short;
    using R = float;
    static constexpr bool shifted = true, scaled = true, unit_c = true;
    static constexpr double unit = 1.0;
    static __device__ __forceinline__ R decode(T v) { return __half2float(__ushort_as_half(v)); }
    static __device__ __forceinline__ T encode(R v) { return __half_as_ushort(__float2half_rn(v)); }
};
template <> struct Storage<MODE_FX16S> {
    using T = unsigned short;
    using R = float;
    static constexpr bool shifted = true, scaled = true, unit_c = true;
    // the collision works on 2^15 v_i directly (the code's integer as a
    // float): a scaling by a power of two, exact, so its results are those
    // of decoding to v_i, with one multiplication per cell instead of one per
    // value and direction
    static constexpr double unit = 1.0 / 32768.0;
    static __device__ __forceinline__ R decode(T v) { return float((short)v); }
    // saturate at +-32767, then round to nearest even, so that an
    // out-of-range value reads back at the bound, which to_f64 reports as
    // not a number.  The clamp is the median of three, which takes a NaN
    // to -32767 (in IEEE mode its minimum of three drops a NaN operand).
    // Adding 1.5 * 2^23 to the clamped value leaves the nearest-even integer
    // in the low mantissa bits (the sum lies in [2^23, 2^24), where the
    // spacing is 1), so the low 16 bits of the sum's bit pattern are the
    // int16 code: the code of rounding, clamping and converting, in two
    // instructions instead of four.
    static __device__ __forceinline__ T encode(R v)
    {
        const float c = __builtin_amdgcn_fmed3f(v, -32767.0f, 32767.0f);
        return (unsigned short)__float_as_uint(c + 12582912.0f);
    }
};

// FP64 value of f_i from a stored population (off the hot path); c: the
// unit of the 16-bit modes.  An FX16 value at the bound of its range (the
// state left the range, or a NaN was stored) reads as NaN.
template <class L, int MODE, int I>
__device__ __forceinline__ double to_f64(typename Storage<MODE>::T raw, double c)
{
    using St = Storage<MODE>;
    if constexpr (MODE == MODE_FX16S) {
        if (raw == 0x7fffu || raw == 0x8000u || raw == 0x8001u) return __builtin_nan("");
    }
    const double v = double(St::decode(raw)) * St::unit;
    if constexpr (!St::shifted) return v;
    else if constexpr (!St::scaled) return L::w[I] + v;
    else if constexpr (!St::unit_c) return L::w[I] + L::w[I] * v;
    else return c * L::w[I] + c * L::w[I] * v;
}

// Unsigned division by a launch-invariant divisor d >= 1 for dividends
// n < 2^31: q = (n * m) >> s with s = 31 + ceil(log2 d), m = ceil(2^s / d)
// (the round-up multiplier of Granlund and Montgomery, 1994).
__device__ __forceinline__ unsigned fdiv(unsigned n, const FastDiv &f)
{
    return (unsigned)(((unsigned long long)n * f.m) >> f.s);
}

// The multiplier of make_fastdiv computed on the device (divisors < 2^31).
__device__ __forceinline__ FastDiv make_fastdiv_dev(unsigned d)
{
    FastDiv f;
    const unsigned l = d > 1 ? 32u - (unsigned)__clz((int)(d - 1)) : 0u;  // ceil(log2 d)
    f.s = 31 + l;
    f.m = (unsigned)(((1ull << f.s) + d - 1) / d);
    return f;
}

// Global memory access at a 32-bit byte offset from a base pointer.  With a
// wave-uniform base the compiler emits the scalar-base (saddr) form, so a
// lane carries one 32-bit offset instead of a 64-bit address.  The access
// goes through a global address-space pointer: pointers that a batched
// launch reads from its table in device memory carry no address space, and
// the compiler would otherwise use flat instructions, which also count
// against the LDS wait counter.
template <class T>
using global_t = __attribute__((address_space(1))) T;
template <class T, bool NT>
__device__ __forceinline__ T ld(const T *base, unsigned byte_off)
{
    const global_t<T> *p =
        (const global_t<T> *)(reinterpret_cast<const char *>(base) + byte_off);
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <class T, bool NT>
__device__ __forceinline__ void st(T *base, unsigned byte_off, T v)
{
    global_t<T> *p = (global_t<T> *)(reinterpret_cast<char *>(base) + byte_off);
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// ---------------------------------------------------------------------------
// Position of one cell and its periodic neighbours.
struct Cell {
    int c;
    int X[3];  // x-1, x, x+1 (wrapped)
    int Y[3];  // (y-1, y, y+1) * nx
    int Z[3];  // (z-1, z, z+1) * nx * ny
    __device__ __forceinline__ int at(int dx, int dy, int dz) const
    {
        return Z[dz + 1] + Y[dy + 1] + X[dx + 1];
    }
};

__device__ __forceinline__ Cell locate(const StepArgs &a, int c)
{
    const Geometry &g = a.geo;
    Cell k;
    k.c = c;
    const int yz = (int)fdiv((unsigned)c, a.fd_nx);
    const int x = c - yz * g.nx;
    const int z = (int)fdiv((unsigned)yz, a.fd_ny);
    const int y = yz - z * g.ny;
    k.X[0] = (x == 0 ? g.nx : x) - 1;
    k.X[1] = x;
    k.X[2] = (x + 1 == g.nx) ? 0 : x + 1;
    k.Y[0] = ((y == 0 ? g.ny : y) - 1) * g.nx;
    k.Y[1] = y * g.nx;
    k.Y[2] = ((y + 1 == g.ny) ? 0 : y + 1) * g.nx;
    k.Z[0] = ((z == 0 ? g.nz : z) - 1) * g.nxy;
    k.Z[1] = z * g.nxy;
    k.Z[2] = ((z + 1 == g.nz) ? 0 : z + 1) * g.nxy;
    return k;
}

// phi(x, t_n) = eps_mean + m(n) pert(x).  Every step kernel evaluates it
// through this one expression, so all launch forms round it alike.
template <class R>
__device__ __forceinline__ R phi_of(R eps_mean, R m, R pert)
{
    return eps_mean + m * pert;
}

// Volume-fraction operators at one cell, at the current time level:
//   I = phi + varpi (sum_{quad axes} (phi(x+e) + phi(x-e)) - 2N phi)
//       (cell integral, eqs. quad / latDiffRuleIIre, Table 3)
//   g = (phi(x+e) - phi(x-e)) / 2  (central-difference gradient of the
//       pressure-correction force)
// e[] holds phi at x, x+ex, x-ex, x+ey, x-ey, x+ez, x-ez.
template <class L, class R>
__device__ __forceinline__ void eps_combine(const R (&e)[7], R wq, R n2, int qmask, R &I,
                                            R &gx, R &gy, R &gz)
{
    R S = R(0);
    if (qmask & 1) S = e[1] + e[2];
    if (qmask & 2) {
        S = S + e[3];
        S = S + e[4];
    }
    if constexpr (L::D == 3) {
        if (qmask & 4) {
            S = S + e[5];
            S = S + e[6];
        }
    }
    I = e[0] + wq * (S - n2 * e[0]);
    gx = R(0.5) * (e[1] - e[2]);
    gy = R(0.5) * (e[3] - e[4]);
    gz = (L::D == 3) ? R(0.5) * (e[5] - e[6]) : R(0);
}

template <class L, class R>
__device__ __forceinline__ void eps_ops(const R *__restrict__ pert, R eps_mean, R m, R wq,
                                        R n2, int qmask, const Cell &k, R &I, R &gx, R &gy,
                                        R &gz)
{
    R e[7];
    e[0] = eps_mean + m * pert[k.c];
    e[1] = eps_mean + m * pert[k.at(1, 0, 0)];
    e[2] = eps_mean + m * pert[k.at(-1, 0, 0)];
    e[3] = eps_mean + m * pert[k.at(0, 1, 0)];
    e[4] = eps_mean + m * pert[k.at(0, -1, 0)];
    e[5] = e[6] = R(0);
    if constexpr (L::D == 3) {
        e[5] = eps_mean + m * pert[k.at(0, 0, 1)];
        e[6] = eps_mean + m * pert[k.at(0, 0, -1)];
    }
    eps_combine<L, R>(e, wq, n2, qmask, I, gx, gy, gz);
}

// ---------------------------------------------------------------------------
// BGK collision with Guo forcing of one cell, in place on the stored values
// v[Q] (f_i, f_i - w_i, or (f_i - w_i)/w_i by storage mode).
//
// Per cell: M0 = sum f (= 1 + sum (f - w) in the shifted modes, since
// sum w = 1 and sum w xi = 0; the 16-bit modes in units of c), rho = M0/I (eq. density), p = rho/3,
// F = p grad(phi) + F_ext (eq. pressForce), u = (j + F/2)/M0 (eq. velocity).
// The update f - (f - f^eq)/tau + Omega^F (eq. lbe with eq. feq, rho I = M0,
// and Guo's forcing term) is evaluated for each pair of opposite directions
// +-xi, whose equilibrium and forcing terms split into a part even in xi
// and a part odd in xi:
//   v'_{+-} = (1 - omega) v_{+-} + W [P0 + cu (a45 cu + b9 cF)]
//                                 +- W [c3 cu + d3 cF]
// with cu = xi.u, cF = xi.F, P0 = omega E - 3 k uF, a45 = 9/2 omega M0,
// b9 = 9 k, c3 = 3 omega M0, d3 = 3 k, k = 1 - omega/2, W = w_i (or 1 when
// the stored value is scaled by 1/w_i), and E = M0 (1 - 3/2 uu) for f, or
// dM0 - 3/2 uu M0 for the shifted values.
// First direction 1 .. H whose velocity has a nonzero component `axis`.
template <class L, int AXIS>
constexpr int first_dir()
{
    for (int i = 1; i <= L::H; ++i)
        if ((AXIS == 0 ? L::cx[i] : AXIS == 1 ? L::cy[i] : L::cz[i]) != 0) return i;
    return 0;
}

// sum_i R(w_i) - 1 for the weights as the collision rounds them (exact in
// double: the terms are at most 27 floats within 8 binades).
template <class L, class R>
constexpr double weight_excess()
{
    double s = 0.0;
    for (int i = 0; i < L::Q; ++i) s += (double)R(L::w[i]);
    return s - 1.0;
}

// F + Fc for a per-cell force value Fc stored in physical units: divided by c
// (times fscale = 1/c) in the 16-bit modes, which step in units of c.
template <class St, class R>
__device__ __forceinline__ R add_force(R F, R Fc, double fscale)
{
    if constexpr (St::unit_c) return F + R(fscale) * Fc;
    else return F + Fc;
}

// a b + c rounded once to binary16, as a float.  The compiler makes this one
// instruction of an FMA and the conversion that stores its result, but only
// where both end up in one basic block; where a kernel's control flow parts
// them the value was rounded to FP32 first, and about one in 2^13 differed
// between kernels that must agree bitwise.  The rest population is the one
// whose update ends in an FMA.
__device__ __forceinline__ float fma_to_half(float a, float b, float c)
{
    unsigned h;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3" : "=v"(h) : "v"(a), "v"(b), "v"(c));
    return __half2float(__ushort_as_half((unsigned short)h));
}

// PIN: round the rest population with fma_to_half, for kernels that keep it in
// registers across branches.  The single-step kernels store it where it is
// computed, which the compiler makes the same instruction, and need not: the
// batched one shares its collision between the two parities of a step, and
// the statement kept them apart (D3Q27 FP16: 122 -> 134 VGPRs, 7% slower).
template <class L, int MODE, class R, bool PIN = false>
__device__ __forceinline__ void collide(R (&v)[L::Q], R I, R gx, R gy, R gz, R omega,
                                        R fcoef, R Fex, R Fey, R Fez)
{
    using St = Storage<MODE>;
    constexpr int H = L::H;
    R s0, jx = R(0), jy = R(0), jz = R(0);
    if constexpr (St::scaled)
        s0 = R(L::w[0]) * v[0];
    else
        s0 = v[0];
    static_for<1, H + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int o = i + H;
        const R sp = v[i] + v[o];
        const R dm = v[i] - v[o];
        constexpr R w = St::scaled ? R(L::w[i]) : R(1);
        s0 = s0 + w * sp;
        // the first direction with a nonzero component starts each sum
        if constexpr (L::cx[i] != 0) {
            const R t = R(L::cx[i]) * w * dm;
            if constexpr (i == first_dir<L, 0>()) jx = t; else jx = jx + t;
        }
        if constexpr (L::cy[i] != 0) {
            const R t = R(L::cy[i]) * w * dm;
            if constexpr (i == first_dir<L, 1>()) jy = t; else jy = jy + t;
        }
        if constexpr (L::cz[i] != 0) {
            const R t = R(L::cz[i]) * w * dm;
            if constexpr (i == first_dir<L, 2>()) jz = t; else jz = jz + t;
        }
    });
    // sums of the stored values, in their units (FX16: 2^-15)
    if constexpr (St::unit != 1.0) {
        s0 = s0 * R(St::unit);
        jx = jx * R(St::unit);
        jy = jy * R(St::unit);
        jz = jz * R(St::unit);
    }
    const R M0 = St::shifted ? R(1) + s0 : s0;
    // eq. density and the 1/M0 of eq. velocity.  In the 16-bit modes, whose
    // rounding dominates the error, the hardware reciprocal (about 1 ulp of
    // FP32) replaces the two correctly rounded divisions: their step is bound
    // by its arithmetic, of which they are about a tenth.
    R rho, inv;
    if constexpr (St::scaled) {
        rho = M0 * __builtin_amdgcn_rcpf(I);
        inv = __builtin_amdgcn_rcpf(M0);
    } else {
        rho = M0 / I;
        inv = R(1) / M0;
    }
    const R p = rho * R(1.0 / 3.0);     // p = rho c_s^2
    const R Fx = p * gx + Fex;          // F_PC + F_ext (eq. pressForce)
    const R Fy = p * gy + Fey;
    const R Fz = (L::D == 3) ? p * gz + Fez : R(0);
    const R ux = (jx + R(0.5) * Fx) * inv;  // eq. velocity
    const R uy = (jy + R(0.5) * Fy) * inv;
    const R uz = (L::D == 3) ? (jz + R(0.5) * Fz) * inv : R(0);
    const R uu = ux * ux + uy * uy + uz * uz;
    const R uF = ux * Fx + uy * Fy + uz * Fz;

    const R om1 = R(1) - omega;
    const R E = St::shifted ? s0 - R(1.5) * uu * M0 : M0 * (R(1) - R(1.5) * uu);
    // the update's coefficients in the units of the stored values (exact:
    // 1/unit is a power of two)
    constexpr R IU = R(1.0 / St::unit);
    const R P0 = (omega * E - R(3) * fcoef * uF) * IU;
    const R a45 = R(4.5) * omega * M0 * IU;
    const R b9 = R(9) * fcoef * IU;
    const R c3 = R(3) * omega * M0 * IU;
    const R d3 = R(3) * fcoef * IU;
    {
        // The collision conserves M0: sum_i W_i (P0 + ...) = P0 in exact
        // arithmetic.  With the weights rounded to R their sum is 1 + delta
        // (FP32 D3Q19: delta = 1.49e-8), which in the shifted modes, where
        // P0 ~ omega (M0 - 1) is not small, would move the mass by delta P0
        // per cell and step, always the same way.  The rest population takes
        // back that excess (C0 P0).  FP64 stores f itself, and its weights'
        // excess (about 1e-16) is left alone.
        constexpr R W0 = St::scaled ? R(1) : R(L::w[0]);
        constexpr R C0 = St::shifted ? R(-weight_excess<L, R>() / (St::scaled ? L::w[0] : 1.0))
                                     : R(0);
        if constexpr (PIN && MODE == MODE_F16S && C0 != R(0))
            v[0] = fma_to_half(C0, P0, om1 * v[0] + W0 * P0);
        else if constexpr (C0 != R(0))
            v[0] = om1 * v[0] + W0 * P0 + C0 * P0;
        else
            v[0] = om1 * v[0] + W0 * P0;
    }
    static_for<1, H + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int o = i + H;
        constexpr R W = St::scaled ? R(1) : R(L::w[i]);
        const R cu = dot3<L::cx[i], L::cy[i], L::cz[i]>(ux, uy, uz);
        const R cF = dot3<L::cx[i], L::cy[i], L::cz[i]>(Fx, Fy, Fz);
        const R sym = W * (P0 + cu * (a45 * cu + b9 * cF));
        const R anti = W * (c3 * cu + d3 * cF);
        v[i] = om1 * v[i] + sym + anti;
        v[o] = om1 * v[o] + sym - anti;
    });
}

// ---------------------------------------------------------------------------
// Block b of a grid of n blocks -> tile number: the hardware deals blocks
// round-robin over the 8 XCDs; this gives each XCD one contiguous range of
// tiles, so y-neighbour tiles run on the same XCD at the same time and the
// rows both re-read can come from its L2.
__device__ __forceinline__ unsigned xcd_contiguous(unsigned b, unsigned n)
{
    const unsigned q = n >> 3, r = n & 7, xcd = b & 7, k = b >> 3;
    return (xcd < r) ? xcd * (q + 1) + k : r * (q + 1) + (xcd - r) * q + k;
}

}  // namespace vanse
