// box.hip -- several time steps of D2Q9 in one launch, on a box of cells held
// in LDS.
//
// A step of a small lattice lasts as long as its launch (3-4 us at 64 x 64),
// and a larger one moves all its populations for one collision per cell.  Here
// a block loads a box of RX x RY cells in natural order at an even level (one
// cell per thread), steps it k times and writes the cells whose values stayed
// free of the box's edge: an interior KMAX - 1 cells in from each side, pushed
// to x + xi_i of the second array (natural order at n + k).  Step j is computed
// k - j cells beyond the interior, so neighbouring boxes repeat each other's
// rims.
//
// The levels between live in one LDS array that is updated in place by the AA
// pattern, as the populations in HBM are by single steps: an even step is local
// to its cell, an odd one gathers from and scatters to the neighbours, each
// location read and written by one thread, so one barrier per step is enough.
// phi's perturbation around a cell and the force on it do not change from step
// to step and stay in registers.  The cell arithmetic is the single-step
// kernel's (phi_of, eps_combine, collide) and every level passes through the
// storage encoding, so k steps here are bitwise equal to k single steps.
//
// Small boxes spread a small lattice over the chip (64 x 64 FP64, 256 boxes of
// 4 x 4: 3.7 -> 1.09 us a step, of which the launch is a quarter); large ones
// repeat less (1000 x 375 FP32: 9.1 -> 3.9 us, bound by vector instructions and
// the launch; 2048 x 2048 FP64: 118 -> 53 us, 4.2 TB/s of loads and stores with
// the rims).  The autotuner picks.  Boxes of two cells per thread (64 x 32)
// repeat less still and were slower everywhere (1000 x 375 FP32 5.5 us,
// 2048 x 2048 FP64 64 us: one block per CU), and boxes of D3Q19 (10 x 10 x 10,
// two steps) lost to single steps at 32^3 to 96^3 (40^3 FP32: 5.8 against 5.5 us).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cell.h"

namespace vanse {

template <int MODE, int RX, int RY, int KMAX>
__global__ void __launch_bounds__((RX * RY + 63) / 64 * 64) box_kernel(StepArgs a, BoxSteps s)
{
    using L = D2Q9;
    using St = Storage<MODE>;
    using T = typename St::T;
    using R = typename St::R;
    constexpr int Q = L::Q, N = RX * RY;
    constexpr int H = KMAX - 1;  // rim cells on each side
    constexpr int BX = RX - 2 * H, BY = RY - 2 * H;
    static_assert(KMAX % 2 == 0 && KMAX <= kBoxMaxSteps && BX > 0 && BY > 0, "a box with an interior");
    __shared__ T box[Q][N];

    const int nx = a.geo.nx, ny = a.geo.ny;
    // box of this block, x-fastest, each XCD a contiguous range: the rims that
    // neighbours share come from its L2
    const unsigned b = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned by = fdiv(b, s.fd_x), bx = b - by * s.nbx;
    const int x0 = (int)bx * BX - H, y0 = (int)by * BY - H;
    // cell of this thread (threads past the box repeat its last cell, unseen)
    const int c = min((int)threadIdx.x, N - 1);
    const int lx = c % RX, ly = c / RX;
    auto wrap = [](int v, int n) {
        const int r = v % n;
        return r < 0 ? r + n : r;
    };
    const int x = wrap(x0 + lx, nx), y = wrap(y0 + ly, ny);
    // distance from the box's edge (threads past the box: -1, they take no step)
    const int in = (int)threadIdx.x < N ? min(min(lx, RX - 1 - lx), min(ly, RY - 1 - ly)) : -1;
    // step j (1 .. k) is computed from H - (k - j) cells in
    const int first = H - s.k;

    const int X[3] = {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1};
    const int yo[3] = {(y == 0 ? ny - 1 : y - 1) * nx, y * nx, (y + 1 == ny ? 0 : y + 1) * nx};
    const int cell = yo[1] + x;
    const long long S = a.geo.stride;
    const T *__restrict__ src = static_cast<const T *>(a.f);
    T *__restrict__ dst = static_cast<T *>(a.f2);
    const R *__restrict__ pert = static_cast<const R *>(a.pert);

    R v[Q];
    if (in >= first + 1)
        static_for<0, Q>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            v[i] = St::decode(src[i * S + cell]);
        });
    const R em = R(a.eps_mean);
    const R q[5] = {pert[cell], pert[yo[1] + X[2]], pert[yo[1] + X[0]], pert[yo[2] + x], pert[yo[0] + x]};
    R Fex = R(a.Fk[0]), Fey = R(a.Fk[1]);
    if (a.force) {
        const R *__restrict__ fc = static_cast<const R *>(a.force);
        Fex = add_force<St>(Fex, fc[cell], a.fscale);
        Fey = add_force<St>(Fey, fc[S + cell], a.fscale);
    }
    auto update = [&](R m) {
        R e[7] = {};
        for (int n = 0; n < 5; ++n) e[n] = phi_of(em, m, q[n]);
        R I, gx, gy, gz;
        eps_combine<L, R>(e, R(a.wq), R(a.n2), a.qmask, I, gx, gy, gz);
        collide<L, MODE, R, true>(v, I, gx, gy, gz, R(a.omega), R(a.fcoef), Fex, Fey, R(a.Fk[2]));
    };
    // element of slot i at the cell, and sign * xi_d away
    auto at = [&](auto slotc, auto dirc, auto signc) -> T & {
        constexpr int d = decltype(dirc)::value, sign = decltype(signc)::value;
        return (&box[decltype(slotc)::value][0])[c + sign * (L::cx[d] + RX * L::cy[d])];
    };
    using Zero = std::integral_constant<int, 0>;
    using Plus = std::integral_constant<int, 1>;
    using Minus = std::integral_constant<int, -1>;
    for (int j = 1;; j += 2) {
        if (in >= first + j) {  // even step: local
            update(R(s.m[j - 1]));
            static_for<0, Q>([&](auto ic) { at(ic, ic, Zero{}) = St::encode(v[decltype(ic)::value]); });
        }
        __syncthreads();
        const bool last = j + 1 == s.k;
        if (in > first + j) {  // odd step: gather from x - xi_i
            static_for<0, Q>([&](auto ic) { v[decltype(ic)::value] = St::decode(at(ic, ic, Minus{})); });
            update(R(s.m[j]));
            if (last) {
                // interior cells of the lattice (the last boxes reach past it)
                if (lx - H < nx - (x0 + H) && ly - H < ny - (y0 + H))
                    static_for<0, Q>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        dst[i * S + yo[L::cy[i] + 1] + X[L::cx[i] + 1]] = St::encode(v[i]);
                    });
            } else {
                // the value for x + xi_i goes where opp(i) was gathered from
                static_for<0, Q>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    at(std::integral_constant<int, opp<L>(i)>{}, ic, Plus{}) = St::encode(v[i]);
                });
            }
        }
        if (last) break;
        __syncthreads();
        if (in > first + j + 1)
            static_for<0, Q>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                v[i] = St::decode(at(std::integral_constant<int, opp<L>(i)>{}, ic, Zero{}));
            });
    }
}

namespace {

// fn(mode, RX, RY, KMAX) of box `kind`.
template <class Fn>
bool box_shapes(int mode, int kind, Fn &&fn)
{
    auto shape = [&](auto rx, auto ry, auto k) {
        if (mode == MODE_F64) fn(std::integral_constant<int, MODE_F64>{}, rx, ry, k);
        else if (mode == MODE_F32S) fn(std::integral_constant<int, MODE_F32S>{}, rx, ry, k);
        else if (mode == MODE_F16S) fn(std::integral_constant<int, MODE_F16S>{}, rx, ry, k);
        else fn(std::integral_constant<int, MODE_FX16S>{}, rx, ry, k);
        return true;
    };
#define VANSE_BOX(x, y, k) \
    shape(std::integral_constant<int, x>{}, std::integral_constant<int, y>{}, std::integral_constant<int, k>{})
    if (kind == 1) return VANSE_BOX(18, 18, 8);  // interior 4 x 4
    if (kind == 2) return VANSE_BOX(22, 22, 8);  // 8 x 8
    if (kind == 3) return VANSE_BOX(32, 32, 8);  // 18 x 18
    if (kind == 4) return VANSE_BOX(32, 16, 4);  // 26 x 10
    if (kind == 5) return VANSE_BOX(64, 16, 4);  // 58 x 10
#undef VANSE_BOX
    return false;
}

}  // namespace

int box_steps(int lattice, int kind)
{
    int k = 0;
    if (lattice == 0) box_shapes(MODE_F64, kind, [&](auto, auto, auto, auto kc) { k = decltype(kc)::value; });
    return k;
}

hipError_t launch_box(const Solver &s, const StepArgs &a, int kind, const double *m, int k)
{
    hipError_t rc = hipErrorInvalidValue;
    if (s.lattice != 0) return rc;
    box_shapes(s.mode, kind, [&](auto mode, auto rx, auto ry, auto kc) {
        constexpr int K = decltype(kc)::value, RX = decltype(rx)::value, RY = decltype(ry)::value;
        constexpr int BX = RX - 2 * (K - 1), BY = RY - 2 * (K - 1);
        if (k < 2 || k > K || k % 2) return;
        BoxSteps b;
        b.k = k;
        for (int j = 0; j < k; ++j) b.m[j] = m[j];
        b.nbx = (unsigned)((a.geo.nx + BX - 1) / BX);
        b.fd_x = make_fastdiv(b.nbx);
        const unsigned nb = b.nbx * (unsigned)((a.geo.ny + BY - 1) / BY);
        box_kernel<decltype(mode)::value, RX, RY, K><<<nb, (RX * RY + 63) / 64 * 64, 0, s.stream>>>(a, b);
        rc = hipGetLastError();
    });
    return rc;
}

}  // namespace vanse
