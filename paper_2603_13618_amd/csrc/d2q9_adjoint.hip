// d2q9_adjoint.hip -- hand-written reverse mode of the D2Q9 step for the
// gradient of the summed smooth KL sensor with respect to the initial
// velocity field.
//
// Forward (per step n): g_n(x)_i = f_{n-1}(x - c_i)_i (pull streaming),
// f_n = C(g_n) = g_n - (g_n - f^eq(g_n))/tau, with f^eq_i = w_i rho P_i(u),
// P_i = 1 + 3 c_i.u + 9/2 (c_i.u)^2 - 3/2 u^2 (order-2 Grad-Hermite
// equilibrium, Sec. II.A.3).  Loss L = sum_x S_KL(g_N(x)), S_KL =
// sum_i [g_i ln(g_i/f^eq_i) - g_i + f^eq_i] (eq. HKL-sensor).
//
// Reverse, with dP_i/du_a = 3 c_ia + 9 (c_i.u) c_ia - 3 u_a:
//   seed   dL/dg_N,j = ln(g_j/f^eq_j) - sum_a B'_a (c_ja - u_a)/rho,
//          B'_a = sum_i (g_i/f^eq_i) w_i rho dP_i/du_a
//          (the derivative through rho vanishes because sum f^eq = sum g);
//   stream dL/df_n,i(x) = dL/dg_{n+1},i(x + c_i)  (a pull by +c_i);
//   collide dL/dg_n,j = (1 - 1/tau) l_j + (1/tau) [sum_i l_i w_i P_i
//          + sum_a B_a (c_ja - u_a)/rho],  B_a = sum_i l_i w_i rho dP_i/du_a,
//          with l = dL/df_n;
//   init   dL/du0_a = sum_i l_i w_i rho0 dP_i/du_a(u0), l = dL/df_0.
// Each reverse step reads the previous state (pulled by -c), the incoming
// adjoint (pulled by +c) and writes the outgoing adjoint: no atomics, every
// output written once.
#include "d2q9_band.h"
#include "lks_device.h"
#include "lks_internal.h"

namespace lks {

__device__ __forceinline__ constexpr int acx(int i) { return i / 3 - 1; }
__device__ __forceinline__ constexpr int acy(int i) { return i % 3 - 1; }
template <typename R>
__device__ __forceinline__ constexpr R aw(int i)
{
    return (i == 4) ? R(4.0 / 9.0) : ((acx(i) == 0 || acy(i) == 0) ? R(1.0 / 9.0) : R(1.0 / 36.0));
}

template <int N, typename F, int I = 0>
__device__ __forceinline__ void sfor(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        sfor<N, F, I + 1>(static_cast<F&&>(f));
    }
}

// one cell's x-shifted read: out = row[(x - CX) mod nx], scalar loads
template <int CX, typename R>
__device__ __forceinline__ R shifted(const R* __restrict__ row, int x, int nx)
{
    int xs = x - CX;
    xs = xs < 0 ? xs + nx : (xs >= nx ? xs - nx : xs);
    return row[xs];
}

template <int SIGN, typename R>
__device__ __forceinline__ void pull9(const R* __restrict__ f, const PopLayout& L, int x, int y, int nx,
                                      int ny, R (&out)[9])
{
    sfor<9>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int cx = SIGN * acx(i), cy = SIGN * acy(i);
        int ys = y - cy;
        ys = ys < 0 ? ys + ny : (ys >= ny ? ys - ny : ys);
        out[i] = shifted<cx>(f + L.at(i, ys, 0), x, nx);
    });
}

// moments of a cell from its stored deviations d_i = f_i - w_i rho0
template <typename R>
__device__ __forceinline__ Divisor<R> cell_moments(const R (&d)[9], R rho0, R& drho, R& rho, R& ux, R& uy)
{
    R jx = R(0), jy = R(0);
    drho = R(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        drho += d[i];
        jx += R(acx(i)) * d[i];
        jy += R(acy(i)) * d[i];
    }
    rho = rho0 + drho;
    const Divisor<R> by_rho(rho);
    ux = by_rho.of(jx);
    uy = by_rho.of(jy);
    return by_rho;
}

template <typename R>
__global__ __launch_bounds__(kBlock) void adj_seed_kernel(int nx, int ny, long long plane, PopLayout L, R rho0,
                                                     const R* __restrict__ fprev,
                                                     R* __restrict__ lam)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= plane) return;
    const int x = (int)(c % nx), y = (int)(c / nx);
    R d[9], drho, rho, ux, uy;
    pull9<1>(fprev, L, x, y, nx, ny, d);
    const Divisor<R> by_rho = cell_moments(d, rho0, drho, rho, ux, uy);
    const R usq15 = R(1.5) * (ux * ux + uy * uy);
    // with x_i = f^neq_i / f^eq_i: g_i / f^eq_i = 1 + x_i, and the "1" part of
    // B'_a vanishes because sum_i w_i dP_i/du_a = 0
    R bx = R(0), by = R(0), lnr[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const R cu = R(acx(i)) * ux + R(acy(i)) * uy;
        const R deq = aw<R>(i) * (drho + rho * (cu * (R(3) + R(4.5) * cu) - usq15));
        const R feq = aw<R>(i) * rho0 + deq;
        const R xi = (d[i] - deq) / feq;
        lnr[i] = kl_dphi(xi);
        const R k = R(3) + R(9) * cu;
        bx += xi * aw<R>(i) * rho * (k * R(acx(i)) - R(3) * ux);
        by += xi * aw<R>(i) * rho * (k * R(acy(i)) - R(3) * uy);
    }
#pragma unroll
    for (int j = 0; j < 9; ++j)
        lam[L.at(j, y, x)] = lnr[j] - by_rho.of(bx * (R(acx(j)) - ux) + by * (R(acy(j)) - uy));
}

// one cell of the reverse step: J_C(g)^T l from the pulled state d (g_i = w_i
// rho0 + d_i) and the pulled adjoint l
template <typename R>
__device__ __forceinline__ void collide_adjoint(const R (&d)[9], const R (&l)[9], R rho0, R tau, R (&out)[9])
{
    R drho, rho, ux, uy;
    const Divisor<R> by_rho = cell_moments(d, rho0, drho, rho, ux, uy);
    const R usq = ux * ux + uy * uy;
    R a0 = R(0), bx = R(0), by = R(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const R cu = R(acx(i)) * ux + R(acy(i)) * uy;
        const R P = R(1) + cu * (R(3) + R(4.5) * cu) - R(1.5) * usq;
        const R k = R(3) + R(9) * cu;
        a0 += l[i] * aw<R>(i) * P;
        bx += l[i] * aw<R>(i) * rho * (k * R(acx(i)) - R(3) * ux);
        by += l[i] * aw<R>(i) * rho * (k * R(acy(i)) - R(3) * uy);
    }
    const R it = R(1) / tau;
#pragma unroll
    for (int j = 0; j < 9; ++j)
        out[j] = (R(1) - it) * l[j] + it * (a0 + by_rho.of(bx * (R(acx(j)) - ux) + by * (R(acy(j)) - uy)));
}

template <typename R>
__global__ __launch_bounds__(kBlock) void adj_step_kernel(int nx, int ny, long long plane, PopLayout L, R rho0, R tau,
                                                     const R* __restrict__ fprev,
                                                     const R* __restrict__ lam_in,
                                                     R* __restrict__ lam_out)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= plane) return;
    const int x = (int)(c % nx), y = (int)(c / nx);
    R d[9], l[9], out[9];
    pull9<1>(fprev, L, x, y, nx, ny, d);
    pull9<-1>(lam_in, L, x, y, nx, ny, l);
    collide_adjoint(d, l, rho0, tau, out);
#pragma unroll
    for (int j = 0; j < 9; ++j) lam_out[L.at(j, y, x)] = out[j];
}

// K reverse steps of a band tile per launch, on the geometry of the forward
// band kernel: the incoming adjoint is read once (the tile and a ring of K
// cells), each later step takes the one before it from LDS (in place: results
// are held in registers across a barrier), and each step reads the state
// before it, pulled, from global memory.  The arithmetic is collide_adjoint's,
// so the result is that of K one-step launches.  Per cell and step K = 3 moves
// 36 + 24 B (FP32) where a step alone moves 108.
template <typename R, int K>
__global__ __launch_bounds__(kBandWaves * kWave) void adj_band_kernel(D2Q9Args a, R rho0, R tau,
                                                                     const R* __restrict__ f0,
                                                                     const R* __restrict__ f1,
                                                                     const R* __restrict__ f2,
                                                                     const R* __restrict__ lam_in,
                                                                     R* __restrict__ lam_out, int ntiles)
{
    using G = Band<K, 2>;
    constexpr int W0 = G::W0, C = G::kCells;
    __shared__ R buf[9 * C];
    const int tile = G::tile();
    if (tile >= ntiles) return;                     // whole workgroups
    const int nx = a.nx, ny = a.ny;
    const int tiles_x = (nx + G::TX - 1) / G::TX;
    const int X0 = (tile % tiles_x) * G::TX, Y0 = (tile / tiles_x) * G::TY;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    unsigned xs[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) xs[q] = (unsigned)G::wrap(X0 + lane + q - 1, nx);

    // row r of this wave: population i at (x - SIGN c_i) of f
    auto pull_row = [&](auto sc, const R* f, int r, R (&v)[9]) {
        constexpr int SIGN = decltype(sc)::value;
        sfor<9>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int ys = G::wrap(Y0 + G::NR * wave + r - SIGN * acy(i), ny);
            v[i] = (f + a.L.at(i, ys, 0))[xs[1 - SIGN * acx(i)]];
        });
    };
    auto pull_cell = [&](auto sc, const R* f, int x, int y, R (&v)[9]) {
        constexpr int SIGN = decltype(sc)::value;
        long long row[3];
        int col[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            row[q] = (long long)G::wrap(Y0 + y + q - 1, ny) * a.L.pr;
            col[q] = G::wrap(X0 + x + q - 1, nx);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) v[i] = f[i * a.L.pp + row[1 - SIGN * acy(i)] + col[1 - SIGN * acx(i)]];
    };
    auto put = [&](int cell, const R (&v)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) buf[i * C + cell] = v[i];
    };
    // the adjoint of streaming: population i at x + c_i
    auto get = [&](int cell, R (&v)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) v[i] = buf[i * C + cell + acy(i) * W0 + acx(i)];
    };
    const std::integral_constant<int, 1> fwd;
    const std::integral_constant<int, -1> bwd;

    // one step: H = cells of the ring it produces; the first reads lam_in, the
    // last writes lam_out
    auto step = [&](auto hc, const R* f) {
        constexpr int H = decltype(hc)::value;
        constexpr bool first = H == K - 1, last = H == 0;
        // the first step's ring goes to the low threads, the next one's to the high
        const int e = first ? (int)threadIdx.x : G::NW * kWave - 1 - (int)threadIdx.x;
        const bool ring = e < G::template ring<H>();
        R out[G::NR][9], og[9];
        int cell = 0;
#pragma unroll
        for (int r = 0; r < G::NR; ++r) {
            R d[9], l[9];
            pull_row(fwd, f, r, d);
            if constexpr (first) pull_row(bwd, lam_in, r, l);
            else get(G::cell(lane, G::NR * wave + r), l);
            collide_adjoint(d, l, rho0, tau, out[r]);
        }
        if constexpr (!last) {
            if (ring) {
                int x, y;
                G::template ring_cell<H>(e, x, y);
                cell = G::cell(x, y);
                R d[9], l[9];
                pull_cell(fwd, f, x, y, d);
                if constexpr (first) pull_cell(bwd, lam_in, x, y, l);
                else get(cell, l);
                collide_adjoint(d, l, rho0, tau, og);
            }
            if constexpr (!first) __syncthreads();
#pragma unroll
            for (int r = 0; r < G::NR; ++r) put(G::cell(lane, G::NR * wave + r), out[r]);
            if (ring) put(cell, og);
            __syncthreads();
        } else if (X0 + lane < nx) {
#pragma unroll
            for (int r = 0; r < G::NR; ++r) {
                const int Y = Y0 + G::NR * wave + r;
                if (Y >= ny) break;
                const long long prow = a.L.at(0, Y, 0);
#pragma unroll
                for (int i = 0; i < 9; ++i) (lam_out + (prow + i * a.L.pp))[(unsigned)(X0 + lane)] = out[r][i];
            }
        }
    };
    step(std::integral_constant<int, K - 1>{}, f0);
    if constexpr (K == 3) step(std::integral_constant<int, 1>{}, f1);
    step(std::integral_constant<int, 0>{}, K == 3 ? f2 : f1);
}

template <typename R>
__global__ __launch_bounds__(kBlock) void adj_init_kernel(int nx, int ny, long long plane, PopLayout L,
                                                     const double* __restrict__ rho0,
                                                     const double* __restrict__ ux0,
                                                     const double* __restrict__ uy0,
                                                     const R* __restrict__ lam0,
                                                     double* __restrict__ gux,
                                                     double* __restrict__ guy)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= plane) return;
    const int x = (int)(c % nx), y = (int)(c / nx);
    R l[9];
    pull9<-1>(lam0, L, x, y, nx, ny, l);
    const double r = rho0[c], u = ux0[c], v = uy0[c];
    double gx = 0.0, gy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double cu = acx(i) * u + acy(i) * v;
        const double k = 3.0 + 9.0 * cu;
        const double wl = (double)l[i] * aw<double>(i) * r;
        gx += wl * (k * acx(i) - 3.0 * u);
        gy += wl * (k * acy(i) - 3.0 * v);
    }
    gux[c] = gx;
    guy[c] = gy;
}

static dim3 cells_grid(long long n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }

hipError_t launch_adj_seed(int dtype, const D2Q9Args& a, const void* pop_prev, void* lam_out,
                           hipStream_t s)
{
    if (dtype == 0)
        adj_seed_kernel<double><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, a.rho0, (const double*)pop_prev, (double*)lam_out);
    else if (dtype == 1)
        adj_seed_kernel<float><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, (float)a.rho0, (const float*)pop_prev, (float*)lam_out);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_adj_step(int dtype, const D2Q9Args& a, const void* pop_prev, const void* lam_in,
                           void* lam_out, hipStream_t s)
{
    if (dtype == 0)
        adj_step_kernel<double><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, a.rho0, a.tau, (const double*)pop_prev, (const double*)lam_in,
            (double*)lam_out);
    else if (dtype == 1)
        adj_step_kernel<float><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, (float)a.rho0, (float)a.tau, (const float*)pop_prev,
            (const float*)lam_in, (float*)lam_out);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_adj_band(const D2Q9Args& a, int k, const void* const* f, const void* lam_in, void* lam_out,
                                  hipStream_t s)
{
    const int n = band_tiles(a.nx, a.ny, 2);
    const dim3 grid((unsigned)((n + 63) / 64 * 64)), block(kBandWaves * kWave);
    if (k == 3)
        adj_band_kernel<R, 3><<<grid, block, 0, s>>>(a, R(a.rho0), R(a.tau), (const R*)f[0], (const R*)f[1],
                                                     (const R*)f[2], (const R*)lam_in, (R*)lam_out, n);
    else
        adj_band_kernel<R, 2><<<grid, block, 0, s>>>(a, R(a.rho0), R(a.tau), (const R*)f[0], (const R*)f[1],
                                                     nullptr, (const R*)lam_in, (R*)lam_out, n);
    return hipGetLastError();
}

hipError_t launch_adj_steps(int dtype, const D2Q9Args& a, int k, const void* const* pop_prev, const void* lam_in,
                            void* lam_out, hipStream_t s)
{
    if ((k != 2 && k != 3) || !band_fits(a.nx, a.ny, 2)) return hipErrorInvalidValue;
    if (dtype == 0) return launch_adj_band<double>(a, k, pop_prev, lam_in, lam_out, s);
    if (dtype == 1) return launch_adj_band<float>(a, k, pop_prev, lam_in, lam_out, s);
    return hipErrorInvalidValue;
}

hipError_t launch_adj_init(int dtype, const D2Q9Args& a, const double* rho0, const double* ux0,
                           const double* uy0, const void* lam0, double* gux, double* guy,
                           hipStream_t s)
{
    if (dtype == 0)
        adj_init_kernel<double><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, rho0, ux0, uy0, (const double*)lam0, gux, guy);
    else if (dtype == 1)
        adj_init_kernel<float><<<cells_grid(a.plane), kBlock, 0, s>>>(
            a.nx, a.ny, a.plane, a.L, rho0, ux0, uy0, (const float*)lam0, gux, guy);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

} // namespace lks
