// d2q9.hip -- D2Q9 lattice-BGK kernels for gfx950: the fused
// stream + collide + sensors + flags + FP64 sums pass, the three passes of the
// unfused baseline, the equilibrium initialiser and the moment readout.
//
// Method (arXiv 2603.13618): D2Q9 = GH3 x GH3 velocity set, order-2
// Grad-Hermite equilibrium (Sec. II.A.3), single-relaxation BGK (the QE
// collision of Sec. II.A.1 with tau1 = tau2), sensors S_KL (eq. HKL-sensor),
// S_NEQ (eq. sensor-neq-kin) and S_PI (eq. sensor-TauNS-kin) on the
// pre-collision populations, refinement flags (Sec. II.B.2, step 1).
//
// Memory layout: deviations d_i = f_i - w_i rho0, population i of cell (x, y)
// at i * pp + y * pr + x (PopLayout: plane-major [9][ny][nx] or
// row-interleaved [ny][9][nx], x fastest in both).  One thread owns VEC
// consecutive cells of a row, so every population row is read with one
// aligned VEC-wide load per thread; the x-shifted populations
// take their one missing neighbour from the adjacent lane (ds_bpermute) and
// only the wave's edge lanes touch memory for it.  Pull streaming reads each
// stored value exactly once, so HBM traffic is one read and one write per
// population plus the sensor planes and the flag byte.
#include "d2q9_band.h"
#include "lks_device.h"
#include "lks_internal.h"

namespace lks {

// velocity i = 3a + b: c = (a - 1, b - 1); weights (1/6, 2/3, 1/6)^2
__device__ __forceinline__ constexpr int cx9(int i) { return i / 3 - 1; }
__device__ __forceinline__ constexpr int cy9(int i) { return i % 3 - 1; }
template <typename R>
__device__ __forceinline__ constexpr R w9(int i)
{
    return (i == 4) ? R(4.0 / 9.0) : ((cx9(i) == 0 || cy9(i) == 0) ? R(1.0 / 9.0) : R(1.0 / 36.0));
}

template <int N, typename F, int I = 0>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F&&>(f));
    }
}

// Load VEC cells of row `row` starting at x0, shifted by cx along x
// (periodic): out[k] = row[(x0 + k - CX) mod nx].
template <int CX, typename S, int VEC>
__device__ __forceinline__ void pull_row(const typename Store<S>::raw* __restrict__ row, int x0,
                                         int nx, bool active, int lane,
                                         typename Store<S>::real (&out)[VEC])
{
    using R = typename Store<S>::real;
    R a[VEC];
    if (active) {
        load_vec<S, VEC>(row + x0, a);
    } else {
#pragma unroll
        for (int k = 0; k < VEC; ++k) a[k] = R(0);
    }
    if constexpr (CX == 0) {
#pragma unroll
        for (int k = 0; k < VEC; ++k) out[k] = a[k];
    } else if constexpr (CX == 1) {
        R prev = __shfl_up(a[VEC - 1], 1, kWave);
        if (active && (lane == 0 || x0 == 0))
            prev = Store<S>::to_real(row[x0 == 0 ? nx - 1 : x0 - 1]);
        out[0] = prev;
#pragma unroll
        for (int k = 1; k < VEC; ++k) out[k] = a[k - 1];
    } else {
        R next = __shfl_down(a[0], 1, kWave);
        if (active && (lane == kWave - 1 || x0 + VEC >= nx))
            next = Store<S>::to_real(row[x0 + VEC >= nx ? 0 : x0 + VEC]);
#pragma unroll
        for (int k = 0; k + 1 < VEC; ++k) out[k] = a[k + 1];
        out[VEC - 1] = next;
    }
}

// Per-cell result of the sensor part of the update.
template <typename R> struct CellSense {
    R kl, neq, pi;
    bool fault;
};

// One cell: moments, equilibrium, sensors and (if COLLIDE) the BGK collision
// of the pre-collision deviations d[0..8] in place.  EXT: also the extension
// sensors into ext[0..kNumExt) (mu = tau rho c_s^2, lambda = 0 on this
// isothermal lattice).
// EXACT (without SENSE): the equilibrium goes to the collision through opaque
// copies, as its other uses in the sensors would make it, so that the
// post-collision state is the same bits as with SENSE.
// read: whether anyone reads the cell's sensors.  A lane that owns no cell holds
// what the lane shifts or the staging area left there, mostly far from any
// equilibrium, and would send its wave through the far branch of S_KL row after row
// (us a step of two steps per launch with / without, 4096^2: FP32 245 / 190, BF16
// 303 / 215, FP64 767 / 408; one step on 1001 x 1503 with extension sensors 54.6 /
// 50.1).
template <typename R, bool SENSE, bool COLLIDE, bool EXT = false, bool EXACT = false,
          typename Read = std::true_type>
__device__ __forceinline__ CellSense<R> cell_update(R (&d)[9], R rho0, R inv_tau, R& drho_out,
                                                    R& jx_out, R& jy_out, Read read = {},
                                                    R* ext = nullptr, unsigned ext_mask = 0)
{
    // moments of the deviation form: rho - rho0 = sum d, j = sum c d
    const R drho = ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7])) + d[8];
    const R jx = (d[6] + d[7] + d[8]) - (d[0] + d[1] + d[2]);
    const R jy = (d[2] + d[5] + d[8]) - (d[0] + d[3] + d[6]);
    const R rho = rho0 + drho;
    const R irho = rcp(rho);
    const R ux = jx * irho, uy = jy * irho;
    // f^eq_i - w_i rho0 = w_i [(rho - rho0) + rho (3 cu + 9/2 cu^2 - 3/2 u^2)]
    const R base = drho - R(1.5) * rho * (ux * ux + uy * uy);
    R deq[9];
    // corners c = (+-1, +-1)
#pragma unroll
    for (int i = 0; i < 9; i += 2) {
        if (i == 4) continue;
        const R cu = R(cx9(i)) * ux + R(cy9(i)) * uy;
        deq[i] = R(1.0 / 36.0) * (base + rho * (cu * (R(3) + R(4.5) * cu)));
    }
    // Axis pairs from their sum (even in u) and the momentum they must carry:
    // this closes sum_i c_i f^eq_i = j exactly up to the last rounding, so no
    // bias from the rounded weights is fed back by the collision.
    {
        const R sx = R(1.0 / 9.0) * (R(2) * base + R(9) * rho * ux * ux);
        const R dx = jx - ((deq[6] + deq[8]) - (deq[0] + deq[2]));
        deq[7] = R(0.5) * (sx + dx);
        deq[1] = R(0.5) * (sx - dx);
        const R sy = R(1.0 / 9.0) * (R(2) * base + R(9) * rho * uy * uy);
        const R dy = jy - ((deq[2] + deq[8]) - (deq[0] + deq[6]));
        deq[5] = R(0.5) * (sy + dy);
        deq[3] = R(0.5) * (sy - dy);
    }
    // rest population closes the mass
    deq[4] = drho - (((deq[0] + deq[1]) + (deq[2] + deq[3])) + ((deq[5] + deq[6]) + (deq[7] + deq[8])));

    CellSense<R> out{R(0), R(0), R(0), false};
    if constexpr (SENSE) {
        R kl = R(0), neq = R(0), pxx = R(0), pxy = R(0), pyy = R(0);
        R xmax = R(0), xmin = R(0), feqmin = R(0);
        bool far;
        {   // multiply-adds fuse within one expression only: the same bits in every kernel
#pragma clang fp contract(on)
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const R fneq = d[i] - deq[i];
                const R feq = w9<R>(i) * rho0 + deq[i];
                const R x = fneq * rcp(feq);
                // S_KL term feq phi(x) = fneq x p(x) on the series branch
                kl += (fneq * x) * kl_series_short(x);
                xmax = i == 0 ? fabs(x) : fmax(xmax, fabs(x));
                feqmin = i == 0 ? feq : fmin(feqmin, feq);
                neq += fabs(fneq);
                if (cx9(i) != 0) pxx += fneq;
                if (cy9(i) != 0) pyy += fneq;
                if (cx9(i) * cy9(i) != 0) pxy += R(cx9(i) * cy9(i)) * fneq;
            }
            // Rare: some population far from equilibrium (or NaN).  Beyond the
            // longer series the smallest x is needed too (x > -1 is f > 0);
            // |x| <= 0.1 already implies it.
            // Cells within the longer series (most of them) take that alone.
            far = !(xmax <= KlShortCut<R>::v);
            if constexpr (!std::is_same<Read, std::true_type>::value) far = far && read;
            if (far) {
                kl = R(0);
                const bool series = xmax <= KlCut<R>::v;
                if (series) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const R feq = w9<R>(i) * rho0 + deq[i];
                        const R x = (d[i] - deq[i]) * rcp(feq);
                        kl += feq * (x * x * kl_series(x));
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const R feq = w9<R>(i) * rho0 + deq[i];
                        const R x = (d[i] - deq[i]) * rcp(feq);
                        xmin = i == 0 ? x : fmin(xmin, x);
                        kl += feq * kl_phi(x);
                    }
                }
            }
        }
        out.fault = !(feqmin > R(0)) || (far && !(xmin > R(-1))) || !(kl == kl);
        out.kl = out.fault ? R(INFINITY) : kl;
        out.neq = neq;
        out.pi = sqrt_r(fma(pxx, pxx, fma(R(2) * pxy, pxy, pyy * pyy)));
        if constexpr (EXT) {
            // The extension sensors work on opaque copies (pin) of the
            // pre-collision deviations, their equilibrium parts and the
            // base quantities they need, and run after the collision: no
            // base expression gains a use and the base arithmetic stays in
            // one block, so its results do not depend on the extension.
            R dp[9], qp[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                dp[i] = pin(d[i]);
                qp[i] = pin(deq[i]);
            }
            const R kl_p = pin(kl), rho0_p = pin(rho0), tau_p = pin(inv_tau), irho_p = pin(irho);
            const R ux_p = pin(ux), uy_p = pin(uy);
            const R pxx_p = pin(pxx), pxy_p = pin(pxy), pyy_p = pin(pyy);
            const bool fault = out.fault;
            if constexpr (COLLIDE) {
#pragma unroll
                for (int i = 0; i < 9; ++i) d[i] -= inv_tau * (d[i] - deq[i]);
            }
            ExtAcc<R> xa;
            const ExtNeed need(ext_mask);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const R fneq = dp[i] - qp[i];
                const R x = fneq * rcp(w9<R>(i) * rho0_p + qp[i]);
                // f = w rho0 + d; f^eq/w - 1 = (rho0 - 1) + deq/w
                xa.add(need, fneq, x, w9<R>(i) * rho0_p + dp[i],
                       (rho0_p - R(1)) + qp[i] * R(1.0 / w9<double>(i)));
            }
            R xv[kNumExt];
            const R inv_mu = R(3) * tau_p * irho_p;          // mu = tau rho / 3
            ext_finish<R>(xa, kl_p, fault, tau_p, inv_mu, pxx_p, pxy_p, pyy_p, ux_p, uy_p, R(0), R(0),
                          false, xv);
#pragma unroll
            for (int k = 0; k < kNumExt; ++k) ext[k] = xv[k];
            drho_out = drho;
            jx_out = jx;
            jy_out = jy;
            return out;
        }
    }
    if constexpr (COLLIDE) {
        if constexpr (EXACT) {
#pragma unroll
            for (int i = 0; i < 9; ++i) deq[i] = pin(deq[i]);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] -= inv_tau * (d[i] - deq[i]);
    }
    drho_out = drho;
    jx_out = jx;
    jy_out = jy;
    return out;
}

// flag levels of the extension sensors
template <typename R>
__device__ __forceinline__ void ext_levels(const D2Q9Args& a, const R (&xv)[kNumExt], LevelAcc& lv)
{
    constexpr bool F32 = sizeof(R) == 4;
#pragma unroll
    for (int q = 0; q < kNumExt; ++q) {
        if (!(a.mask & (1u << (kExtFlagShift + q)))) continue;
        lv.add(xv[q], F32 ? R(a.x.thr_f[q][0]) : R(a.x.thr[q][0]), F32 ? R(a.x.thr_f[q][1]) : R(a.x.thr[q][1]));
    }
}

template <typename S, int VEC, bool PULL>
__device__ __forceinline__ void load_row(const typename Store<S>::raw* __restrict__ fin, const PopLayout& L,
                                         int y, int nx, int ny, int x0, bool active, int lane,
                                         typename Store<S>::real (&d)[9][VEC])
{
    using R = typename Store<S>::real;
    static_for<9>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int cx = PULL ? cx9(i) : 0;
        constexpr int cy = PULL ? cy9(i) : 0;
        int ys = y - cy;
        ys = ys < 0 ? ys + ny : (ys >= ny ? ys - ny : ys);
        R v[VEC];
        pull_row<cx, S, VEC>(fin + L.at(i, ys, 0), x0, nx, active, lane, v);
#pragma unroll
        for (int k = 0; k < VEC; ++k) d[i][k] = v[k];
    });
}

// One workgroup: `rows` consecutive rows of one x-tile.  The next row's
// populations are loaded before the current row is computed, so each wave
// keeps a row of loads in flight behind its arithmetic.
template <typename S, int VEC, int PASS>
__global__ __launch_bounds__(kBlock) LKS_CELL_KERNEL_ATTR void d2q9_kernel(
    D2Q9Args a, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ fout,
    typename Store<S>::real* __restrict__ sens, uint8_t* __restrict__ flags,
    double* __restrict__ partials, unsigned long long* __restrict__ faults)
{
    using R = typename Store<S>::real;
    constexpr bool PULL = (PASS == kFused || PASS == kStream);
    constexpr bool SENSE = (PASS == kFused || PASS == kSense);
    constexpr bool COLLIDE = (PASS == kFused || PASS == kCollide);

    const int nx = a.nx, ny = a.ny;
    const long long plane = a.plane;
    const int lane = threadIdx.x & (kWave - 1);
    const int tx = blockIdx.x % a.g.tiles_x;
    const int rg = blockIdx.x / a.g.tiles_x;
    const int x0 = (tx * kBlock + threadIdx.x) * VEC;
    const bool active = x0 < nx;
    const int y0 = rg * a.g.rows;
    const int y1 = min(y0 + a.g.rows, ny);

    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    R th[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        th[s][0] = F32 ? R(a.thr_f[s][0]) : R(a.thr[s][0]);
        th[s][1] = F32 ? R(a.thr_f[s][1]) : R(a.thr[s][1]);
    }
    double acc[kNsums];
#pragma unroll
    for (int k = 0; k < kNsums; ++k) acc[k] = 0.0;
    unsigned nfault = 0;

    // ring of PF + 1 rows: rows y .. y + PF - 1 are loaded or in flight while
    // row y is computed
    constexpr int PF = LKS_D2Q9_PREFETCH;
    R ring[PF + 1][9][VEC];
#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (y0 + p < y1) load_row<S, VEC, PULL>(fin, a.L, y0 + p, nx, ny, x0, active, lane, ring[p]);
    for (int y = y0; y < y1; ++y) {                 // uniform across the workgroup
        if (y + PF < y1) load_row<S, VEC, PULL>(fin, a.L, y + PF, nx, ny, x0, active, lane, ring[PF]);
        R (&cur)[9][VEC] = ring[0];
        const long long off = (long long)y * nx + x0;
        const long long poff = a.L.at(0, y, x0);

        if constexpr (PASS == kStream) {
            if (active) {
#pragma unroll
                for (int i = 0; i < 9; ++i) store_vec<S, VEC>(fout + i * a.L.pp + poff, cur[i]);
            }
        } else {
            R s_kl[VEC], s_neq[VEC], s_pi[VEC];
            uint8_t fl[VEC];
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                R dc[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) dc[i] = cur[i][k];
                R drho, jx, jy;
                LKS_CELL_BARRIER();
                const CellSense<R> cs = cell_update<R, SENSE, COLLIDE>(dc, rho0, inv_tau, drho, jx, jy, active);
#pragma unroll
                for (int i = 0; i < 9; ++i) cur[i][k] = dc[i];
                if constexpr (SENSE) {
                    LevelAcc lv;
                    const R sv[3] = {cs.kl, cs.neq, cs.pi};
#pragma unroll
                    for (int s = 0; s < 3; ++s) lv.add(sv[s], th[s][0], th[s][1]);
                    fl[k] = cs.fault ? uint8_t(0x82) : uint8_t(lv.level());
                    s_kl[k] = cs.kl;
                    s_neq[k] = cs.neq;
                    s_pi[k] = cs.pi;
                    if (active) {
                        // each cell's terms widen to FP64 before any add: FP64
                        // sums of FP32 values do not depend on the grouping,
                        // i.e. on the launch shape
                        acc[0] += (double)drho;
                        acc[1] += (double)jx;
                        acc[2] += (double)jy;
                        acc[4] += (double)cs.kl;
                        acc[5] += (double)cs.neq;
                        acc[6] += (double)cs.pi;
                        nfault += cs.fault ? 1u : 0u;
                    }
                }
            }
            if (active) {
                if constexpr (COLLIDE) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) store_vec<S, VEC>(fout + i * a.L.pp + poff, cur[i]);
                }
                if constexpr (SENSE) {
                    store_pack<R, VEC>(sens + off, s_kl);
                    store_pack<R, VEC>(sens + plane + off, s_neq);
                    store_pack<R, VEC>(sens + 2 * plane + off, s_pi);
                    store_pack<uint8_t, VEC>(flags + off, fl);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PF; ++p)
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int k = 0; k < VEC; ++k) ring[p][i][k] = ring[p + 1][i][k];
    }
    if constexpr (SENSE) {
        if (nfault) atomicAdd(faults, (unsigned long long)nfault);
        block_sums(acc, partials + (long long)blockIdx.x * kNsums);
    }
}

// Fused step with the next row staged through LDS by direct global->LDS
// loads: the row in flight occupies no registers.  Each wave owns a private
// 9 x 1 KB staging area.  A lane's VEC cells of population i are CHUNK bytes;
// they arrive in NP pieces of PS bytes (the direct loads move 1, 2, 4, 12 or
// 16 bytes per lane), piece p of lane l at i*1024 + p*64*PS + l*PS, and are
// read back by the same lane.
// how a lane's VEC cells of one population travel through the staging area
template <typename S, int VEC> struct StageGeom {
    static constexpr int CHUNK = VEC * (int)sizeof(typename Store<S>::raw);
    static constexpr int NP0 = CHUNK == 8 ? 2 : 1;
    static constexpr int PS0 = CHUNK / NP0;
    static constexpr int PE0 = PS0 / (int)sizeof(typename Store<S>::raw);
    // usable when every piece holds whole elements and is a whole number of
    // dwords: a sub-dword direct load writes lane l's value into the 4-byte
    // LDS slot l, not at (piece size) x l, so 1- and 2-byte pieces would not
    // land contiguously
    static constexpr bool ok = PE0 >= 1 && (PS0 == 4 || PS0 == 16);
    // (a geometry that is not ok is never launched; keep it compilable)
    static constexpr int NP = ok ? NP0 : 1;           // pieces per lane
    static constexpr int PS = ok ? PS0 : 4;           // bytes per piece
    static constexpr int PE = ok ? PE0 : 1;           // elements per piece
};

// NT: stores with the non-temporal hint (the launcher sets it when the two
// state buffers exceed the last-level cache, so the next step's loads come
// from HBM anyway)
template <typename S, int VEC, bool EXT = false, bool NT = false>
__global__ __launch_bounds__(kBlock) LKS_CELL_KERNEL_ATTR void d2q9_fused_lds(
    D2Q9Args a, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ fout,
    typename Store<S>::real* __restrict__ sens, uint8_t* __restrict__ flags,
    double* __restrict__ partials, unsigned long long* __restrict__ faults)
{
    using R = typename Store<S>::real;
    using raw = typename Store<S>::raw;
    using G = StageGeom<S, VEC>;
    typedef __attribute__((address_space(1))) void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    // per wave: one row of the nine planes, and for each x-shifted plane the
    // one value just outside the wave's span of cells
    __shared__ __attribute__((aligned(16))) unsigned char stage[kBlock / kWave][9][1024];
    __shared__ __attribute__((aligned(16))) unsigned char halo[kBlock / kWave][9][8];
    constexpr int ES = (int)sizeof(raw);        // bytes per element
    constexpr int EP = ES < 4 ? ES : 4;         // bytes per direct-load piece of an edge value
    constexpr int NEP = ES / EP;                // pieces per edge value

    const int nx = a.nx, ny = a.ny;
    const long long plane = a.plane;
    const int lane = threadIdx.x & (kWave - 1);
    // 16-bit storage (VALU-bound): the wave index taken wave-uniform, so the
    // staging area's LDS addresses are scalar, and row accesses as a uniform
    // row base plus a 32-bit lane offset (BF16 at 8192^2 649 -> 639 us; the
    // same forms made FP32 3 % slower, which keeps the plain ones)
    constexpr bool kHalf = sizeof(raw) == 2;
    const int wave = kHalf ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : threadIdx.x / kWave;
    const int tx = blockIdx.x % a.g.tiles_x;
    const int rg = blockIdx.x / a.g.tiles_x;
    const int x0 = (tx * kBlock + threadIdx.x) * VEC;
    const bool active = x0 < nx;
    const int y0 = rg * a.g.rows;
    const int y1 = min(y0 + a.g.rows, ny);
    // the wave's span of cells and its periodic neighbours (nx % VEC == 0)
    const int xw = (tx * kBlock + wave * kWave) * VEC;
    const bool wave_active = xw < nx;
    const int xl = xw == 0 ? nx - 1 : xw - 1;
    const int xr = xw + kWave * VEC >= nx ? 0 : xw + kWave * VEC;
    const bool last_lane = lane == kWave - 1 || x0 + VEC >= nx;

    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    R th[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        th[s][0] = F32 ? R(a.thr_f[s][0]) : R(a.thr[s][0]);
        th[s][1] = F32 ? R(a.thr_f[s][1]) : R(a.thr[s][1]);
    }
    double acc[kNsums];
#pragma unroll
    for (int k = 0; k < kNsums; ++k) acc[k] = 0.0;
    unsigned nfault = 0;

    // Row y of every plane into this wave's staging area.  Only direct
    // global->LDS loads: no register results, so nothing here makes the
    // wave wait for the loads it has just issued.
    auto issue = [&](int y) {
        static_for<9>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int cx = cx9(i), cy = cy9(i);
            int ys = y - cy;
            ys = ys < 0 ? ys + ny : (ys >= ny ? ys - ny : ys);
            const raw* row = fin + a.L.at(i, ys, 0);
            if (active) {
#pragma unroll
                for (int p = 0; p < G::NP; ++p) {
                    gvoid* g = kHalf ? (gvoid*)(row + (unsigned)(x0 + p * G::PE)) : (gvoid*)(row + x0 + p * G::PE);
                    lvoid* l = (lvoid*)&stage[wave][i][p * kWave * G::PS];
                    if constexpr (G::PS == 16) __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
                    else __builtin_amdgcn_global_load_lds(g, l, 4, 0, 0);
                }
            }
            if constexpr (cx != 0) {
                // lanes 0 .. NEP-1 fetch the pieces of the edge value (for a
                // 16-bit value only lane 0, whose LDS slot starts at offset 0)
                if (wave_active && lane < NEP) {
                    const int xe = cx == 1 ? xl : xr;
                    gvoid* g = (gvoid*)(reinterpret_cast<const unsigned char*>(row + xe) + lane * EP);
                    lvoid* l = (lvoid*)&halo[wave][i][0];
                    if constexpr (EP == 4) __builtin_amdgcn_global_load_lds(g, l, 4, 0, 0);
                    else if constexpr (EP == 2) __builtin_amdgcn_global_load_lds(g, l, 2, 0, 0);
                    else __builtin_amdgcn_global_load_lds(g, l, 1, 0, 0);
                }
            }
        });
    };

    // results of one row, stored while the next row computes
    R res[9][VEC];
    R s_kl[VEC], s_neq[VEC], s_pi[VEC];
    uint8_t fl[VEC];
    R xres[EXT ? kNumExt : 1][VEC];
    auto store_row = [&](int y) {
        if (active) {
            const long long off = (long long)y * nx + x0;
            if constexpr (kHalf) {
                const unsigned ux = (unsigned)x0;
                const long long srow = (long long)y * nx, prow = a.L.at(0, y, 0);
#pragma unroll
                for (int i = 0; i < 9; ++i) store_vec<S, VEC, NT>(fout + (i * a.L.pp + prow) + ux, res[i]);
                store_pack<R, VEC, NT>(sens + srow + ux, s_kl);
                store_pack<R, VEC, NT>(sens + (plane + srow) + ux, s_neq);
                store_pack<R, VEC, NT>(sens + (2 * plane + srow) + ux, s_pi);
                store_pack<uint8_t, VEC, NT>(flags + srow + ux, fl);
            } else {
                const long long poff = a.L.at(0, y, x0);
#pragma unroll
                for (int i = 0; i < 9; ++i) store_vec<S, VEC, NT>(fout + i * a.L.pp + poff, res[i]);
                store_pack<R, VEC, NT>(sens + off, s_kl);
                store_pack<R, VEC, NT>(sens + plane + off, s_neq);
                store_pack<R, VEC, NT>(sens + 2 * plane + off, s_pi);
                store_pack<uint8_t, VEC, NT>(flags + off, fl);
            }
            if constexpr (EXT) {
#pragma unroll
                for (int q = 0; q < kNumExt; ++q)
                    if (a.x.plane[q] >= 0) store_pack<R, VEC, NT>(sens + a.x.plane[q] * plane + off, xres[q]);
            }
        }
    };

    if (y0 < y1) issue(y0);
    for (int y = y0; y < y1; ++y) {                 // uniform across the workgroup
        // row y has landed in LDS (and the stores of row y - 2 have completed)
        wait_vmem_all();
        R cur[9][VEC];
        static_for<9>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            constexpr int cx = cx9(i);
            R v[VEC];
#pragma unroll
            for (int p = 0; p < G::NP; ++p) {
                R piece[G::PE];
                load_vec<S, G::PE>(reinterpret_cast<const raw*>(
                                       &stage[wave][i][p * kWave * G::PS + lane * G::PS]), piece);
#pragma unroll
                for (int k = 0; k < G::PE; ++k) v[p * G::PE + k] = piece[k];
            }
            if constexpr (cx == 0) {
#pragma unroll
                for (int k = 0; k < VEC; ++k) cur[i][k] = v[k];
            } else {
                const R e = Store<S>::to_real(*reinterpret_cast<const raw*>(&halo[wave][i][0]));
                if constexpr (cx == 1) {
                    const R prev = __shfl_up(v[VEC - 1], 1, kWave);
                    cur[i][0] = lane == 0 ? e : prev;
#pragma unroll
                    for (int k = 1; k < VEC; ++k) cur[i][k] = v[k - 1];
                } else {
                    const R next = __shfl_down(v[0], 1, kWave);
#pragma unroll
                    for (int k = 0; k + 1 < VEC; ++k) cur[i][k] = v[k + 1];
                    cur[i][VEC - 1] = last_lane ? e : next;
                }
            }
        });
        // the staging area is rewritten by the next row's loads only after
        // every lane's reads of this row have completed
        wait_lds_all();
        if (y + 1 < y1) issue(y + 1);
        // the previous row's stores go out after the next row's loads, so
        // the wait for those loads at the top of the next iteration has this
        // row's whole computation to cover both (stores count in vmcnt too)
        if (y > y0) store_row(y - 1);

#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            R dc[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) dc[i] = cur[i][k];
            R drho, jx, jy;
            R xv[kNumExt];
            LKS_CELL_BARRIER();
            const CellSense<R> cs = cell_update<R, true, true, EXT>(dc, rho0, inv_tau, drho, jx, jy, active,
                                                                    xv, a.x.mask);
#pragma unroll
            for (int i = 0; i < 9; ++i) res[i][k] = dc[i];
            LevelAcc lv;
            const R sv[3] = {cs.kl, cs.neq, cs.pi};
#pragma unroll
            for (int s = 0; s < 3; ++s) lv.add(sv[s], th[s][0], th[s][1]);
            if constexpr (EXT) {
#pragma unroll
                for (int q = 0; q < kNumExt; ++q) xres[q][k] = xv[q];
                ext_levels(a, xv, lv);
            }
            fl[k] = cs.fault ? uint8_t(0x82) : uint8_t(lv.level());
            s_kl[k] = cs.kl;
            s_neq[k] = cs.neq;
            s_pi[k] = cs.pi;
            if (active) {
                // each cell's terms widen to FP64 before any add (as above)
                acc[0] += (double)drho;
                acc[1] += (double)jx;
                acc[2] += (double)jy;
                acc[4] += (double)cs.kl;
                acc[5] += (double)cs.neq;
                acc[6] += (double)cs.pi;
                nfault += cs.fault ? 1u : 0u;
            }
        }
    }
    if (y0 < y1) store_row(y1 - 1);
    if (nfault) atomicAdd(faults, (unsigned long long)nfault);
    block_sums(acc, partials + (long long)blockIdx.x * kNsums);
}

// k steps of one tile per launch, small grids.  A step of a small grid is
// launch, load and store latency, not arithmetic: a workgroup that loads its
// TX x TY tile with a ring of k cells advances the tile k steps (odd k <= K,
// the ring shrinking by one cell a step) for one launch.  Step 0 gathers its
// populations from global memory, the later ones from LDS, where a step's
// post-collision values, rounded to the storage type as a stored state would
// be, replace those of the step before the last; one cell per thread and
// iteration, one copy of the cell update for all steps, so that little code is
// fetched.  Every cell's arithmetic is cell_update: state, sensors, flags and
// fault counts are the same bits as k one-step launches, and since each step's
// sums are taken over the same tiles in the same order whatever k is, so are
// the sums of any split of a run into launches.
// FP32, us per step of a 64-step call (the one-step row kernel in brackets):
// 64^2 1.8 (14.8), 128^2 1.9 (16.4), 256^2 2.6 (16.1); FP64 128^2 3.4 (14.9),
// BF16 256^2 2.5 (7.1).
// EXT: a call's last step with the extension sensors (K = 1; no staging buffer).
// Here and in the band kernel below one cell per lane holds 100-108 registers
// (FP64 164-192) where the row kernel with four holds 247 (FP64, two: 312), so
// that two to four times as many waves hide its latency.  A call of one step with
// nine of them, us, the row kernel in brackets: FP32 128^2 11.2 (14.4), 512^2 16.2
// (21.5), 2048^2 123 (141-149), 4096^2 445 (486); FP64 512^2 38 (45), 2048^2 517 (560).
template <typename S, int TX, int TY, int K> struct TileSteps {
    using raw = typename Store<S>::raw;
    using R = typename Store<S>::real;
    static constexpr int kCells = (TX + 2 * (K - 1)) * (TY + 2 * (K - 1));   // cells step 0 may produce
    static constexpr int kThreads = kCells >= 1024 ? 1024 : (kCells + kWave - 1) / kWave * kWave;
    static constexpr int kTile = TX * TY;
    static constexpr int kSums = 6;                                          // sums a D2Q9 step has
    static_assert(kTile % kWave == 0, "a wave reads whole rows of terms");
};

// Sum of one value per lane over the wave, in lane 63: additions of the lanes
// below within rows of 16 (DPP row shifts), then of the rows.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
    return v + __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum_lane63(double v)
{
    v = dpp_add<0x111, 0xf>(v);      // row_shr:1
    v = dpp_add<0x112, 0xf>(v);      // row_shr:2
    v = dpp_add<0x114, 0xf>(v);      // row_shr:4
    v = dpp_add<0x118, 0xf>(v);      // row_shr:8
    v = dpp_add<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}

template <typename S, int TX, int TY, int K, bool EXT = false>
__global__ __launch_bounds__((TileSteps<S, TX, TY, K>::kThreads)) void d2q9_tile_kernel(
    D2Q9Args a, int k, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ fout,
    typename Store<S>::real* __restrict__ sens, uint8_t* __restrict__ flags, double* __restrict__ partials,
    int first, unsigned long long* __restrict__ faults)
{
    using G = TileSteps<S, TX, TY, K>;
    using R = typename G::R;
    using raw = typename G::raw;
    __shared__ raw buf[2][K > 1 ? 9 * G::kCells : 1];
    __shared__ R terms[2][G::kSums][G::kTile];

    const int nx = a.nx, ny = a.ny;
    const int tiles_x = (nx + TX - 1) / TX;
    const int X0 = (blockIdx.x % tiles_x) * TX, Y0 = (blockIdx.x / tiles_x) * TY;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nwaves = blockDim.x / kWave;
    const unsigned pp = (unsigned)a.L.pp, pr = (unsigned)a.L.pr, plane = (unsigned)a.plane;

    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    R th[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        th[s][0] = F32 ? R(a.thr_f[s][0]) : R(a.thr[s][0]);
        th[s][1] = F32 ? R(a.thr_f[s][1]) : R(a.thr[s][1]);
    }
    const int h0 = k - 1, W0 = TX + 2 * h0;        // LDS cell (x, y) of the tile: (y + h0) W0 + x + h0
    unsigned nfault = 0;

    // the sums of one step from its terms: one wave per quantity (the sums
    // of steps before `first` are not kept)
    auto reduce = [&](int j) {
        if (j < first) return;
        for (int q = wave; q < G::kSums; q += nwaves) {
            double v = 0.0;
#pragma unroll
            for (int m = 0; m < G::kTile / kWave; ++m) v += (double)terms[j & 1][q][m * kWave + lane];
            v = wave_sum_lane63(v);
            // quantities 0..2: mass, momentum; 3..5: the sensors, sums 4..6
            double* out = partials + ((long long)(j - first) * gridDim.x + blockIdx.x) * kNsums;
            if (lane == kWave - 1) {
                out[q < 3 ? q : q + 1] = v;
                if (q == 0) out[3] = out[7] = 0.0;
            }
        }
    };

    for (int j = 0; j < k; ++j) {
        const int h = k - 1 - j, W = TX + 2 * h, n = W * (TY + 2 * h);
        const float rW = 1.0f / (float)W;
        const bool last = j == k - 1;
        for (int e = threadIdx.x; e < n; e += blockDim.x) {
            // e = r W + c; exact: e < 4096 and (e + 0.5)/W is at least 1/(2W) off an integer
            const int r = (int)(((float)e + 0.5f) * rW);
            const int x = e - r * W - h, y = r - h;
            const int cell = (y + h0) * W0 + x + h0;
            R d[9];
            if (K == 1 || j == 0) {
                const int gx = X0 + x, gy = Y0 + y;
                // one period off at most (tile_fits)
                unsigned xs[3], ys[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    int u = gx + q - 1, v = gy + q - 1;
                    u += u < 0 ? nx : 0;
                    u -= u >= nx ? nx : 0;
                    v += v < 0 ? ny : 0;
                    v -= v >= ny ? ny : 0;
                    xs[q] = (unsigned)u;
                    ys[q] = (unsigned)v * pr;
                }
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    d[i] = Store<S>::to_real(fin[i * pp + ys[1 - cy9(i)] + xs[1 - cx9(i)]]);
            } else {
                const raw* src = buf[(j - 1) & 1];
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    d[i] = Store<S>::to_real(src[i * G::kCells + cell - cy9(i) * W0 - cx9(i)]);
            }
            R drho, jx, jy;
            R xv[EXT ? kNumExt : 1];
            const CellSense<R> cs = cell_update<R, true, true, EXT>(d, rho0, inv_tau, drho, jx, jy, {}, xv,
                                                                    a.x.mask);
            if (K > 1 && !last) {
                raw* dst = buf[j & 1];
#pragma unroll
                for (int i = 0; i < 9; ++i) dst[i * G::kCells + cell] = Store<S>::from_real(d[i]);
            }
            if (x >= 0 && x < TX && y >= 0 && y < TY) {
                const bool own = X0 + x < nx && Y0 + y < ny;
                const int t = y * TX + x;
                terms[j & 1][0][t] = own ? drho : R(0);
                terms[j & 1][1][t] = own ? jx : R(0);
                terms[j & 1][2][t] = own ? jy : R(0);
                terms[j & 1][3][t] = own ? cs.kl : R(0);
                terms[j & 1][4][t] = own ? cs.neq : R(0);
                terms[j & 1][5][t] = own ? cs.pi : R(0);
                nfault += own && cs.fault ? 1u : 0u;
                if (last && own) {
                    const unsigned off = (unsigned)(Y0 + y) * (unsigned)nx + (unsigned)(X0 + x);
                    const unsigned po = (unsigned)(Y0 + y) * pr + (unsigned)(X0 + x);
#pragma unroll
                    for (int i = 0; i < 9; ++i) fout[i * pp + po] = Store<S>::from_real(d[i]);
                    // a call's last step is a launch of its own: longer
                    // launches' sensors and flags would be overwritten
                    if (k == 1) {
                        LevelAcc lv;
                        const R sv[3] = {cs.kl, cs.neq, cs.pi};
#pragma unroll
                        for (int s = 0; s < 3; ++s) lv.add(sv[s], th[s][0], th[s][1]);
                        if constexpr (EXT) {
                            ext_levels(a, xv, lv);
#pragma unroll
                            for (int q = 0; q < kNumExt; ++q)
                                if (a.x.plane[q] >= 0) sens[a.x.plane[q] * a.plane + off] = xv[q];
                        }
                        sens[off] = cs.kl;
                        sens[plane + off] = cs.neq;
                        sens[2 * plane + off] = cs.pi;
                        flags[off] = cs.fault ? uint8_t(0x82) : uint8_t(lv.level());
                    }
                }
            }
        }
        __syncthreads();
        // the terms of step j are rewritten in step j + 2, behind another barrier
        reduce(j);
    }
    if (nfault) atomicAdd(faults, (unsigned long long)nfault);
}

// Sums over the wave of six values: halves, then 16-lane rows, then 8-lane
// halves of rows, of two values are exchanged and added (each lane then
// carries one of them), and the eight lanes that are left added up.  Lanes 0, 16, 32, 48
// return values 0, 2, 1, 3, lanes 8 and 40 values 4 and 5.
__device__ __forceinline__ double swap_add32(double x, double y)
{
    const unsigned long long ux = __builtin_bit_cast(unsigned long long, x), uy = __builtin_bit_cast(unsigned long long, y);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ux, (unsigned)uy, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ux >> 32), (unsigned)(uy >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double swap_add16(double x, double y)
{
    const unsigned long long ux = __builtin_bit_cast(unsigned long long, x), uy = __builtin_bit_cast(unsigned long long, y);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ux, (unsigned)uy, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ux >> 32), (unsigned)(uy >> 32), false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}
template <int CTRL> __device__ __forceinline__ double dpp_move(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sums6(const double (&v)[6], bool upper8)
{
    const double p = swap_add32(v[0], v[1]), q = swap_add32(v[2], v[3]), r = swap_add32(v[4], v[5]);
    const double a = swap_add16(p, q), b = swap_add16(r, r);
    double s = (upper8 ? b : a) + dpp_move<0x128>(upper8 ? a : b);      // row_ror:8
    s += dpp_move<0x141>(s);                                            // row_half_mirror
    s += dpp_move<0x4e>(s);                                             // quad_perm 2 3 0 1
    return s + dpp_move<0xb1>(s);                                       // quad_perm 1 0 3 2
}

// Three steps of one tile per launch, mid-size and large grids.  A one-step
// kernel moves 85 B per cell and step (FP32) and waits for HBM; three steps
// for one pass leave the VALU issue as the bound.  A workgroup of eight waves
// owns 64 columns and 8 NR rows, NR rows a wave, one lane a column.  Step 0 reads
// its populations from global memory (the tile and a ring of two cells, whose
// cells are dealt out densely over the waves) and writes the post-collision
// values, rounded to the storage type, to LDS; step 1 (the tile and a ring of
// one cell) reads them, holds its results in registers across a barrier and
// writes them in their place; step 2 stores the state.  In place, the 68 x 20
// (NR = 2) or 68 x 28 cells take 49 or 69 KB in FP32, so that two workgroups
// share a CU and one's loads and stores hide behind the other's arithmetic.
// Populations reach their neighbours in x and y through the LDS buffer alone.
// K = 1: a single step on the same tiles, so that every step's sums are added
// in the same order whichever launch it runs in.  Cell arithmetic:
// cell_update (246 VALU instructions, of which ring cells need 100).  A row's
// sums cost 88 instructions with a reduction of each of the six values; what
// is left after sharing it (wave_sums6), keeping lanes outside the grid out of
// it only where there are any, and counting faults by ballot took 142 to 129 us
// per step at FP32 4096^2, NR = 2.
// us per step (the one-step row kernel in brackets): FP32 512^2 4.0 (17.5),
// 1024^2 10.9 (17.9), 2048^2 34 (68.8), 4096^2 122 (239); FP64 1024^2 24
// (33.6), 4096^2 310 (468); BF16 1024^2 10.9 (16.1), 4096^2 125 (178).
template <typename S, int K, int NR, bool NT, bool EXT = false>
__global__ __launch_bounds__(kBandWaves * kWave) __attribute__((amdgpu_waves_per_eu(sizeof(typename Store<S>::real) == 4 && !EXT ? 4 : 2))) void d2q9_band_kernel(
    D2Q9Args a, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ fout,
    typename Store<S>::real* __restrict__ sens, uint8_t* __restrict__ flags, double* __restrict__ partials,
    int first, int nblocks, unsigned long long* __restrict__ faults)
{
    static_assert(K == 1 || (K == 3 && !EXT), "one or three steps, extension sensors in single ones");
    using G = Band<K, NR>;
    using R = typename Store<S>::real;
    using raw = typename Store<S>::raw;
    constexpr int NW = G::NW, TX = G::TX, TY = G::TY, W0 = G::W0, C = G::kCells;
    __shared__ raw buf[9 * C];
    __shared__ double red[K][NW][6];

    const int tile = G::tile();
    if (tile >= nblocks) return;                    // whole workgroups
    const int nx = a.nx, ny = a.ny;
    const int tiles_x = (nx + TX - 1) / TX;
    const int X0 = (tile % tiles_x) * TX, Y0 = (tile / tiles_x) * TY;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);

    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    R th[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        th[s][0] = F32 ? R(a.thr_f[s][0]) : R(a.thr[s][0]);
        th[s][1] = F32 ? R(a.thr_f[s][1]) : R(a.thr[s][1]);
    }
    unsigned nfault = 0;
    unsigned xs[3];                                 // this lane's column and its neighbours
#pragma unroll
    for (int q = 0; q < 3; ++q) xs[q] = (unsigned)G::wrap(X0 + lane + q - 1, nx);

    auto put = [&](int cell, const R (&d)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) buf[i * C + cell] = Store<S>::from_real(d[i]);
    };
    auto get = [&](int cell, R (&d)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = Store<S>::to_real(buf[i * C + cell - cy9(i) * W0 - cx9(i)]);
    };
    // the owned rows of this wave at one step, after their gather
    const bool whole = X0 + TX <= nx && Y0 + TY <= ny;      // no cell outside the grid
    auto owned = [&](int j, R (&d)[G::NR][9], bool last) {
        R t[G::NR][6];                                  // the step's sums: mass, momentum, sensors
#pragma unroll
        for (int r = 0; r < G::NR; ++r) {
            const int y = G::NR * wave + r;
            const bool own = X0 + lane < nx && Y0 + y < ny;
            R drho, jx, jy;
            R xv[EXT ? kNumExt : 1];
            const CellSense<R> cs = cell_update<R, true, true, EXT>(d[r], rho0, inv_tau, drho, jx, jy, {}, xv,
                                                                    a.x.mask);
            t[r][0] = drho;
            t[r][1] = jx;
            t[r][2] = jy;
            t[r][3] = cs.kl;
            t[r][4] = cs.neq;
            t[r][5] = cs.pi;
            nfault += (unsigned)__builtin_popcountll(__ballot(own && cs.fault));
            if (last && own) {
                const unsigned X = (unsigned)(X0 + lane);
                const long long prow = a.L.at(0, Y0 + y, 0), srow = (long long)(Y0 + y) * nx;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const R o[1] = {d[r][i]};
                    store_vec<S, 1, NT>(fout + (prow + i * a.L.pp) + X, o);
                }
                // a call's last step is a launch of its own: longer launches'
                // sensors and flags would be overwritten
                if constexpr (K == 1) {
                    LevelAcc lv;
                    const R sv[3] = {cs.kl, cs.neq, cs.pi};
#pragma unroll
                    for (int s = 0; s < 3; ++s) lv.add(sv[s], th[s][0], th[s][1]);
                    if constexpr (EXT) {
                        ext_levels(a, xv, lv);
#pragma unroll
                        for (int q = 0; q < kNumExt; ++q) {
                            const R x[1] = {xv[q]};
                            if (a.x.plane[q] >= 0)
                                store_pack<R, 1, NT>(sens + (a.x.plane[q] * a.plane + srow) + X, x);
                        }
                    }
                    const R kl[1] = {cs.kl}, neq[1] = {cs.neq}, pi[1] = {cs.pi};
                    const uint8_t fl[1] = {cs.fault ? uint8_t(0x82) : uint8_t(lv.level())};
                    store_pack<R, 1, NT>(sens + srow + X, kl);
                    store_pack<R, 1, NT>(sens + (a.plane + srow) + X, neq);
                    store_pack<R, 1, NT>(sens + (2 * a.plane + srow) + X, pi);
                    store_pack<uint8_t, 1, NT>(flags + srow + X, fl);
                }
            }
        }
        if (j < first) return;                      // sums not kept
        if (!whole) {
#pragma unroll
            for (int r = 0; r < G::NR; ++r) {
                const bool own = X0 + lane < nx && Y0 + G::NR * wave + r < ny;
#pragma unroll
                for (int q = 0; q < 6; ++q) t[r][q] = own ? t[r][q] : R(0);
            }
        }
        // each cell's terms widen to FP64 before any add
        double v[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            v[q] = (double)t[0][q];
#pragma unroll
            for (int r = 1; r < G::NR; ++r) v[q] += (double)t[r][q];
        }
        const double s = wave_sums6(v, lane & 8);
        if (lane % 8 == 0) {
            const int row = lane / 16;              // values 0, 2, 1, 3 by row; 4 and 5 in lanes 8 and 40
            if (!(lane & 8)) red[j][wave][row == 1 ? 2 : row == 2 ? 1 : row] = s;
            else if (row % 2 == 0) red[j][wave][4 + row / 2] = s;
        }
    };
    auto ring_update = [&](R (&d)[9]) {
        R drho, jx, jy;
        (void)cell_update<R, true, true>(d, rho0, inv_tau, drho, jx, jy);
    };

    {   // ---- step 0: from global memory
        R d[G::NR][9];
#pragma unroll
        for (int r = 0; r < G::NR; ++r) {
            static_for<9>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const int ys = G::wrap(Y0 + G::NR * wave + r - cy9(i), ny);
                d[r][i] = Store<S>::to_real((fin + a.L.at(i, ys, 0))[xs[1 - cx9(i)]]);
            });
        }
        R g[9];
        int cell = 0;
        bool ring = false;
        if constexpr (K > 1) {
            int x, y;
            ring = (int)threadIdx.x < G::template ring<G::H0>();
            if (ring) {
                G::template ring_cell<G::H0>(threadIdx.x, x, y);
                cell = G::cell(x, y);
                long long row[3];
                int col[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    row[q] = (long long)G::wrap(Y0 + y + q - 1, ny) * a.L.pr;
                    col[q] = G::wrap(X0 + x + q - 1, nx);
                }
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    g[i] = Store<S>::to_real(fin[i * a.L.pp + row[1 - cy9(i)] + col[1 - cx9(i)]]);
            }
        }
        owned(0, d, K == 1);
        if constexpr (K > 1) {
#pragma unroll
            for (int r = 0; r < G::NR; ++r) put(G::cell(lane, G::NR * wave + r), d[r]);
            if (ring) {
                ring_update(g);
                put(cell, g);
            }
        }
    }
    __syncthreads();
    if constexpr (K > 1) {
        {   // ---- step 1: in place
            R d[G::NR][9], g[9];
            int cell = 0;
            // the ring goes to the waves that had none, or less, of step 0's
            const int e = NW * kWave - 1 - (int)threadIdx.x;
            const bool ring = e < G::template ring<1>();
#pragma unroll
            for (int r = 0; r < G::NR; ++r) get(G::cell(lane, G::NR * wave + r), d[r]);
            owned(1, d, false);
            if (ring) {
                int x, y;
                G::template ring_cell<1>(e, x, y);
                cell = G::cell(x, y);
                get(cell, g);
                ring_update(g);
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < G::NR; ++r) put(G::cell(lane, G::NR * wave + r), d[r]);
            if (ring) put(cell, g);
        }
        __syncthreads();
        {   // ---- step 2: to global memory
            R d[G::NR][9];
#pragma unroll
            for (int r = 0; r < G::NR; ++r) get(G::cell(lane, G::NR * wave + r), d[r]);
            owned(2, d, true);
        }
        __syncthreads();
    }
    if (threadIdx.x < K * kNsums) {
        const int j = threadIdx.x / kNsums, k = threadIdx.x % kNsums;
        double s = 0.0;
        if (k != 3 && k != 7) {
#pragma unroll
            for (int w = 0; w < NW; ++w) s += red[j][w][k < 3 ? k : k - 1];
        }
        if (j >= first) partials[((long long)(j - first) * nblocks + tile) * kNsums + k] = s;
    }
    if (nfault && lane == 0) atomicAdd(faults, (unsigned long long)nfault);      // counted per wave
}

// K steps of the state alone (no sensors, flags, sums or fault count), as the
// adjoint replays a trajectory: the band kernel's geometry and staging, each
// step's state stored where the caller wants it (out0, out1: null to skip).
// HBM-bound with every state stored (FP32 1024^2: 12 B read + 36 B written per
// cell and step), VALU-bound with the last one only.
template <typename S, int K>
__global__ __launch_bounds__(kBandWaves * kWave) void d2q9_band_state_kernel(
    D2Q9Args a, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ out0,
    typename Store<S>::raw* __restrict__ out1, typename Store<S>::raw* __restrict__ out2, int ntiles)
{
    static_assert(K == 1 || K == 3, "one or three steps");
    using G = Band<K, 2>;
    using R = typename Store<S>::real;
    using raw = typename Store<S>::raw;
    constexpr int W0 = G::W0, C = G::kCells;
    __shared__ raw buf[9 * C];

    const int tile = G::tile();
    if (tile >= ntiles) return;                     // whole workgroups
    const int nx = a.nx, ny = a.ny;
    const int tiles_x = (nx + G::TX - 1) / G::TX;
    const int X0 = (tile % tiles_x) * G::TX, Y0 = (tile / tiles_x) * G::TY;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    unsigned xs[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) xs[q] = (unsigned)G::wrap(X0 + lane + q - 1, nx);

    auto put = [&](int cell, const R (&d)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) buf[i * C + cell] = Store<S>::from_real(d[i]);
    };
    auto get = [&](int cell, R (&d)[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = Store<S>::to_real(buf[i * C + cell - cy9(i) * W0 - cx9(i)]);
    };
    auto step = [&](R (&d)[9]) {
        R drho, jx, jy;
        (void)cell_update<R, false, true, false, true>(d, rho0, inv_tau, drho, jx, jy);
    };
    auto store = [&](raw* out, const R (&d)[G::NR][9]) {
        if (!out || X0 + lane >= nx) return;
#pragma unroll
        for (int r = 0; r < G::NR; ++r) {
            const int Y = Y0 + G::NR * wave + r;
            if (Y >= ny) break;
            const long long prow = a.L.at(0, Y, 0);
#pragma unroll
            for (int i = 0; i < 9; ++i)
                (out + (prow + i * a.L.pp))[(unsigned)(X0 + lane)] = Store<S>::from_real(d[r][i]);
        }
    };

    {   // ---- step 0: from global memory
        R d[G::NR][9], g[9];
#pragma unroll
        for (int r = 0; r < G::NR; ++r) {
            static_for<9>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const int ys = G::wrap(Y0 + G::NR * wave + r - cy9(i), ny);
                d[r][i] = Store<S>::to_real((fin + a.L.at(i, ys, 0))[xs[1 - cx9(i)]]);
            });
        }
        const bool ring = K > 1 && (int)threadIdx.x < G::template ring<G::H0>();
        int cell = 0;
        if constexpr (K > 1) {
            if (ring) {
                int x, y;
                G::template ring_cell<G::H0>(threadIdx.x, x, y);
                cell = G::cell(x, y);
                long long row[3];
                int col[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    row[q] = (long long)G::wrap(Y0 + y + q - 1, ny) * a.L.pr;
                    col[q] = G::wrap(X0 + x + q - 1, nx);
                }
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    g[i] = Store<S>::to_real(fin[i * a.L.pp + row[1 - cy9(i)] + col[1 - cx9(i)]]);
            }
        }
#pragma unroll
        for (int r = 0; r < G::NR; ++r) step(d[r]);
        store(out0, d);
        if constexpr (K > 1) {
#pragma unroll
            for (int r = 0; r < G::NR; ++r) put(G::cell(lane, G::NR * wave + r), d[r]);
            if (ring) {
                step(g);
                put(cell, g);
            }
        }
    }
    if constexpr (K > 1) {
        __syncthreads();
        {   // ---- step 1: in place
            R d[G::NR][9], g[9];
            int cell = 0;
            // the ring goes to the waves that had none, or less, of step 0's
            const int e = G::NW * kWave - 1 - (int)threadIdx.x;
            const bool ring = e < G::template ring<1>();
#pragma unroll
            for (int r = 0; r < G::NR; ++r) get(G::cell(lane, G::NR * wave + r), d[r]);
#pragma unroll
            for (int r = 0; r < G::NR; ++r) step(d[r]);
            if (ring) {
                int x, y;
                G::template ring_cell<1>(e, x, y);
                cell = G::cell(x, y);
                get(cell, g);
                step(g);
            }
            store(out1, d);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < G::NR; ++r) put(G::cell(lane, G::NR * wave + r), d[r]);
            if (ring) put(cell, g);
        }
        __syncthreads();
        {   // ---- step 2: to global memory
            R d[G::NR][9];
#pragma unroll
            for (int r = 0; r < G::NR; ++r) get(G::cell(lane, G::NR * wave + r), d[r]);
#pragma unroll
            for (int r = 0; r < G::NR; ++r) step(d[r]);
            store(out2, d);
        }
    }
}

// Two fused steps per pass over HBM (temporal blocking): the API keeps
// only the last step's sensors and flags, so a wave can advance its cells two
// steps from one read of the state.  Each wave owns a strip of kSweepW = 60
// columns and kSweepH rows: its 64 lanes hold the strip and a two-column ring
// (periodic), one column per lane, and the wave sweeps down the rows with its
// state in registers.  Raw row q arrives; step A runs on row q - 1 (lanes 1 to
// 62: the strip and a one-column ring), with the x neighbours from the
// adjacent lanes (DPP wave shifts) and the y neighbours from the two previous
// raw rows; its post-collision values, rounded to the storage type as a stored
// state would be, feed step B in the same way.  Step B runs on row q - 3
// (lanes 2 to 61) from step-A rows of earlier iterations, so the two cell
// updates of an iteration are independent and their instructions interleave.
// The strip's rows plus a two-row ring are read once; step B stores
// populations, sensors and flags.  No LDS and no barrier until the final sums.
// Each cell's sums and faults are counted by the wave that owns it, for both
// steps.  The loads of raw rows q + 1 and q + 2 are in flight while row q is
// used.  kSweepH = 16 rows per wave: short strips give more independent waves,
// which hides latency better than the shorter ring of tall strips saves bytes.
// Each cell's arithmetic is cell_update, as in the one-step kernels, so the
// results are bit-identical to two one-step launches.  A step that has no
// partner (an odd batch end) runs in the one-step kernel: this sweep with a
// single step measured 362.8 against 233.2 us at 4096^2.
constexpr int kSweepW = kWave - 4;
constexpr int kSweepH = 16;

// Periodic index for j in [-2, n + 1] (exact for n >= 2; n = 1 maps every j
// to 0).  Indexes further out only feed cells that are not stored: any
// in-range index serves them, so they are clamped.
__device__ __forceinline__ int wrap_index(int j, int n)
{
    j += j < 0 ? n : 0;
    j -= j >= n ? n : 0;
    return min(max(j, 0), n - 1);
}

// The value of lane l - CX (CX = +1: from the lane below, -1: from the lane
// above); lanes whose source is outside the wave get 0.
template <int CX>
__device__ __forceinline__ float lane_shift(float v)
{
    if constexpr (CX == 0) {
        return v;
    } else {
        constexpr int ctrl = CX > 0 ? 0x138 : 0x130;    // wave_shr:1 / wave_shl:1
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl,
                                                                     0xf, 0xf, false));
    }
}
template <int CX>
__device__ __forceinline__ double lane_shift(double v)
{
    if constexpr (CX == 0) {
        return v;
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const float lo = lane_shift<CX>(__builtin_bit_cast(float, (unsigned)u));
        const float hi = lane_shift<CX>(__builtin_bit_cast(float, (unsigned)(u >> 32)));
        return __builtin_bit_cast(double, (unsigned long long)__builtin_bit_cast(unsigned, lo) |
                                              ((unsigned long long)__builtin_bit_cast(unsigned, hi) << 32));
    }
}

// Pre-step values of a cell at row y: population i from row y - cy_i (prev2,
// prev, cur for cy = +1, 0, -1) and lane l - cx_i.
template <typename R>
__device__ __forceinline__ void gather_pull(R (&d)[9], const R (&prev2)[9], const R (&prev)[9], const R (&cur)[9])
{
    static_for<9>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int cy = cy9(i), cx = cx9(i);
        const R v = cy > 0 ? prev2[i] : (cy == 0 ? prev[i] : cur[i]);
        d[i] = lane_shift<cx>(v);
    });
}

template <typename S>
__global__ __launch_bounds__(kBlock) void d2q9_fused2_kernel(
    D2Q9Args a, const typename Store<S>::raw* __restrict__ fin, typename Store<S>::raw* __restrict__ fout,
    typename Store<S>::real* __restrict__ sens, uint8_t* __restrict__ flags, double* __restrict__ part_a,
    double* __restrict__ part_b, unsigned long long* __restrict__ faults)
{
    using R = typename Store<S>::real;
    const int nx = a.nx, ny = a.ny;
    const long long plane = a.plane;
    const int lane = threadIdx.x & (kWave - 1);
    const int strips = (nx + kSweepW - 1) / kSweepW, segs = (ny + kSweepH - 1) / kSweepH;
    const int wid = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const bool has = wid < strips * segs;
    const int X0 = (wid % strips) * kSweepW, Yb = (wid / strips) * kSweepH;
    const int Ye = min(Yb + kSweepH, ny);
    const int X = X0 - 2 + lane;                  // this lane's column
    const int gx = wrap_index(X, nx);
    const bool own_col = lane >= 2 && lane < kSweepW + 2 && X < nx;

    constexpr bool F32 = sizeof(R) == 4;
    const R rho0 = F32 ? R(a.rho0_f) : R(a.rho0);
    const R inv_tau = F32 ? R(a.inv_tau_f) : R(1.0 / a.tau);
    R th[3][2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        th[k][0] = F32 ? R(a.thr_f[k][0]) : R(a.thr[k][0]);
        th[k][1] = F32 ? R(a.thr_f[k][1]) : R(a.thr[k][1]);
    }
    auto level_of = [&](const CellSense<R>& cs) {
        LevelAcc lv;
        const R sv[3] = {cs.kl, cs.neq, cs.pi};
#pragma unroll
        for (int k = 0; k < 3; ++k) lv.add(sv[k], th[k][0], th[k][1]);
        return cs.fault ? uint8_t(0x82) : uint8_t(lv.level());
    };
    auto store_cell = [&](int Y, const R (&d)[9], const CellSense<R>& cs) {
        const long long off = (long long)Y * nx + X;
#pragma unroll
        for (int i = 0; i < 9; ++i) fout[a.L.at(i, Y, X)] = Store<S>::from_real(d[i]);
        sens[off] = cs.kl;
        sens[plane + off] = cs.neq;
        sens[2 * plane + off] = cs.pi;
        flags[off] = level_of(cs);
    };
    auto add_sums = [&](double (&acc)[kNsums], unsigned& nf, R drho, R jx, R jy, const CellSense<R>& cs) {
        acc[0] += (double)drho;
        acc[1] += (double)jx;
        acc[2] += (double)jy;
        acc[4] += (double)cs.kl;
        acc[5] += (double)cs.neq;
        acc[6] += (double)cs.pi;
        nf += cs.fault ? 1u : 0u;
    };
    auto load_row = [&](int q, R (&r)[9]) {
        const int gy = wrap_index(q, ny);
#pragma unroll
        for (int i = 0; i < 9; ++i) r[i] = Store<S>::to_real(fin[a.L.at(i, gy, gx)]);
    };

    double acc_a[kNsums], acc_b[kNsums];
#pragma unroll
    for (int k = 0; k < kNsums; ++k) acc_a[k] = acc_b[k] = 0.0;
    unsigned nfault = 0;

    if (has) {
        // raw rows qs .. qe; step A on rows qs + 1 .. qe - 1, step B on Yb .. Ye - 1
        const int qs = Yb - 2, qe = Ye + 1;
        R prev2[9], prev[9], cur[9], nxt[9] = {}, nxt2[9] = {};
        R aprev3[9], aprev2[9], aprev[9];
        load_row(qs, prev2);
        load_row(qs + 1, prev);
        load_row(qs + 2, cur);
        if (qs + 3 <= qe) load_row(qs + 3, nxt);
        const int qend = qe + 1;
        for (int q = qs + 2; q <= qend; ++q) {
            if (q + 2 <= qe) load_row(q + 2, nxt2);
            // ---- step B on row q - 3 (step A rows q - 4, q - 3, q - 2 of earlier iterations)
            if (q >= qs + 5) {
                R e[9];
                gather_pull(e, aprev3, aprev2, aprev);
                R drho2, jx2, jy2;
                const CellSense<R> cs2 = cell_update<R, true, true>(e, rho0, inv_tau, drho2, jx2, jy2, own_col);
                if (own_col) {
                    store_cell(q - 3, e, cs2);
                    add_sums(acc_b, nfault, drho2, jx2, jy2, cs2);
                }
            }
            if (q <= qe) {
                const int ya = q - 1;
                R d[9];
                gather_pull(d, prev2, prev, cur);
                R drho, jx, jy;
                const bool own_a = own_col && ya >= Yb && ya < Ye;
                const CellSense<R> cs = cell_update<R, true, true>(d, rho0, inv_tau, drho, jx, jy, own_a);
                if (own_a) add_sums(acc_a, nfault, drho, jx, jy, cs);
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    aprev3[i] = aprev2[i];
                    aprev2[i] = aprev[i];
                    aprev[i] = Store<S>::to_real(Store<S>::from_real(d[i]));
                }
            }
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                prev2[i] = prev[i];
                prev[i] = cur[i];
                cur[i] = nxt[i];
                nxt[i] = nxt2[i];
            }
        }
    }
    block_sums(acc_a, part_a + (long long)blockIdx.x * kNsums);
    __syncthreads();                              // block_sums' LDS is read before it is written again
    block_sums(acc_b, part_b + (long long)blockIdx.x * kNsums);
    if (nfault) atomicAdd(faults, (unsigned long long)nfault);
}

template <typename S>
static hipError_t launch_two(const D2Q9Args& a, const void* fin, void* fout, void* sens, uint8_t* flags,
                             double* part_a, double* part_b, unsigned long long* faults, hipStream_t st)
{
    using raw = typename Store<S>::raw;
    using R = typename Store<S>::real;
    const dim3 grid((unsigned)d2q9_two_blocks(sizeof(raw) == 8 ? 0 : 1, a.nx, a.ny)), block(kBlock);
    d2q9_fused2_kernel<S><<<grid, block, 0, st>>>(a, (const raw*)fin, (raw*)fout, (R*)sens, flags, part_a,
                                                  part_b, faults);
    return hipGetLastError();
}

// Workgroups of the two-step launches: one wave per strip of kSweepW columns
// and kSweepH rows.
int d2q9_two_blocks(int dtype, int nx, int ny)
{
    (void)dtype;
    const long long waves = (long long)((nx + kSweepW - 1) / kSweepW) * ((ny + kSweepH - 1) / kSweepH);
    return (int)((waves + kBlock / kWave - 1) / (kBlock / kWave));
}

hipError_t launch_d2q9_two(int dtype, const D2Q9Args& a, const void* fin, void* fout, void* sens,
                           uint8_t* flags, double* part_a, double* part_b, unsigned long long* faults,
                           hipStream_t s)
{
    switch (dtype) {
    case 0: return launch_two<double>(a, fin, fout, sens, flags, part_a, part_b, faults, s);
    case 1: return launch_two<float>(a, fin, fout, sens, flags, part_a, part_b, faults, s);
    case 2: return launch_two<bf16_t>(a, fin, fout, sens, flags, part_a, part_b, faults, s);
    case 3: return launch_two<f16_t>(a, fin, fout, sens, flags, part_a, part_b, faults, s);
    default: return hipErrorInvalidValue;
    }
}

// Grids that the tile kernel takes: its tiles fit, and the element indexes of
// the state, which it forms in 32 bits, lie below 2^32 (477 million cells; a
// grid that long and too narrow for the band kernel, whose indexes have 64
// bits, runs the row kernel).
static bool tile_takes(int nx, int ny, int TX, int TY, int K)
{
    return tile_fits(nx, TX, K) && tile_fits(ny, TY, K) && 9LL * nx * ny <= 1LL << 32;
}

template <typename S, int TX, int TY, int K>
static hipError_t launch_tile_steps(const D2Q9Args& a, int k, const void* fin, void* fout, void* sens,
                                    uint8_t* flags, double* partials, int first, unsigned long long* faults,
                                    hipStream_t st)
{
    using G = TileSteps<S, TX, TY, K>;
    if (k < 1 || k > K || !tile_takes(a.nx, a.ny, TX, TY, K)) return hipErrorInvalidValue;
    const int cells = (TX + 2 * (k - 1)) * (TY + 2 * (k - 1));
    const int threads = cells >= G::kThreads ? G::kThreads : (cells + kWave - 1) / kWave * kWave;
    const unsigned blocks = (unsigned)(((a.nx + TX - 1) / TX) * ((a.ny + TY - 1) / TY));
    if (a.x.mask) {
        // extension sensors: single steps of F32 and F64 states
        if constexpr (std::is_same<S, float>::value || std::is_same<S, double>::value) {
            if (k != 1) return hipErrorInvalidValue;
            using G1 = TileSteps<S, TX, TY, 1>;
            d2q9_tile_kernel<S, TX, TY, 1, true><<<dim3(blocks), dim3(G1::kThreads), 0, st>>>(
                a, 1, (const typename G::raw*)fin, (typename G::raw*)fout, (typename G::R*)sens, flags, partials,
                first, faults);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    d2q9_tile_kernel<S, TX, TY, K><<<dim3(blocks), dim3(threads), 0, st>>>(
        a, k, (const typename G::raw*)fin, (typename G::raw*)fout, (typename G::R*)sens, flags, partials, first,
        faults);
    return hipGetLastError();
}

template <typename S, int NR>
static hipError_t launch_band_steps(const D2Q9Args& a, int k, const void* fin, void* fout, void* sens,
                                    uint8_t* flags, double* partials, int first, unsigned long long* faults,
                                    hipStream_t st)
{
    using raw = typename Store<S>::raw;
    using R = typename Store<S>::real;
    if ((k != 1 && k != 3) || !band_fits(a.nx, a.ny, NR)) return hipErrorInvalidValue;
    const int n = band_tiles(a.nx, a.ny, NR);
    const dim3 grid((unsigned)((n + 63) / 64 * 64)), block(kBandWaves * kWave);
    // The non-temporal hint where rows are whole half lines only: partial
    // lines that leave the cache early are written twice (a step alone, plain /
    // hint: FP32 5000 x 4000 363 / 454 us, BF16 235 / 333; FP32 4016 x 3000 203 /
    // 196, 4096^2 266 / 255).
    const bool nt = a.nt_stores && (size_t)a.nx * sizeof(raw) % 64 == 0;
    const raw* in = (const raw*)fin;
    raw* out = (raw*)fout;
    R* sv = (R*)sens;
    if (a.x.mask) {
        // extension sensors: single steps of F32 and F64 states
        if constexpr (std::is_same<S, float>::value || std::is_same<S, double>::value) {
            if (k != 1) return hipErrorInvalidValue;
            if (nt)
                d2q9_band_kernel<S, 1, NR, true, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
            else
                d2q9_band_kernel<S, 1, NR, false, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (k == 3 && nt)
        d2q9_band_kernel<S, 3, NR, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
    else if (k == 3)
        d2q9_band_kernel<S, 3, NR, false><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
    else if (nt)
        d2q9_band_kernel<S, 1, NR, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
    else
        d2q9_band_kernel<S, 1, NR, false><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, first, n, faults);
    return hipGetLastError();
}

template <typename S>
static hipError_t launch_state(const D2Q9Args& a, int k, const void* fin, void* const* out, hipStream_t st)
{
    using raw = typename Store<S>::raw;
    const int n = band_tiles(a.nx, a.ny, 2);
    const dim3 grid((unsigned)((n + 63) / 64 * 64)), block(kBandWaves * kWave);
    if (k == 3)
        d2q9_band_state_kernel<S, 3><<<grid, block, 0, st>>>(a, (const raw*)fin, (raw*)out[0], (raw*)out[1],
                                                             (raw*)out[2], n);
    else
        d2q9_band_state_kernel<S, 1><<<grid, block, 0, st>>>(a, (const raw*)fin, (raw*)out[0], nullptr, nullptr, n);
    return hipGetLastError();
}

bool d2q9_band_fits(int nx, int ny) { return band_fits(nx, ny, 2); }

hipError_t launch_d2q9_state(int dtype, const D2Q9Args& a, int k, const void* fin, void* const* out, hipStream_t s)
{
    if ((k != 1 && k != 3) || !band_fits(a.nx, a.ny, 2)) return hipErrorInvalidValue;
    switch (dtype) {
    case 0: return launch_state<double>(a, k, fin, out, s);
    case 1: return launch_state<float>(a, k, fin, out, s);
    default: return hipErrorInvalidValue;
    }
}

// Tile forms (F(form, columns, rows, most steps)): the tile kernel's three,
// then the band kernel with two and three rows a wave.
#define LKS_TILE_FORMS(F) F(1, 8, 8, 7) F(2, 16, 16, 7) F(3, 32, 16, 5)
constexpr int kBandForm = 4, kTallForm = 5;

// The smallest tiles that one workgroup a CU can take (the fewest cells for
// the ring's share of work: at FP32 128^2 8 x 8 tiles 1.9, 16 x 16 2.2 us a step;
// at 256^2 16 x 16 2.6, 32 x 16 2.9, band 3.7; at 320^2 32 x 16 3.2, band 3.9; with
// more tiles than CUs 16 x 16 takes 4.4 there), then the band kernel (384^2: 4.0
// against 5.6), and on grids too narrow for it the largest tile that fits.  The
// band kernel takes three rows a wave (a smaller share of ring cells, but fewer
// and longer workgroups) from eight tiles a CU on: FP32 us a step with two /
// three rows 512^2 4.0 / 4.9, 1024^2 10.9 / 11.2, 2048^2 36.3 / 34.1, 4096^2 129.2 /
// 122.3, FP64 4096^2 321 / 310, BF16 131 / 125.  32 x 16 tiles of FP64 cells do not fit the LDS.
int d2q9_tile_of(int dtype, int nx, int ny)
{
    constexpr long long kCUs = 256;
#define LKS_TILE_FITS(V, TX, TY, K)                                                                         \
    if ((V < 3 || dtype != 0) && tile_takes(nx, ny, TX, TY, K) &&                                           \
        (long long)((nx + TX - 1) / TX) * ((ny + TY - 1) / TY) <= kCUs)                                     \
        return V;
    LKS_TILE_FORMS(LKS_TILE_FITS)
#undef LKS_TILE_FITS
    if (band_fits(nx, ny, 3) && band_tiles(nx, ny, 3) >= 8 * kCUs) return kTallForm;
    if (band_fits(nx, ny, 2)) return kBandForm;
    if (dtype != 0 && tile_takes(nx, ny, 32, 16, 5)) return 3;
    if (tile_takes(nx, ny, 16, 16, 7)) return 2;
    return tile_takes(nx, ny, 8, 8, 7) ? 1 : 0;
}

int d2q9_tile_steps(int tile)
{
    switch (tile) {
#define LKS_TILE_STEPS(V, TX, TY, K) case V: return K;
    LKS_TILE_FORMS(LKS_TILE_STEPS)
#undef LKS_TILE_STEPS
    case kBandForm:
    case kTallForm: return kBandK;
    default: return 0;
    }
}

int d2q9_tile_steps_upto(int tile, int n)
{
    const int most = d2q9_tile_steps(tile);
    if (n >= most) return most;
    return tile == kBandForm || tile == kTallForm ? 1 : (n - 1) / 2 * 2 + 1;      // n >= 1
}

int d2q9_tile_blocks(int tile, int nx, int ny)
{
    switch (tile) {
#define LKS_TILE_BLOCKS(V, TX, TY, K) case V: return ((nx + TX - 1) / TX) * ((ny + TY - 1) / TY);
    LKS_TILE_FORMS(LKS_TILE_BLOCKS)
#undef LKS_TILE_BLOCKS
    case kBandForm: return band_tiles(nx, ny, 2);
    case kTallForm: return band_tiles(nx, ny, 3);
    default: return 0;
    }
}

template <typename S>
static hipError_t launch_tile_form(const D2Q9Args& a, int k, const void* fin, void* fout, void* sens,
                                   uint8_t* flags, double* partials, int first, unsigned long long* faults,
                                   hipStream_t st)
{
    switch (a.tile) {
    case 1: return launch_tile_steps<S, 8, 8, 7>(a, k, fin, fout, sens, flags, partials, first, faults, st);
    case 2: return launch_tile_steps<S, 16, 16, 7>(a, k, fin, fout, sens, flags, partials, first, faults, st);
    case 3:
        if constexpr (sizeof(typename Store<S>::raw) <= 4)
            return launch_tile_steps<S, 32, 16, 5>(a, k, fin, fout, sens, flags, partials, first, faults, st);
        return hipErrorInvalidValue;
    case kBandForm: return launch_band_steps<S, 2>(a, k, fin, fout, sens, flags, partials, first, faults, st);
    case kTallForm: return launch_band_steps<S, 3>(a, k, fin, fout, sens, flags, partials, first, faults, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_d2q9_tile(int dtype, const D2Q9Args& a, int k, const void* fin, void* fout, void* sens,
                            uint8_t* flags, double* partials, int first, unsigned long long* faults, hipStream_t s)
{
    switch (dtype) {
    case 0: return launch_tile_form<double>(a, k, fin, fout, sens, flags, partials, first, faults, s);
    case 1: return launch_tile_form<float>(a, k, fin, fout, sens, flags, partials, first, faults, s);
    case 2: return launch_tile_form<bf16_t>(a, k, fin, fout, sens, flags, partials, first, faults, s);
    case 3: return launch_tile_form<f16_t>(a, k, fin, fout, sens, flags, partials, first, faults, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename S, int VEC>
static hipError_t launch_pass(int pass, const D2Q9Args& a, const void* fin, void* fout, void* sens,
                              uint8_t* flags, double* partials, unsigned long long* faults,
                              hipStream_t st)
{
    using raw = typename Store<S>::raw;
    using R = typename Store<S>::real;
    const raw* in = static_cast<const raw*>(fin);
    raw* out = static_cast<raw*>(fout);
    R* sv = static_cast<R*>(sens);
    const dim3 grid(a.g.nblocks), block(kBlock);
    switch (pass) {
    case kFused:
        if (a.x.mask) {
            // extension sensors: F32 and F64 storage, whose pieces always stage
            if constexpr (std::is_same<S, float>::value || std::is_same<S, double>::value) {
                if (!(LKS_D2Q9_LDS_STAGE && StageGeom<S, VEC>::ok)) return hipErrorInvalidValue;
                if (a.nt_stores)
                    d2q9_fused_lds<S, VEC, true, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
                else
                    d2q9_fused_lds<S, VEC, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
            } else {
                return hipErrorInvalidValue;
            }
        } else if (LKS_D2Q9_LDS_STAGE && StageGeom<S, VEC>::ok && a.nt_stores)
            d2q9_fused_lds<S, VEC, false, true><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        else if (LKS_D2Q9_LDS_STAGE && StageGeom<S, VEC>::ok)
            d2q9_fused_lds<S, VEC><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        else
            d2q9_kernel<S, VEC, kFused><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        break;
    case kStream:
        d2q9_kernel<S, VEC, kStream><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        break;
    case kSense:
        d2q9_kernel<S, VEC, kSense><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        break;
    case kCollide:
        d2q9_kernel<S, VEC, kCollide><<<grid, block, 0, st>>>(a, in, out, sv, flags, partials, faults);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename S, int VWIDE>
static hipError_t launch_vec(int pass, const D2Q9Args& a, const void* fin, void* fout, void* sens,
                             uint8_t* flags, double* partials, unsigned long long* faults,
                             hipStream_t st)
{
    switch (a.g.vec) {
    case 1: return launch_pass<S, 1>(pass, a, fin, fout, sens, flags, partials, faults, st);
    case 2: return launch_pass<S, 2>(pass, a, fin, fout, sens, flags, partials, faults, st);
    case 4:
        if constexpr (VWIDE >= 4) return launch_pass<S, 4>(pass, a, fin, fout, sens, flags, partials, faults, st);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_d2q9(int dtype, int pass, const D2Q9Args& a, const void* fin, void* fout,
                       void* sens, uint8_t* flags, double* partials, unsigned long long* faults,
                       hipStream_t s)
{
    switch (dtype) {
    case 0: return launch_vec<double, 2>(pass, a, fin, fout, sens, flags, partials, faults, s);
    case 1: return launch_vec<float, 4>(pass, a, fin, fout, sens, flags, partials, faults, s);
    case 2: return launch_vec<bf16_t, 4>(pass, a, fin, fout, sens, flags, partials, faults, s);
    case 3: return launch_vec<f16_t, 4>(pass, a, fin, fout, sens, flags, partials, faults, s);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// Equilibrium initialiser and moment readout (one thread per cell, FP64 math)
// ---------------------------------------------------------------------------
template <typename S>
__global__ __launch_bounds__(kBlock) void d2q9_init_kernel(long long n, PopLayout L, double rho0, const double* __restrict__ rho,
                                                      const double* __restrict__ ux,
                                                      const double* __restrict__ uy,
                                                      typename Store<S>::raw* __restrict__ pop)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= n) return;
    const double r = rho[c], u = ux[c], v = uy[c];
    const double usq15 = 1.5 * (u * u + v * v);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double cu = cx9(i) * u + cy9(i) * v;
        const double deq = w9<double>(i) * ((r - rho0) + r * (cu * (3.0 + 4.5 * cu) - usq15));
        pop[L.cell(i, c)] = Store<S>::from_real((typename Store<S>::real)deq);
    }
}

template <typename S>
__global__ __launch_bounds__(kBlock) void d2q9_moments_kernel(long long n, PopLayout L, double rho0,
                                                         const typename Store<S>::raw* __restrict__ pop,
                                                         double* __restrict__ rho, double* __restrict__ ux,
                                                         double* __restrict__ uy, double* __restrict__ T)
{
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= n) return;
    double drho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double d = (double)Store<S>::to_real(pop[L.cell(i, c)]);
        drho += d;
        jx += cx9(i) * d;
        jy += cy9(i) * d;
    }
    const double r = rho0 + drho;
    rho[c] = r;
    ux[c] = jx / r;
    uy[c] = jy / r;
    if (T) T[c] = 1.0 / 3.0;
}

hipError_t launch_d2q9_init(int dtype, long long n, const PopLayout& L, double rho0, const double* rho,
                            const double* ux, const double* uy, void* pop, hipStream_t s)
{
    const dim3 grid((unsigned)((n + kBlock - 1) / kBlock)), block(kBlock);
    switch (dtype) {
    case 0: d2q9_init_kernel<double><<<grid, block, 0, s>>>(n, L, rho0, rho, ux, uy, (double*)pop); break;
    case 1: d2q9_init_kernel<float><<<grid, block, 0, s>>>(n, L, rho0, rho, ux, uy, (float*)pop); break;
    case 2: d2q9_init_kernel<bf16_t><<<grid, block, 0, s>>>(n, L, rho0, rho, ux, uy, (uint16_t*)pop); break;
    case 3: d2q9_init_kernel<f16_t><<<grid, block, 0, s>>>(n, L, rho0, rho, ux, uy, (uint16_t*)pop); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_d2q9_moments(int dtype, long long n, const PopLayout& L, double rho0, const void* pop,
                               double* rho, double* ux, double* uy, double* T, hipStream_t s)
{
    const dim3 grid((unsigned)((n + kBlock - 1) / kBlock)), block(kBlock);
    switch (dtype) {
    case 0: d2q9_moments_kernel<double><<<grid, block, 0, s>>>(n, L, rho0, (const double*)pop, rho, ux, uy, T); break;
    case 1: d2q9_moments_kernel<float><<<grid, block, 0, s>>>(n, L, rho0, (const float*)pop, rho, ux, uy, T); break;
    case 2: d2q9_moments_kernel<bf16_t><<<grid, block, 0, s>>>(n, L, rho0, (const uint16_t*)pop, rho, ux, uy, T); break;
    case 3: d2q9_moments_kernel<f16_t><<<grid, block, 0, s>>>(n, L, rho0, (const uint16_t*)pop, rho, ux, uy, T); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

} // namespace lks
