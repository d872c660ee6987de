// The CG iteration of solves that fit on the chip (gfx950, wave64).
//
// A grid is cut into bricks of whole rows (rby rows x rbz planes), one
// workgroup each and all of them resident at once (a cooperative launch).  A
// workgroup keeps its brick's z = D^-1 r and x (FP32 + refinement: the
// correction d) in registers and its direction p in LDS from one iteration
// to the next, so an iteration moves only the bricks' faces and three sums:
//   p = z + beta p (own cells, and the rows and planes around the brick from
//   the neighbours' z), q = A p, p.A p                        -> exchange 1
//   x += alpha p, z -= alpha q / diag, r.z, r.r, faces of z   -> exchange 2
// This is the textbook order of the two-pass iteration.  It ends where the
// two-pass state machine would leave the loop (convergence, iteration cap,
// breakdown) or after `budget` iterations, with z, x and p back in the slot's
// vectors.
//
// What bounds it: the two exchanges, about 1.5 us each across the eight XCDs
// (a store that reaches memory, a load that sees it), and for bricks of many
// cells their LDS accesses and arithmetic.  Counted a cell and iteration: 20
// LDS and 123 vector instructions at 320 x 128 x 96 FP64 (30 cells a thread,
// the row formed twice; 16 and 106 where one density fills the grid), 23 and
// 187 at 101 x 77 x 59 FP32 (four cells); of the wave cycles 21 and 16 % issue
// vector instructions, 58 and 68 % wait.  A launch per iteration instead waits for memory plane after plane
// and streams 41 B a cell.  Measured per iteration of whole solves, launches
// against this: FP64 33^3 14.6 -> 5.9 us, 64^3 18.7 -> 7.4, 128^3 32 -> 15,
// 320 x 128 x 96 52 -> 32; FP32 33^3 14.5 -> 6.1, 64^3 18.0 -> 7.5, 128^3 33
// -> 12.5, 150 x 141 x 250 64 -> 33.
//
// Densities without classes and cut cells hold the face coefficients in
// registers beside z and x (FACES), 16 words a cell FP64, which bounds them
// to ten or twelve cells a thread.  Launches against this: densities FP64 110
// x 128 x 90 (twelve cells) 30.7 -> 16.1 us, 109 x 119 x 101 35 -> 17; FP32
// 125 x 125 x 150 42 -> 15, 150 x 141 x 133 46 -> 22; smaller ones 64^3 7.8,
// 96^3 11.3 (FP64), cut cells 64^3 8.2, 96^3 11.9.
//
// Exchange: a workgroup's sums go out as words of half a double beside a
// 32-bit tag, the number of the exchange, written and read with relaxed
// device-scope atomics (which reach the memory all XCDs share); a reader
// polls until every workgroup's words bear the tag, so no flag, fence or
// counter is needed.  The face values are written the same way before the
// sums (s_waitcnt between them), so whoever has seen the sums may read the
// faces.  All workgroups add the sums in the same order and so take the same
// decisions.  A word is rewritten only after an exchange that its readers
// have all passed.
//
// Polling is bounded.  Where not all workgroups come to run beside each other
// in that time (other work holds compute units of the device for 0.3 s) a
// workgroup that waits in vain sets SlotState::rfail and all of them end, the
// solve's later launches at once; the host then starts it again on the tile
// passes.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "device_common.h"
#include "pcg.h"
#include "resident_shapes.h"

namespace pcgmi {

namespace {

typedef unsigned long long u64;

template <typename T>
__device__ __forceinline__ T dev_load(const GLB T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void dev_store(GLB T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Lane i - d's value of v (0 where there is none) through the data-parallel
// path of the vector unit: a shuffle through LDS takes several times as long.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v)
{
    typedef int i2 __attribute__((ext_vector_type(2)));
    i2 h = __builtin_bit_cast(i2, v);
    h.x = __builtin_amdgcn_update_dpp(0, h.x, CTRL, ROWS, 0xf, false);
    h.y = __builtin_amdgcn_update_dpp(0, h.y, CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, h);
}

// Sum over the wave, in lane 63: within rows of 16 lanes (shifts by 1, 2, 4,
// 8), then from row to row.
__device__ __forceinline__ double wave_sum63(double v)
{
    v += dpp<0x111, 0xf>(v);
    v += dpp<0x112, 0xf>(v);
    v += dpp<0x114, 0xf>(v);
    v += dpp<0x118, 0xf>(v);
    v += dpp<0x142, 0xa>(v);
    v += dpp<0x143, 0xc>(v);
    return v;
}

// a / b by a refined reciprocal.  SCALED: b by its exponent first, and a by the
// same power of two (which is exact), since the sums of solves scaled near the
// ends of the number range (a source of 1e-150 with densities of 1e-9) have no
// reciprocal within it.
template <bool SCALED>
struct Divisor {
    double y;
    int e;
    __device__ __forceinline__ explicit Divisor(double b)
        : e(SCALED ? -__builtin_amdgcn_frexp_exp(b) : 0)
    {
        y = recip(SCALED ? __builtin_amdgcn_ldexp(b, e) : b);
    }
    __device__ __forceinline__ double under(double a) const
    {
        return (SCALED ? __builtin_amdgcn_ldexp(a, e) : a) * y;
    }
};

// Holds the compiler to the value in a register: what is derived from it in
// the iteration loop (coefficient addresses, lane masks) is formed there
// again instead of being kept in registers of its own, several a cell.
template <typename V>
__device__ __forceinline__ void keep_here(V &v) { asm volatile("" : "+v"(v)); }

constexpr int kWaves = kResThreads / 64;

// The eight waves' values of v at red, added pairwise.
__device__ __forceinline__ double add_waves(const double *red)
{
    static_assert(kWaves == 8, "eight waves");
    return ((red[0] + red[1]) + (red[2] + red[3])) + ((red[4] + red[5]) + (red[6] + red[7]));
}

// Sum NV values over the workgroups of a solve: every thread brings its part
// and leaves with the total, added in an order fixed by the bricks.  The
// workgroup's earlier stores have reached memory before its sums go out.
// False when a workgroup did not answer within `polls` looks.
template <int NV>
__device__ __forceinline__ bool all_sum(double (&v)[NV], GLB u64 *area, int G, int g, uint32_t tag,
                                        int polls, double (*red)[4 * kWaves], int *fail)
{
    const int t = (int)threadIdx.x, w = t >> 6, lane = t & 63;
    // calls alternate the halves: a wave may still read the last call's
    const int r0 = (tag & 1) ? 2 * kWaves : 0;
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] = wave_sum63(v[m]);
    if (lane == 63) {
#pragma unroll
        for (int m = 0; m < NV; ++m) red[m][r0 + w] = v[m];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] = add_waves(red[m] + r0);
    if (G == 1) return true;
    if (t < 2 * NV) {
        double mine = v[0];
#pragma unroll
        for (int m = 1; m < NV; ++m) mine = (t >> 1) == m ? v[m] : mine;
        const u64 bits = (u64)__double_as_longlong(mine);
        const u64 half = (t & 1) ? bits >> 32 : bits & 0xffffffffull;
        dev_store(area + (size_t)g * 2 * NV + t, ((u64)tag << 32) | half);
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] = 0.0;
    bool ok = true;
    // value m of brick b: pair b NV + m of words
    for (int e = t; e < G * NV; e += kResThreads) {
        const GLB u64 *src = area + 2 * (size_t)e;
        u64 lo = 0, hi = 0;
        for (int n = 0;; ++n) {
            if (n >= polls) { ok = false; break; }
            lo = dev_load(src);
            hi = dev_load(src + 1);
            if ((uint32_t)(lo >> 32) == tag && (uint32_t)(hi >> 32) == tag) break;
        }
        const double d = __longlong_as_double((long long)((lo & 0xffffffffull) | (hi << 32)));
#pragma unroll
        for (int m = 0; m < NV; ++m)
            if (e % NV == m) v[m] += d;
    }
    if (!ok) *fail = 1;
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] = wave_sum63(v[m]);
    if (lane == 63) {
#pragma unroll
        for (int m = 0; m < NV; ++m) red[m][r0 + kWaves + w] = v[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NV; ++m) v[m] = add_waves(red[m] + r0 + kWaves);
    return *fail == 0;
}

// The operator row of one cell of a column, and its faces' share of p.A p.
template <typename T>
struct Row {
    T q, dg, s;
};

template <typename T>
struct Betas {
    T xm, xp, ym, yp, zm, zp;
    bool wx, wy, wz;   // p = 0 walls above the cell
};

template <typename T, bool SUM>
__device__ __forceinline__ Row<T> row_of(const Betas<T> &b, T pc, T xm, T xp, T ym, T yp, T zm, T zp)
{
    const T dxm = pc - xm, dxp = pc - xp, dym = pc - ym, dyp = pc - yp, dzm = pc - zm, dzp = pc - zp;
    const T txm = b.xm * dxm, txp = b.xp * dxp, tym = b.ym * dym, typ = b.yp * dyp,
            tzm = b.zm * dzm, tzp = b.zp * dzp;
    Row<T> r;
    r.q = ((txm + txp) + (tym + typ)) + (tzm + tzp);
    r.dg = ((b.xm + b.xp) + (b.ym + b.yp)) + (b.zm + b.zp);
    r.s = T(0);
    if (SUM) {
        // each face from its upper cell, and the p = 0 walls above a cell
        r.s = (txm * dxm + tym * dym) + tzm * dzm;
        r.s += b.wx ? txp * dxp : T(0);
        r.s += b.wy ? typ * dyp : T(0);
        r.s += b.wz ? tzp * dzp : T(0);
    }
    return r;
}

// From a cell's class nibbles (own, x-, x+, y-, y+, z-, z+), or one
// coefficient for the whole wave where every cell of the column and its
// neighbours are of one class (UNI; the x walls of a row then scale it by 0
// or 2).  bzm: the low z coefficient, replaced by the high one.
template <typename T, bool UNI, bool SUM>
__device__ __forceinline__ Row<T> cell_row(uint32_t code, const T *tab, T bu, T fxm, T fxp, T &bzm,
                                           T pc, T xm, T xp, T ym, T yp, T zm, T zp)
{
    Betas<T> b;
    if (UNI) {
        b = { bu * fxm, bu * fxp, bu, bu, bu, bu, fxp == T(2), false, false };
    } else {
        const T *row = tab + (code & 15u) * kClasses;
        const uint32_t kx = (code >> 8) & 15u, ky = (code >> 16) & 15u, kz = (code >> 24) & 15u;
        b = { row[(code >> 4) & 15u], row[kx], row[(code >> 12) & 15u], row[ky], bzm, row[kz],
              kx == (uint32_t)kClsWallD, ky == (uint32_t)kClsWallD, kz == (uint32_t)kClsWallD };
    }
    bzm = b.zp;
    return row_of<T, SUM>(b, pc, xm, xp, ym, yp, zm, zp);
}

}  // namespace

// T: double (FP64 solves) or float (inner solves of FP32 + refinement); NC
// columns of NZ cells a thread; KEEP: q and the diagonal stay in registers
// between the two halves of an iteration, else they are formed again (the
// largest bricks); FACES: the face coefficients are formed once, from the
// densities and with the area fractions where a solve has them, and stay in
// registers (five a cell; z faces are shared by a column's cells), instead of
// being looked up by class.
template <typename T, int NC, int NZ, bool KEEP, bool FACES>
__global__ void __launch_bounds__(kResThreads)
k_resident(const Slot *__restrict__ slots, int s0, int s1, int budget, int polls)
{
    constexpr bool F64 = std::is_same<T, double>::value;
    constexpr int NH = res_halo(NC * NZ);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    T *Lp = reinterpret_cast<T *>(smem);
    __shared__ T tab[kClasses * kClasses];
    __shared__ double red[2][4 * kWaves];
    __shared__ int s_fail;
    const int t = (int)threadIdx.x;
    int s = s0;
    while (s + 1 < s1 && slots[s + 1].rblk <= (int)blockIdx.x) ++s;
    const Slot &S = slots[s];
    const int g = (int)blockIdx.x - S.rblk, G = S.rnby * S.rnbz;
    if (!S.resident || g >= G) return;
    SlotState &st = *S.st;
    if (st.rfail || st.phase != (F64 ? K1_CG_A : K1_IR_A)) return;

    const int nx = S.nx, ny = S.ny, nz = S.nz, P = nx * ny, bm = S.bcmask;
    const bool px = (S.permask & 1) && nx > 1, py = (S.permask & 2) && ny > 1;
    const int gy = g % S.rnby, gz = g / S.rnby, j0 = gy * S.rby, k0 = gz * NZ;
    const int by = min(S.rby, ny - j0), bz = min(NZ, nz - k0), C = nx * by;
    const bool ylo = j0 > 0 || py, yhi = j0 + by < ny || py, zlo = k0 > 0, zhi = k0 + bz < nz;
    const int RS = nx + 2, PS = (S.rby + 2) * RS;
    GLB T *zg = gp((T *)S.z), *pg = gp((T *)dir_buf(S, st.pbuf));
    GLB T *xg = gp(F64 ? (T *)S.x : (T *)S.d32);
    const GLB uint8_t *gcls = gp(S.cls);

    for (int i = t; i < NZ * PS; i += kResThreads) Lp[i] = T(0);
    for (int i = t; i < kClasses * kClasses; i += kResThreads)
        tab[i] = F64 ? (T)gp(S.tab64)[i] : (T)gp(S.tab32)[i];
    if (t == 0) s_fail = 0;
    __syncthreads();

    const bool first = st.first != 0;
    const double tol2 = st.tol2, goal2 = F64 ? 0.0 : st.inner_goal2 * st.rr0_inner;
    const int maxit = st.maxit, inner_max = st.inner_maxit;
    int iter = st.iter, inner = st.inner_iter;
    uint32_t tag = st.repoch;
    double rz = st.rz, rr = st.rr, pap = st.pap, alpha = st.alpha;
    double beta = first ? 0.0 : st.beta;
    GLB u64 *area1 = gp(S.rsync), *area2 = area1 + 2 * (size_t)G;

    T z[NC][NZ], x[NC][NZ], pl[NC], ph[NC], q[KEEP ? NC : 1][KEEP ? NZ : 1],
        dg[KEEP && !FACES ? NC : 1][KEEP && !FACES ? NZ : 1];
    uint32_t code[FACES ? 1 : NC][FACES ? 1 : NZ];
    constexpr int FC = FACES ? NC : 1, FZ = FACES ? NZ : 1;
    T fxl[FC][FZ], fxh[FC][FZ], fyl[FC][FZ], fyh[FC][FZ], fz[FC][FZ + 1];
    uint32_t wflag = 0;   // FACES, 2 bits a column: p = 0 walls above it in x, y
    int off[NC], gi[NC];  // LDS and grid cell of the column's first plane
    uint32_t cflag = 0;   // 4 bits a column: active, i == 0, i == nx - 1, on a y face
    uint32_t uni = 0;     // columns of one class throughout the wave
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int col = t + c * kResThreads;
        const bool act = col < C;
        const int jl = act ? col / nx : 0, i = act ? col - jl * nx : 0, j = j0 + jl;
        gi[c] = k0 * P + j * nx + i;
        off[c] = (jl + 1) * RS + i + 1;
        cflag |= ((act ? 1u : 0u) | (i == 0 ? 2u : 0u) | (i == nx - 1 ? 4u : 0u) |
                  ((jl == 0 && ylo) || (jl == by - 1 && yhi) ? 8u : 0u))
                 << (4 * c);
        const int oxm = i > 0 ? -1 : (px ? nx - 1 : 0), oxp = i < nx - 1 ? 1 : (px ? 1 - nx : 0);
        const int oym = j > 0 ? -nx : (py ? (ny - 1) * nx : 0);
        const int oyp = j < ny - 1 ? nx : (py ? -(ny - 1) * nx : 0);
        bool same = act && bz == NZ;
        uint32_t kc0 = 0;
        if constexpr (FACES) {
            // densities of solids are +inf: no flow through their faces; the
            // wall stands for density 0 (p = 0 on its face) or for a solid
            const GLB T *rho = gp((const T *)(F64 ? (const void *)S.rho64 : (const void *)S.rho32));
            auto wall = [&](int w) { return (bm >> w) & 1 ? T(0) : (T)INFINITY; };
            wflag |= ((act && i == nx - 1 && !px && (bm & 2) ? 1u : 0u) |
                      (act && j == ny - 1 && !py && (bm & 8) ? 2u : 0u)) << (2 * c);
            const int j1 = py && j == ny - 1 ? 0 : j + 1, i1 = px && i == nx - 1 ? 0 : i + 1;
#pragma unroll
            for (int k = 0; k < NZ; ++k) {
                const bool in = act && k < bz;
                const int m = in ? gi[c] + k * P : 0, kk = k0 + k;
                T b[6] = { T(0), T(0), T(0), T(0), T(0), T(0) };
                if (in) {
                    const T rc = rho[m];
                    b[0] = fb(rc + (oxm ? rho[m + oxm] : wall(0)));
                    b[1] = fb(rc + (oxp ? rho[m + oxp] : wall(1)));
                    b[2] = fb(rc + (oym ? rho[m + oym] : wall(2)));
                    b[3] = fb(rc + (oyp ? rho[m + oyp] : wall(3)));
                    b[4] = fb(rc + (kk > 0 ? rho[m - P] : wall(4)));
                    b[5] = fb(rc + (kk < nz - 1 ? rho[m + P] : wall(5)));
                    if (S.ax) {
                        const GLB double *ax = gp(S.ax) + ((int64_t)kk * ny + j) * (nx + 1);
                        const GLB double *ay = gp(S.ay) + (int64_t)kk * (ny + 1) * nx + i;
                        const GLB double *az = gp(S.az) + m;
                        b[0] *= (T)ax[i];
                        b[1] *= (T)ax[i1];
                        b[2] *= (T)ay[(int64_t)j * nx];
                        b[3] *= (T)ay[(int64_t)j1 * nx];
                        b[4] *= (T)az[0];
                        b[5] *= (T)az[P];
                    }
                }
                fxl[c][k] = b[0];
                fxh[c][k] = b[1];
                fyl[c][k] = b[2];
                fyh[c][k] = b[3];
                if (k == 0) fz[c][0] = b[4];
                // (above the brick's last plane: that cell's high face stays)
                fz[c][k + 1] = b[5];
            }
        }
#pragma unroll
        for (int k = 0; k < NZ; ++k) {
            const bool in = act && k < bz;
            const int m = in ? gi[c] + k * P : 0;
            z[c][k] = x[c][k] = T(0);
            if (in) {
                z[c][k] = zg[m];
                x[c][k] = xg[m];
                if (!first) Lp[off[c] + k * PS] = pg[m];
            }
            if constexpr (FACES) continue;
            uint32_t cd = 0x0fffffffu;
            if (in) {
                const int kk = k0 + k;
                const uint32_t kc = gcls[m];
                auto key = [&](bool there, int o, int wall) -> uint32_t {
                    if (there) return gcls[m + o];
                    return (uint32_t)((bm >> wall) & 1 ? kClsWallD : kClsSolid);
                };
                const uint32_t w[6] = { key(oxm != 0, oxm, 0), key(oxp != 0, oxp, 1),
                                        key(oym != 0, oym, 2), key(oyp != 0, oyp, 3),
                                        key(kk > 0, -P, 4),    key(kk < nz - 1, P, 5) };
                if (kc != (uint32_t)kClsSolid)
                    cd = kc | w[0] << 4 | w[1] << 8 | w[2] << 12 | w[3] << 16 | w[4] << 20 | w[5] << 24;
            }
            code[FACES ? 0 : c][FACES ? 0 : k] = cd;
            // one class throughout, the x walls of the row aside
            if (k == 0) kc0 = __builtin_amdgcn_readfirstlane(cd) & 15u;
            uint32_t want = kc0 * 0x1111111u, have = cd;
            if (i == 0 && !px) { want &= ~0xf0u; have &= ~0xf0u; }
            if (i == nx - 1 && !px) { want &= ~0xf00u; have &= ~0xf00u; }
            same = same && kc0 < (uint32_t)kMaxFluidClasses && have == want;
        }
        if (!FACES && __all(same)) uni |= 1u << c;
        // p of the planes below and above the brick
        pl[c] = ph[c] = T(0);
        if (act && !first && zlo) pl[c] = pg[gi[c] - P];
        if (act && !first && zhi) ph[c] = pg[gi[c] + NZ * P];
    }
    // The rows beside the brick: value e of this thread, m = t + e kResThreads
    // of them all, belongs to row m / nx (below and above the brick in turn,
    // plane by plane), is grid cell hg and lives at LDS cell hl (-1: none).
    // m / nx is exact from the rounded-up reciprocal for m, nx < 2^12.
    const int nhalo = 2 * bz * nx;
    const uint32_t inv_nx = ((1u << 24) + (uint32_t)nx - 1u) / (uint32_t)nx;
    uint32_t tk = (uint32_t)t;
    const int glo = j0 > 0 ? j0 - 1 : ny - 1, ghi = j0 + by < ny ? j0 + by : 0;
    auto beside = [&](int e, int &hl, int &hg) __attribute__((always_inline)) {
        const uint32_t m = tk + (uint32_t)(e * kResThreads);
        const uint32_t r = nx > 1 ? __umulhi(m << 8, inv_nx) : m, i = m - r * (uint32_t)nx;
        const bool up = r & 1u;
        const int k = (int)(r >> 1);
        hl = k < bz && (up ? yhi : ylo) ? k * PS + (up ? by + 1 : 0) * RS + (int)i + 1 : -1;
        hg = (k0 + k) * P + (up ? ghi : glo) * nx + (int)i;
    };
#pragma unroll
    for (int e = 0; e < NH; ++e) {
        int hl, hg;
        beside(e, hl, hg);
        if (e * kResThreads < nhalo && hl >= 0 && !first) Lp[hl] = pg[hg];
    }
    int end = 0;   // 0: budget spent, 1: converged or capped, 2: breakdown, 3: vanished direction

    for (int n = 0;; ++n) {
        if (n == budget) break;
        // p = z + beta p, of the rows and planes around the brick too: their
        // z is in flight during the own cells' update
        const T tb = (T)beta;
        T zl[NC], zh[NC], hz[NH];
        keep_here(cflag);
        keep_here(tk);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            keep_here(gi[c]);
            const bool act = (cflag >> (4 * c)) & 1u;
            zl[c] = zh[c] = T(0);
            if (zlo && act) zl[c] = dev_load(zg + gi[c] - P);
            if (zhi && act) zh[c] = dev_load(zg + gi[c] + NZ * P);
        }
#pragma unroll
        for (int e = 0; e < NH; ++e) {
            hz[e] = T(0);
            if (e * kResThreads < nhalo) {
                int hl, hg;
                beside(e, hl, hg);
                if (hl >= 0) hz[e] = dev_load(zg + hg);
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint32_t f = cflag >> (4 * c);
            keep_here(off[c]);
            if (f & 1u) {
#pragma unroll
                for (int k = 0; k < NZ; ++k) {
                    T *a = Lp + off[c] + k * PS;
                    const T pn = z[c][k] + tb * *a;
                    *a = pn;
                    if (px && (f & 2u)) a[nx] = pn;
                    if (px && (f & 4u)) a[-nx] = pn;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            pl[c] = zl[c] + tb * pl[c];
            ph[c] = zh[c] + tb * ph[c];
        }
        keep_here(tk);
#pragma unroll
        for (int e = 0; e < NH; ++e)
            if (e * kResThreads < nhalo) {
                int hl, hg;
                beside(e, hl, hg);
                if (hl >= 0) Lp[hl] = hz[e] + tb * Lp[hl];
            }
        __syncthreads();

        // q = A p and p.A p
        double sum = 0.0;
        auto column = [&](auto U, auto SUM, int c, auto &&each) __attribute__((always_inline)) {
            constexpr bool kU = decltype(U)::value, kS = decltype(SUM)::value;
            keep_here(off[c]);
            keep_here(cflag);
            const T *a = Lp + off[c];
            const uint32_t f = cflag >> (4 * c);
            T bu = T(0), fxm = T(1), fxp = T(1);
            if (kU) {
                bu = tab[(__builtin_amdgcn_readfirstlane(code[c][0]) & 15u) * (kClasses + 1)];
                if (!px && (f & 2u)) fxm = bm & 1 ? T(2) : T(0);
                if (!px && (f & 4u)) fxp = bm & 2 ? T(2) : T(0);
            }
            T zm = pl[c], pc = a[0];
            T bzm = kU ? bu : tab[(code[c][0] & 15u) * kClasses + ((code[c][0] >> 20) & 15u)];
#pragma unroll
            for (int k = 0; k < NZ; ++k) {
                const T *b = a + k * PS;
                keep_here(code[c][k]);
                const T zp = k + 1 < NZ ? b[PS] : ph[c];
                const Row<T> r = cell_row<T, kU, kS>(code[c][k], tab, bu, fxm, fxp, bzm, pc, b[-1],
                                                     b[1], b[-RS], b[RS], zm, zp);
                each(c, k, r, pc);
                // above the grid's last plane there is no cell to share a face with
                if (!kU) bzm = k + 1 < bz ? bzm : T(0);
                zm = pc;
                pc = zp;
            }
        };
        // the same with the coefficients of FACES
        auto column_faces = [&](auto SUM, int c, auto &&each) __attribute__((always_inline)) {
            constexpr bool kS = decltype(SUM)::value;
            keep_here(off[c]);
            keep_here(wflag);
            const T *a = Lp + off[c];
            const uint32_t f = wflag >> (2 * c);
            T zm = pl[c], pc = a[0];
#pragma unroll
            for (int k = 0; k < NZ; ++k) {
                const T *b = a + k * PS;
                const T zp = k + 1 < NZ ? b[PS] : ph[c];
                keep_here(fxl[c][k]);
                keep_here(fyl[c][k]);
                keep_here(fz[c][k]);
                // planes past the grid's last one hold no cells
                const T bzm = k < bz ? fz[c][k] : T(0);
                const Betas<T> bt = { fxl[c][k], fxh[c][k], fyl[c][k], fyh[c][k], bzm, fz[c][k + 1],
                                      (f & 1u) != 0, (f & 2u) != 0,
                                      k0 + k == nz - 1 && (bm & 32) };
                each(c, k, row_of<T, kS>(bt, pc, b[-1], b[1], b[-RS], b[RS], zm, zp), pc);
                zm = pc;
                pc = zp;
            }
        };
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
        auto first_half = [&](int c, int k, const Row<T> &r, T) __attribute__((always_inline)) {
            sum += (double)r.s;
            if constexpr (KEEP) q[c][k] = r.q;
            // (formed here: not its products kept for later)
            if constexpr (KEEP && FACES) keep_here(q[c][k]);
            if constexpr (KEEP && !FACES) dg[c][k] = r.dg;
        };
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (FACES) column_faces(Yes{}, c, first_half);
            else if ((uni >> c) & 1u) column(Yes{}, Yes{}, c, first_half);
            else column(No{}, Yes{}, c, first_half);
        }
        double v1[1] = { sum };
        if (!all_sum<1>(v1, area1, G, g, ++tag, polls, red, &s_fail)) break;
        pap = v1[0];
        if (!isfinite(pap) || !(pap > 0.0)) { end = (F64 || !isfinite(pap)) ? 2 : 3; break; }
        alpha = Divisor<F64>(pap).under(rz);

        // x += alpha p, z -= alpha q / diag, the faces of z, r.z and r.r
        const T ta = (T)alpha;
        keep_here(cflag);
        const Divisor<F64> by_rz(rz);   // ready before the sums are
        double v2[2] = { 0.0, 0.0 };
        auto second_half = [&](int c, int k, const Row<T> &r, T pc) __attribute__((always_inline)) {
            const T inv = r.dg > T(0) ? recip(r.dg) : T(0);   // hull rows keep z = 0
            const T zn = z[c][k] - ta * r.q * inv;
            z[c][k] = zn;
            x[c][k] = fma(ta, pc, x[c][k]);
            const double res = (double)r.dg * (double)zn;
            v2[0] += res * (double)zn;
            v2[1] += res * res;
            // the faces the neighbours wait for
            const uint32_t f = cflag >> (4 * c);
            if ((f & 1u) && k < bz &&
                ((f & 8u) || (k == 0 && zlo) || (k == NZ - 1 && zhi)))
                dev_store(zg + gi[c] + k * P, zn);
        };
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            keep_here(off[c]);
            keep_here(gi[c]);
            if constexpr (KEEP) {
#pragma unroll
                for (int k = 0; k < NZ; ++k) {
                    T d;
                    if constexpr (FACES) {
                        keep_here(fxl[c][k]);
                        keep_here(fyl[c][k]);
                        keep_here(fz[c][k]);
                        d = ((fxl[c][k] + fxh[c][k]) + (fyl[c][k] + fyh[c][k])) +
                            ((k < bz ? fz[c][k] : T(0)) + fz[c][k + 1]);
                    } else {
                        d = dg[c][k];
                    }
                    second_half(c, k, Row<T>{ q[c][k], d, T(0) }, Lp[off[c] + k * PS]);
                }
            } else {
                if constexpr (FACES) column_faces(No{}, c, second_half);
                else if ((uni >> c) & 1u) column(Yes{}, No{}, c, second_half);
                else column(No{}, No{}, c, second_half);
            }
        }
        if (!all_sum<2>(v2, area2, G, g, ++tag, polls, red, &s_fail)) break;
        beta = by_rz.under(v2[0]);
        rz = v2[0];
        rr = v2[1];
        ++iter;
        ++inner;
        if (!isfinite(rr) || (F64 && !isfinite(rz))) { end = 2; break; }
        if (F64 ? (rr <= tol2 || iter >= maxit)
                : (rr <= goal2 || inner >= inner_max || iter >= maxit)) { end = 1; break; }
    }
    __syncthreads();
    if (s_fail) {
        if (t == 0) dev_store(gp(&st.rfail), 1);
        return;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if ((cflag >> (4 * c)) & 1u) {
#pragma unroll
            for (int k = 0; k < NZ; ++k)
                if (k < bz) {
                    const int m = gi[c] + k * P;
                    zg[m] = z[c][k];
                    xg[m] = x[c][k];
                    pg[m] = Lp[off[c] + k * PS];
                }
        }
    }
    if (g == 0 && t == 0) {
        st.rz = rz;
        st.rr = rr;
        st.pap = pap;
        st.alpha = alpha;
        st.beta = beta;
        st.iter = iter;
        st.inner_iter = inner;
        st.first = 0;
        st.repoch = tag;
        if (end == 2) {
            st.status = PCG_EBREAKDOWN;
            st.phase = PH_DONE;
        } else if (F64) {
            if (end == 1) st.phase = K1_CHECK64;
        } else if (end) {
            // refine (a vanished direction too)
            st.scale = pow2_scale(sqrt(st.rr_true * st.inner_tol2));
            st.phase = K1_IR_RESID;
        }
    }
}

namespace {
struct Entry {
    ResidentShape shape;
    const void *fn;
};
#define PCG_ENTRY64(c, p, keep, faces, batch) \
    { { c, p, keep, faces, batch }, (const void *)k_resident<double, c, p, keep, faces> },
#define PCG_ENTRY32(c, p, keep, faces, batch) \
    { { c, p, keep, faces, batch }, (const void *)k_resident<float, c, p, keep, faces> },
const Entry kF64[] = { PCG_RESIDENT_FP64(PCG_ENTRY64) };
const Entry kF32[] = { PCG_RESIDENT_FP32(PCG_ENTRY32) };
}  // namespace

int resident_shapes(int family, ResidentShape *out, int cap)
{
    const Entry *t = family == PCG_PREC_FP64 ? kF64 : kF32;
    const int n = family == PCG_PREC_FP64 ? (int)(sizeof(kF64) / sizeof(Entry))
                                          : (int)(sizeof(kF32) / sizeof(Entry));
    for (int i = 0; i < n && i < cap; ++i) out[i] = t[i].shape;
    return n;
}

// Lets a shape's workgroups take up to kResLds bytes of LDS.  The attribute
// belongs to the process, so every caller sets the same value: one thread's
// launch never meets a smaller one that another has set for its own grid.
static hipError_t resident_fn(int family, int shape, const void **fn)
{
    *fn = (family == PCG_PREC_FP64 ? kF64 : kF32)[shape].fn;
    return hipFuncSetAttribute(*fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
}

// Workgroups of a shape that a CU holds at once with lds bytes each.
hipError_t resident_occupancy(int family, int shape, unsigned lds, int *wgs)
{
    const void *fn = nullptr;
    const hipError_t e = resident_fn(family, shape, &fn);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(wgs, fn, kResThreads, lds);
}

// One launch of the resident kernel of shape `shape` over slots [s0, s1) of
// the table: `blocks` workgroups, all resident at once, `lds` bytes each; at
// most `budget` iterations, and `polls` looks at a word before an exchange
// counts as timed out.
hipError_t launch_resident(int family, int shape, int blocks, unsigned lds, const Slot *slots,
                           int s0, int s1, int budget, int polls, hipStream_t s)
{
    const void *fn = nullptr;
    const hipError_t e = resident_fn(family, shape, &fn);
    if (e != hipSuccess) return e;
    void *args[] = { (void *)&slots, (void *)&s0, (void *)&s1, (void *)&budget, (void *)&polls };
    return hipLaunchCooperativeKernel(fn, dim3((unsigned)blocks), dim3(kResThreads), args, lds, s);
}

}  // namespace pcgmi
