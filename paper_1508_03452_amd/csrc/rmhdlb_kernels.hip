// rmhdlb_kernels.hip -- gfx950 kernels of the resistive relativistic MHD
// lattice Boltzmann step (arXiv:1508.03452, Sec. III).
//
// Layout in HBM: chunks of 64 cells (x fastest), each holding every array of
// its cells: the distributions F[0..18], G[0..18], h*[0..24] of storage type
// TS as (f_i, g_i) pairs (FP64), as quads of opposite directions (FP32) or as
// records of two such quads (FP16), then E_prev of type TE (TS, or FP32 when
// TS is FP16); the layouts are described in rmhdlb_device.h.  Two buffers, read
// one and write the other.  The stored state is post-collision.  On the FP32
// and FP16 storage paths F and G are stored as deviations from w_i E_ref and
// w'_i N_ref (references from the initial fields) and the step runs in FP32
// arithmetic, with the recovery and the Ohm solve in FP64.
#include <hip/hip_cooperative_groups.h>

#include "rmhdlb_device.h"
#include "rmhdlb_internal.h"
#include "rmhdlb_mlp.h"

#ifndef RMHDLB_FORM
#error "compile once per storage form with -DRMHDLB_FORM=64, 32 and 16"
#endif

namespace rmhd {

constexpr int TX = 64, TY = 4, TPB = TX * TY;

template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
template <typename T>
using vec4 = T __attribute__((ext_vector_type(4)));

// The value of type T at byte offset o of a state buffer, as V.
template <typename V, typename T>
__device__ __forceinline__ V ldv(const char* __restrict__ s, int64_t o) {
    return static_cast<V>(*reinterpret_cast<const T*>(s + o));
}
template <typename T>
__device__ __forceinline__ double ld(const char* __restrict__ s, int64_t o) {
    return ldv<double, T>(s, o);
}

// Loads of values that no other cell of the step reads (each streamed h* is
// pulled by exactly one cell): the non-temporal hint keeps them from
// evicting the stencil lines that the neighbours' loads will hit (256x256x256,
// ms per step without / with: FP64 4.74 / 4.69, FP32 2.40 / 2.38, FP16 1.677 /
// 1.663).
template <typename V, typename T>
__device__ __forceinline__ V ldv_once(const char* __restrict__ s, int64_t o) {
    return static_cast<V>(__builtin_nontemporal_load(reinterpret_cast<const T*>(s + o)));
}

template <typename V, typename T>
__device__ __forceinline__ vec2<V> ldv2(const char* __restrict__ s, int64_t o) {
    const vec2<T> v = *reinterpret_cast<const vec2<T>*>(s + o);
    vec2<V> r;
    r.x = static_cast<V>(v.x);
    r.y = static_cast<V>(v.y);
    return r;
}

template <typename V, typename T>
__device__ __forceinline__ vec4<V> ldv4(const char* __restrict__ s, int64_t o) {
    const vec4<T> v = *reinterpret_cast<const vec4<T>*>(s + o);
    vec4<V> r;
    r.x = static_cast<V>(v.x);
    r.y = static_cast<V>(v.y);
    r.z = static_cast<V>(v.z);
    r.w = static_cast<V>(v.w);
    return r;
}

// Stores of the next state are never read again in this step: the
// non-temporal hint keeps them from evicting the stencil lines from L2.
template <bool NT, typename T>
__device__ __forceinline__ void put_raw(char* __restrict__ d, int64_t o, T v) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, reinterpret_cast<T*>(d + o));
    else
        *reinterpret_cast<T*>(d + o) = v;
}
template <bool NT, typename T, typename V>
__device__ __forceinline__ void st(char* __restrict__ d, int64_t o, V v) {
    put_raw<NT, T>(d, o, static_cast<T>(v));
}
template <bool NT, typename T, typename V>
__device__ __forceinline__ void st2(char* __restrict__ d, int64_t o, V f, V g) {
    vec2<T> v;
    v.x = static_cast<T>(f);
    v.y = static_cast<T>(g);
    put_raw<NT>(d, o, v);
}
template <bool NT, typename T, typename V>
__device__ __forceinline__ void st4(char* __restrict__ d, int64_t o, const vec4<V>& q) {
    vec4<T> v;
    v.x = static_cast<T>(q.x);
    v.y = static_cast<T>(q.y);
    v.z = static_cast<T>(q.z);
    v.w = static_cast<T>(q.w);
    put_raw<NT>(d, o, v);
}

// FP64 storage uses the pair layout (two lanes per cell), FP32 the quad and
// FP16 the double-quad layout (one lane per cell; see rmhdlb_device.h).
template <typename TS>
constexpr bool quad_layout() {  // one lane per cell
    return sizeof(TS) != 8;
}
template <typename TS>
constexpr bool dquad_layout() {
    return sizeof(TS) == 2;
}
// Byte offsets of single values at position p, for the kernels that read or
// write them one by one: the f-g record of direction i (quad: of its slot's half of the record), ...
template <typename TS>
__host__ __device__ constexpr int rec_off(int i) {  // ... within the chunk, without the lane
    if (dquad_layout<TS>())
        return CHUNK * 16 * dquad_rec(quad_slot(i)) + 2 * (dquad_off(quad_slot(i)) + quad_pos(i));
    if (quad_layout<TS>()) return CHUNK * 16 * quad_slot(i) + 4 * quad_pos(i);
    return CHUNK * 16 * i;
}
template <typename TS>
__device__ __forceinline__ int64_t f_at(const Consts& K, int i, int p) {
    return lane_off<16>(K, p) + rec_off<TS>(i);
}
template <typename TS>
__device__ __forceinline__ int64_t g_at(const Consts& K, int i, int p) {
    return f_at<TS>(K, i, p) + (int)sizeof(TS);
}
template <typename TS>
__device__ __forceinline__ int64_t h_at(const Consts& K, int k, int p) {
    if constexpr (quad_layout<TS>()) {
        if (k == QH) return f_at<TS>(K, 0, p) + 2 * (int)sizeof(TS);  // third value of the rest quad
        return lane_off<Lay<TS>::HREC>(K, p) + Lay<TS>::H + CHUNK * Lay<TS>::HREC * (k / 2) +
               (k & 1) * (int)sizeof(TS);
    } else {
        return lane_off<8>(K, p) + Lay<TS>::H + CHUNK * 8 * k;
    }
}
// E_prev (a = 0..2) and, with the previous-B reading, B_prev (a = 3..5)
template <typename TS>
__device__ __forceinline__ int64_t e_at(const Consts& K, int a, int p) {
    return lane_off<Lay<TS>::EREC>(K, p) + Lay<TS>::E + CHUNK * Lay<TS>::EREC * a;
}

// Shift of the stored f, g of direction i (0 on the plain FP64 path).
__device__ __forceinline__ double fshift(const Consts& K, int i) { return K.fsh[i == 0 ? 0 : (i <= 6 ? 1 : 2)]; }
__device__ __forceinline__ double gshift(const Consts& K, int i) { return K.gsh[i == 0 ? 0 : (i <= 6 ? 1 : 2)]; }

// Neighbour offsets of one cell along one axis for displacements -2..+2,
// with periodic wrap or (open face) a copy of the first interior cell; with
// keep_low the coordinates -1, -2 stay (the ghost planes of a driven face).
__device__ __forceinline__ int map_coord(int v, int n, int periodic, int keep_low) {
    if (v < 0) return periodic ? (v + n >= 0 ? v + n : v + 2 * n) : (keep_low ? v : 0);
    if (v >= n) return periodic ? (v - n < n ? v - n : v - 2 * n) : n - 1;
    return v;
}

struct Nbr {
    int ox[5], oy[5], oz[5];  // element offsets for displacement d = -2..2 (index d + 2)
    __device__ __forceinline__ int at(int dx, int dy, int dz) const { return ox[dx + 2] + oy[dy + 2] + oz[dz + 2]; }
};

// STATE: offsets into the state arrays, which hold the ghost planes of a
// driven face below z = 0; otherwise offsets into plain N-cell field arrays
// (a driven face then acts as open).
// FLAT: one z-plane and no driven face, where every z-displacement leads back to the cell.
template <bool STATE, bool FLAT = false>
__device__ __forceinline__ Nbr make_nbr(const Consts& K, int x, int y, int z) {
    Nbr n;
    const int sy = K.nx, sz = K.nx * K.ny;
#pragma unroll
    for (int d = -2; d <= 2; ++d) {
        n.ox[d + 2] = map_coord(x + d, K.nx, K.per[0], 0) - x;
        n.oy[d + 2] = (map_coord(y + d, K.ny, K.per[1], 0) - y) * sy;
        n.oz[d + 2] = FLAT ? 0 : (map_coord(z + d, K.nz, K.per[2], STATE ? K.drv : 0) - z) * sz;
    }
    return n;
}

// Derivative along `axis` of a quantity X(x, y, z) at a cell: central
// differences (periodic wrap on periodic axes), one-sided towards the
// interior on the faces of a non-periodic axis, zero on an axis of one cell.
// The divergence operator of the normal-B adjustment and of max |div B|.
template <typename Fn>
__device__ __forceinline__ double axis_derivative(const Consts& K, int axis, int x, int y, int z, Fn&& X) {
    const int n = axis == 0 ? K.nx : (axis == 1 ? K.ny : K.nz);
    const int v = axis == 0 ? x : (axis == 1 ? y : z);
    const int ex = axis == 0, ey = axis == 1, ez = axis == 2;
    if (n == 1) return 0.0;
    if (!K.per[axis] && v == 0) return (X(x + ex, y + ey, z + ez) - X(x, y, z)) / K.dx;
    if (!K.per[axis] && v == n - 1) return (X(x, y, z) - X(x - ex, y - ey, z - ez)) / K.dx;
    const int wp = map_coord(v + 1, n, K.per[axis], 0) - v, wm = map_coord(v - 1, n, K.per[axis], 0) - v;
    return (X(x + ex * wp, y + ey * wp, z + ez * wp) - X(x + ex * wm, y + ey * wm, z + ez * wm)) / (2.0 * K.dx);
}

// Index of a face cell in the adjusted-normal-B arrays (face f = 2 axis + high).
__device__ __forceinline__ int64_t face_slot(const Consts& K, int f, int x, int y, int z) {
    const int a = f >> 1;
    const int64_t j = a == 0 ? y + (int64_t)K.ny * z : (a == 1 ? x + (int64_t)K.nx * z : x + (int64_t)K.nx * y);
    return K.fo[f] + j;
}

// Whether a cell lies on a face of a non-periodic axis other than `a` (an
// edge or corner cell when it also lies on a face of `a`).
__device__ __forceinline__ bool on_other_face(const Consts& K, int a, int x, int y, int z) {
    const int pos[3] = {x, y, z}, dims[3] = {K.nx, K.ny, K.nz};
    bool e = false;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b != a && dims[b] >= 2 && !K.per[b] && (pos[b] == 0 || pos[b] == dims[b] - 1)) e = true;
    return e;
}

// Normal-B adjustment of an open-face cell (Sec. IV, KH set-up): on a face
// cell that is not an edge or corner cell, replace the normal component by
// the value the face pass computed.
__device__ __forceinline__ void apply_face_b(const Consts& K, const double* __restrict__ faceB, int x, int y, int z,
                                             double B[3]) {
    const int pos[3] = {x, y, z}, dims[3] = {K.nx, K.ny, K.nz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool lo = pos[a] == 0 && K.open_lo[a], hi = pos[a] == dims[a] - 1 && K.open_hi[a];
        if ((lo || hi) && !on_other_face(K, a, x, y, z)) B[a] = faceB[face_slot(K, lo ? 2 * a : 2 * a + 1, x, y, z)];
    }
}

// Tile index with XCD-aware placement: block b runs on XCD b % 8, so XCD k is
// given the contiguous tile range [k P, (k + 1) P).
__device__ __forceinline__ int tile_of_block(int nblocks) {
    const int P = (nblocks + 7) / 8;
    return (blockIdx.x % 8) * P + blockIdx.x / 8;
}

// Moments and macroscopic solution of one cell in one step.
struct CellSol {
    double T00, T0[3], Tab[6], N0;   // moments (Tab: xx, yy, zz, xy, xz, yz)
    double Ep[3], B[3], rho, rho_g;  // previous E, this step's B, charge, Gauss charge
    double Epr[3];                   // E' of Eq. Cal_E
    double eps, p, n, gam, beta[3], E[3], J[3];
    int iters;
    int fallback;  // the learned guess was rejected (Newton started from E_f)
    bool ok;
};

// Fluid tensor T_fl = T - T_EM of the recovery: E_f = T_fl^00, S = T_fl^0a,
// Pi = T_fl^ab (xx, yy, zz, xy, xz, yz), with E_prev and the recovery's B
// (this step's, or with the previous-B reading the previous step's).
__device__ __forceinline__ void fluid_tensor(const Consts& K, const CellSol& M, const double (&B)[3], double& Ef,
                                             double S[3], double Pi[6]) {
    const double c = K.c, c2 = c * c;
    const double* E = M.Ep;
    const double E2 = E[0] * E[0] + E[1] * E[1] + E[2] * E[2];
    const double B2 = B[0] * B[0] + B[1] * B[1] + B[2] * B[2];
    const double U = 0.5 * (E2 + c2 * B2);
    Ef = M.T00 - K.eps0 * U;
    S[0] = M.T0[0] - K.eps0 * c * (E[1] * B[2] - E[2] * B[1]);
    S[1] = M.T0[1] - K.eps0 * c * (E[2] * B[0] - E[0] * B[2]);
    S[2] = M.T0[2] - K.eps0 * c * (E[0] * B[1] - E[1] * B[0]);
    Pi[0] = M.Tab[0] - K.eps0 * (U - E[0] * E[0] - c2 * B[0] * B[0]);
    Pi[1] = M.Tab[1] - K.eps0 * (U - E[1] * E[1] - c2 * B[1] * B[1]);
    Pi[2] = M.Tab[2] - K.eps0 * (U - E[2] * E[2] - c2 * B[2] * B[2]);
    Pi[3] = M.Tab[3] + K.eps0 * (E[0] * E[1] + c2 * B[0] * B[1]);
    Pi[4] = M.Tab[4] + K.eps0 * (E[0] * E[2] + c2 * B[0] * B[2]);
    Pi[5] = M.Tab[5] + K.eps0 * (E[1] * E[2] + c2 * B[1] * B[2]);
}

// Where the learned guess comes from: none (Newton from E_f), or the
// network evaluated on the wavefront with two lanes per cell (PAIR) or one
// lane per cell (SINGLE, two passes of 32 cells); MONITOR: Newton from E_f in
// a step with the guess enabled whose gate is closed, recording whether the
// gate opens for the next step.
enum GuessMode { GUESS_NONE = 0, GUESS_PAIR = 1, GUESS_SINGLE = 2, GUESS_MONITOR = 3 };

// Below this flow ratio |S| / E_f a cell takes no guess (Newton from E_f needs
// at most a few steps there, and on the flare box the network saved none for
// cells between 0.02 and 0.1), a wavefront of only such cells skips the
// network, and a step that meets no other cell closes the gate for the next.
#ifndef RMHDLB_GUESS_MIN_FLOW
#define RMHDLB_GUESS_MIN_FLOW 0.1
#endif
constexpr double GUESS_MIN_FLOW = RMHDLB_GUESS_MIN_FLOW;

// Record that this step met a cell above the gate (the lowest such lane of the
// wavefront stores; skipped once the slot holds this step's number).  Lanes
// that left the wavefront early do not take part.
__device__ __forceinline__ void open_gate(const Consts& K, bool moving) {
    const uint64_t m = __ballot(moving);
    if (K.gflag_wr && m && (int)(threadIdx.x & 63) == __builtin_ctzll(m) && *K.gflag_wr != K.gstep)
        *K.gflag_wr = K.gstep;
}

// Network guess of the eigenvalue for this lane's cell (all lanes of the
// wavefront call it together).  E_f (no guess) for nearly resting cells; NaN
// when the predicted |beta| >= 0.999 (those cells fall back to E_f).
template <int GM>
__device__ __forceinline__ double guess_lambda(const GuessTables* __restrict__ gt, double Ef, const double S[3],
                                               const double Pi[6], double N0, bool* gate) {
    double f[6], s;
    f[0] = flow_ratio(Ef, S, s);
    const bool moving = f[0] > GUESS_MIN_FLOW;
    if (!__any(moving)) return Ef;  // uniform over the wavefront
    if (gate) *gate = true;
    mlp_features(Ef, S, Pi, N0, s, f);
    float x[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) x[j] = (float)((f[j] - (double)gt->mu_x[j]) * (double)gt->inv_sd_x[j]);
    const int lane = threadIdx.x & 63;
    float y0, y1;
    if constexpr (GM == GUESS_PAIR) {
        mlp_wave(gt, x, lane & 31, lane & 31, y0, y1);  // cell n of the wavefront is lane n (and n + 32)
    } else {
        float a0, a1, c0, c1;
        mlp_wave(gt, x, lane & 31, lane & 31, a0, a1);
        mlp_wave(gt, x, 32 + (lane & 31), lane & 31, c0, c1);
        y0 = lane < 32 ? a0 : c0;
        y1 = lane < 32 ? a1 : c1;
    }
    const double t0 = (double)gt->mu_t[0] + (double)gt->sd_t[0] * (double)y0;
    const double bn = (double)gt->mu_t[1] + (double)gt->sd_t[1] * (double)y1;
    if (!moving) return Ef;
    return bn < 0.999 ? Ef * t0 : __builtin_nan("");
}

// Recovery and the Ohm-coupled E, J of one cell from its moments (M.T00,
// M.T0, M.Tab, M.N0, M.Epr, M.B, M.Ep, M.rho_g): fills eps, p, n, gam, beta,
// E, J, iters, fallback, ok.  Brec is the B of the recovery's T_EM (M.B, or
// the previous step's B); the Ohm solve always takes M.B.  With a guess mode
// every lane of the wavefront must call it together, and *gate (when given,
// uniform over the wavefront) is set when a cell of the wavefront lies above
// the guess's flow-ratio gate.
template <int GM = GUESS_NONE>
__device__ __forceinline__ void solve_cell(const Consts& K, CellSol& M, const double (&Brec)[3],
                                           const GuessTables* __restrict__ gt = nullptr, bool* gate = nullptr) {
    const double c = K.c, c2 = c * c;
    const double* B = M.B;
    double Ef, S[3], Pi[6];
    fluid_tensor(K, M, Brec, Ef, S, Pi);
    double lam;
    if constexpr (GM == GUESS_MONITOR)
        if (gate && __any(S[0] * S[0] + S[1] * S[1] + S[2] * S[2] > (GUESS_MIN_FLOW * Ef) * (GUESS_MIN_FLOW * Ef)))
            *gate = true;
    if constexpr (GM == GUESS_NONE || GM == GUESS_MONITOR) {
        M.iters = recover(Ef, S, Pi, lam, M.beta);
        M.fallback = 0;
    } else {
        const double lam0 = guess_lambda<GM>(gt, Ef, S, Pi, M.N0, gate);
        M.iters = recover_from_guess(Ef, S, Pi, lam0, lam, M.beta, M.fallback);
    }
    const double b2 = norm2(M.beta);
    M.gam = 1.0 / sqrt(1.0 - b2);
    M.n = M.N0 / M.gam;
    M.p = K.gm1 * (lam - M.n * c2);
    M.eps = lam;
    M.ok = (b2 < 1.0) && (lam > 0.0) && (M.n > 0.0) && (M.p >= 0.0) && isfinite(M.p);
    if (!M.ok) {
        const double nan = __builtin_nan("");
        M.eps = M.p = M.n = M.gam = nan;
#pragma unroll
        for (int a = 0; a < 3; ++a) M.beta[a] = M.E[a] = M.J[a] = nan;
        return;
    }

    // E from E = E' - (dt/2) mu0 c^2 J(E) with Eq. Ohm, by Sherman-Morrison:
    // (1 + K) E - (K / c^2)(E.u) u = R, R = E' - K u x B - q rho_G u
    const double u0 = c * M.beta[0], u1 = c * M.beta[1], u2 = c * M.beta[2];
    const double Kf = K.q * K.sigma * M.gam;
    const double uxB0 = u1 * B[2] - u2 * B[1], uxB1 = u2 * B[0] - u0 * B[2], uxB2 = u0 * B[1] - u1 * B[0];
    const double qr = K.q * M.rho_g;
    const double R0 = M.Epr[0] - Kf * uxB0 - qr * u0;
    const double R1 = M.Epr[1] - Kf * uxB1 - qr * u1;
    const double R2 = M.Epr[2] - Kf * uxB2 - qr * u2;
    const double uR = u0 * R0 + u1 * R1 + u2 * R2;
    const double coef = (Kf / c2) * uR / (1.0 + Kf * (1.0 - b2));
    const double inv1K = 1.0 / (1.0 + Kf);
    M.E[0] = (R0 + coef * u0) * inv1K;
    M.E[1] = (R1 + coef * u1) * inv1K;
    M.E[2] = (R2 + coef * u2) * inv1K;
    const double Eu = (M.E[0] * u0 + M.E[1] * u1 + M.E[2] * u2) / c2;
    const double sg = K.sigma * M.gam;
    M.J[0] = sg * (M.E[0] + uxB0 - Eu * u0) + M.rho_g * u0;
    M.J[1] = sg * (M.E[1] + uxB1 - Eu * u1) + M.rho_g * u1;
    M.J[2] = sg * (M.E[2] + uxB2 - Eu * u2) + M.rho_g * u2;
}

// f_eq of Eq. Dis_fun_EM in normalised variables (F = (c_t/c_0)^2 f), with
// the corrections that make its moments T_fluid + T_EM: the delta_i0
// coefficient 361 (3p - eps) / (33 (p + eps)), the minus sign of the
// (E.c_i)^2 term, the y-z cross terms, and c on the (B x E).c_i term.
// The per-cell setup runs in FP64; the per-direction evaluation in V (FP64 on
// the plain path, FP32 on the mixed-storage paths).
template <typename V>
struct FeqCellT {
    V P34, A1, Bc, g2, beta[3], b2, eps0;
    V X, BxE[3], E[3], cB[3];
    __device__ __forceinline__ void setup(double eps, double p, double gam, const double bta[3], const double Ev[3],
                                          const double Bv[3], double c, double e0) {
        P34 = (V)(0.75 * (eps + p));
        A1 = (V)(1.0 + (3.0 * p - eps) / (p + eps));
        Bc = (V)(361.0 * (3.0 * p - eps) / (33.0 * (p + eps)));
        g2 = (V)(gam * gam);
        b2 = (V)norm2(bta);
        double cb[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            beta[a] = (V)bta[a];
            E[a] = (V)Ev[a];
            cb[a] = c * Bv[a];
            cB[a] = (V)cb[a];
        }
        X = (V)(cb[0] * cb[0] + cb[1] * cb[1] + cb[2] * cb[2] + Ev[0] * Ev[0] + Ev[1] * Ev[1] + Ev[2] * Ev[2]);
        // c (B x E)
        BxE[0] = (V)(cb[1] * Ev[2] - cb[2] * Ev[1]);
        BxE[1] = (V)(cb[2] * Ev[0] - cb[0] * Ev[2]);
        BxE[2] = (V)(cb[0] * Ev[1] - cb[1] * Ev[0]);
        eps0 = (V)e0;
    }
    template <int I>
    __device__ __forceinline__ V eq() const;
};
using FeqCell = FeqCellT<double>;

// e_I . v, and the product over the axis pair that a face diagonal spans, without the terms that a zero
// component takes away (the compiler has to keep 0 x, which is not 0 for every x).
template <int I, typename V>
__device__ __forceinline__ V along(const V v[3]) {
    constexpr int ex = EX[I], ey = EY[I], ez = EZ[I];
    V r = V(0);
    if constexpr (ex != 0) r = ex * v[0];
    if constexpr (ey != 0) r = ex != 0 ? r + ey * v[1] : ey * v[1];
    if constexpr (ez != 0) r = ex != 0 || ey != 0 ? r + ez * v[2] : ez * v[2];
    return r;
}
template <int I, typename V, typename Fn>
__device__ __forceinline__ V across(Fn&& prod) {
    constexpr int ex = EX[I], ey = EY[I], ez = EZ[I];
    if constexpr (ex * ey != 0)
        return (ex * ey) * prod(0, 1);
    else if constexpr (ex * ez != 0)
        return (ex * ez) * prod(0, 2);
    else if constexpr (ey * ez != 0)
        return (ey * ez) * prod(1, 2);
    else
        return V(0);
}

// f_eq of direction sgn * e_I (sgn = +-1): the odd terms change sign, the
// weight is that of e_I.
template <int I, typename V>
__device__ __forceinline__ V feq_signed(const FeqCellT<V>& f, V sgn) {
    constexpr int ex = EX[I], ey = EY[I], ez = EZ[I];
    const V eb = sgn * along<I>(f.beta);
    const V cross = across<I, V>([&](int a, int b) { return f.beta[a] * f.beta[b]; });
    constexpr int a0 = ex ? 0 : (ey ? 1 : 2), a1 = ez ? 2 : 1;  // the axes of e_I
    // their squares; the rounding of the sum is fixed, so that a state does not depend on the compiler's choice
    V diag = V(0);
    if constexpr (I > 6)
        diag = a1 == 1 && sizeof(V) == 8 ? fma(f.beta[a0], f.beta[a0], f.beta[a1] * f.beta[a1])
                                         : fma(f.beta[a1], f.beta[a1], f.beta[a0] * f.beta[a0]);
    else if constexpr (I > 0)
        diag = f.beta[a0] * f.beta[a0];
    V fluid = f.A1 + V(19) * f.g2 * cross + V(4 * KAPPA) * f.g2 * eb +
              V(4.0 / 15.0) * f.g2 * (V(19) * diag - V(4) * f.b2);
    if constexpr (I == 0) fluid += f.Bc;
    const V Be = along<I>(f.cB), Ee = along<I>(f.E);
    const V BxEe = sgn * along<I>(f.BxE);
    const V crossEB = across<I, V>([&](int a, int b) { return f.E[a] * f.E[b] + f.cB[a] * f.cB[b]; });
    const V em = V(2.3) * f.X - V(SQRT19_3) * BxEe - V(3.8) * (Be * Be + Ee * Ee) - V(6.65) * crossEB;
    return V(weight(I)) * (f.P34 * fluid + f.eps0 * em);
}
template <typename V>
template <int I>
__device__ __forceinline__ V FeqCellT<V>::eq() const {
    return feq_signed<I>(*this, V(1));
}

template <int I, typename Fn>
__device__ __forceinline__ void static_for(Fn&& fn) {
    if constexpr (I < Q) {
        fn(std::integral_constant<int, I>{});
        static_for<I + 1>(fn);
    }
}

// ---------------------------------------------------- two lanes per cell

// The fused step with the populations of one cell split over a lane pair
// (lanes l and l ^ 32 of a wavefront, h = 0, 1).  Slot s = 1..9 of f and g is direction 2s-1+h,
// i.e. sgn * e_{2s-1} with sgn = +1 / -1, so both lanes run the same
// instructions on opposite directions; slot m = 0..11 of h is population
// 2m+h (same streaming offset, opposite e and b).  Lane 0 also owns the rest
// populations f_0, g_0; lane 1 owns h_rest.  Partial moments are summed over
// the pair with one xor-32 shuffle each, and both lanes then run the recovery
// and the Ohm solve on identical inputs.
//
// f and g are handled as stored deviations d (the shift is 0 on the plain
// path): the transport is linear and the shift is uniform, so the transported
// value is shift + transport(d); the moments add the exact sums of the shifts;
// the collisions write the new deviations directly.
constexpr int PTPB = 256;  // threads of a fused-step block: 128 cells, two lanes each (FP64), or 256, one lane each
// Waves per SIMD the fused kernels are compiled for: two in every form, which
// leaves a wave the 256 registers that the cell's populations and two records'
// loads in flight take (three spill in the FP32 batch kernels: 24 registers on
// single planes, 41-46 on boxes).
constexpr int FUSED_WAVES = 2;
// minmod(a, b): the median of a, b and 0, one instruction in FP32 (FP64: four) instead of five (seven).
__device__ __forceinline__ float median0(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
__device__ __forceinline__ double median0(double a, double b) { return fmax(fmin(a, b), fmin(fmax(a, b), 0.0)); }
// The same where a may be a NaN and b is then the slope: FP64's minima and maxima give b by themselves; in FP32 the
// median is taken of them (of a NaN itself it would be min(b, 0)).
__device__ __forceinline__ float median0_known(float a, float b) {
    return __builtin_amdgcn_fmed3f(fminf(a, b), fmaxf(a, b), 0.0f);
}
__device__ __forceinline__ double median0_known(double a, double b) { return median0(a, b); }

// x + y and x - y of stored values in the step's arithmetic.  FP16 values go
// through a fused multiply-add by a 1 that the compiler does not see, which
// the mixed-precision instruction takes with both conversions in one.
template <typename V, typename T>
__device__ __forceinline__ V sum_of(T x, T y, V one) {
    return sizeof(T) == sizeof(V) ? V(x) + V(y) : fma(V(x), one, V(y));
}
template <typename V, typename T>
__device__ __forceinline__ V difference(T x, T y, V one) {
    return sizeof(T) == sizeof(V) ? V(x) - V(y) : fma(V(x), one, -V(y));
}

// A population after its transport along the link without viscosity:
// f - C (face_p - face_m), face values f + slope minmod of the differences
// on both sides.  minmod takes no part of a value that it does not choose: an
// infinite downwind neighbour p1 leaves the finite slope f - m1, a NaN two
// cells upwind (m2) likewise.  A NaN of p1 has to reach the cell; the median
// does not carry it, so b = p1 - f goes back to the caller, who tests it
// (unordered, two populations per comparison).  Against b 0 added to f, which
// carries a NaN but turns an infinity into one too, and a plain median upwind
// (ms per step, then / now): FP16 256x256x256 1.663 / 1.664, its slab of
// 1024x2048 0.187 / 0.189, FP32 2.342 / 2.337 and 0.257 / 0.258.
template <typename V, typename T>
__device__ __forceinline__ V advect(T f, T m1, T m2, T p1, V cour, V slope, V one, V& b) {
    const V a = difference<V>(f, m1, one), c = difference<V>(m1, m2, one);
    b = difference<V>(p1, f, one);
    const V face_p = fma(slope, median0(a, b), V(f));
    const V face_m = fma(slope, median0_known(c, a), V(m1));
    return fma(-cour, face_p - face_m, V(f));
}

// Link of a slot as the step walks it (direction 2s - 1).  FLAT: the grid has
// one z-plane whose z-neighbours are the cell itself, so links and the
// Laplacian lie in the plane.
template <int S, bool FLAT>
struct Link {
    static constexpr int x = EX[2 * S - 1], y = EY[2 * S - 1], z = FLAT ? 0 : EZ[2 * S - 1];
    static constexpr int axes = (x != 0) + (y != 0) + (z != 0);
    // an axis link's points x -+ e are also the Laplacian's neighbours along that axis
    static constexpr bool lap_x = !(axes == 1 && x != 0), lap_y = !(axes == 1 && y != 0),
                          lap_z = !FLAT && !(axes == 1 && z != 0);
};

// Keeps a value in a register from here on.  As the statement is volatile and
// clobbers memory, loads written before it are issued before it and loads
// written after it are not issued earlier: the order in which the source
// issues a slot's loads and uses the slot before it holds in the machine code.
// What bounds the step without it is latency: scheduled freely, the compiler
// waited for nearly every load by itself to save registers, and a wave took
// about 400 cycles per vector-memory instruction (FP16, two waves per SIMD).
// With the next record's loads in flight while one is used (256x256x512, ms
// per step, chunked layout, before -> after): FP16 8.07 -> 3.55, FP32 6.22 ->
// 5.08, FP64 10.6 -> 10.2; before both changes 5.11, 5.53 and 11.0.
template <typename T>
__device__ __forceinline__ void pin(T& v) {
    asm volatile("" : "+v"(v)::"memory");
}
// Likewise a mask of lanes, in scalar registers.
__device__ __forceinline__ void pin_mask(uint64_t& m) { asm volatile("" : "+s"(m)); }

// Transport (collide-then-transport reading of Eq. rlb): link-wise
// minmod-MUSCL flux difference, plus the 7-point bulk-viscosity Laplacian
// for i != 0; g without viscosity.  Then the streaming of h, the moments,
// the recovery and E, J.
// One thread per cell, FP64 arithmetic (moments and diagnostics pass).  The
// shift of a stored array is constant in space, so it transports to itself
// and is added back after the transport.  What bounds it is what bounds the
// step, so a slot's loads (its two opposite directions) are likewise in
// flight while the slot before it is used; 256x256x512, the whole pass in
// FP64: 20.4 ms with loads where the compiler put them (100 registers
// spilled), 10.2 so; FP16 10.8 and 3.8.
template <int GM, typename TS, typename TE>
__device__ __forceinline__ void macroscopic(const char* __restrict__ src, const double* __restrict__ faceB,
                                            const GuessTables* __restrict__ gt, const Consts& K, int cell,
                                            const Nbr& nb, int x, int y, int z, CellSol& M) {
    constexpr bool PAIR = !quad_layout<TS>();
    const int pos = (int)K.g0 + cell;
    double t0x = 0, t0y = 0, t0z = 0, txx = 0, tyy = 0, tzz = 0, txy = 0, txz = 0, tyz = 0;
    // (f, g) of the slot's direction 2s - 1 and of 2s
    using Both = vec4<TS>;
    // f of both directions (quads come whole)
    using Fs = std::conditional_t<PAIR, vec2<TS>, vec4<TS>>;
    struct Raw {
        Both c, m1, p1;
        std::conditional_t<PAIR, vec2<TS>, vec4<TS>> m2, p2;  // FP64: of the direction that needs them
        Fs xp, xm, yp, ym, zp, zm;
    };
    auto issue = [&](auto ic, Raw& r) {
        constexpr int s = decltype(ic)::value;
        using K_ = Link<s, false>;
        constexpr int i0 = 2 * s - 1, i1 = 2 * s;
        auto both = [&](int o) {
            const int64_t q = lane_off<16>(K, pos + o);
            Both v;
            if constexpr (PAIR) {
                const vec2<TS> a = *reinterpret_cast<const vec2<TS>*>(src + q + rec_off<TS>(i0));
                const vec2<TS> b = *reinterpret_cast<const vec2<TS>*>(src + q + rec_off<TS>(i1));
                v.x = a.x, v.y = a.y, v.z = b.x, v.w = b.y;
            } else {
                v = *reinterpret_cast<const Both*>(src + q + rec_off<TS>(i0));
            }
            return v;
        };
        auto one_of = [&](int i, int o) {
            return *reinterpret_cast<const std::conditional_t<PAIR, vec2<TS>, vec4<TS>>*>(
                src + lane_off<16>(K, pos + o) + rec_off<TS>(PAIR ? i : i0));
        };
        auto fs = [&](int o) {
            if constexpr (PAIR) {
                const int64_t q = lane_off<16>(K, pos + o);
                Fs v;
                v.x = *reinterpret_cast<const TS*>(src + q + rec_off<TS>(i0));
                v.y = *reinterpret_cast<const TS*>(src + q + rec_off<TS>(i1));
                return v;
            } else {
                return both(o);
            }
        };
        r.c = both(0);
        r.m1 = both(nb.at(-K_::x, -K_::y, -K_::z));
        r.p1 = both(nb.at(K_::x, K_::y, K_::z));
        r.m2 = one_of(i0, nb.at(-2 * K_::x, -2 * K_::y, -2 * K_::z));
        r.p2 = one_of(i1, nb.at(2 * K_::x, 2 * K_::y, 2 * K_::z));
        if constexpr (K_::lap_x) r.xp = fs(nb.at(1, 0, 0)), r.xm = fs(nb.at(-1, 0, 0));
        if constexpr (K_::lap_y) r.yp = fs(nb.at(0, 1, 0)), r.ym = fs(nb.at(0, -1, 0));
        if constexpr (K_::lap_z) r.zp = fs(nb.at(0, 0, 1)), r.zm = fs(nb.at(0, 0, -1));
    };
    auto arrive = [&](auto ic, Raw& r) {
        using K_ = Link<decltype(ic)::value, false>;
        pin(r.c), pin(r.m1), pin(r.p1), pin(r.m2), pin(r.p2);
        auto from_link = [](const Both& v) {
            Fs f;
            if constexpr (PAIR)
                f.x = v.x, f.y = v.z;
            else
                f = v;
            return f;
        };
        if constexpr (K_::lap_x)
            pin(r.xp), pin(r.xm);
        else
            r.xp = from_link(r.p1), r.xm = from_link(r.m1);
        if constexpr (K_::lap_y)
            pin(r.yp), pin(r.ym);
        else
            r.yp = from_link(r.p1), r.ym = from_link(r.m1);
        if constexpr (K_::lap_z)
            pin(r.zp), pin(r.zm);
        else
            r.zp = from_link(r.p1), r.zm = from_link(r.m1);
    };
    TS hraw[QH];
    auto issue_h = [&]() {
#pragma unroll
        for (int m = 0; m < QH / 2; ++m) {
            const int k0 = 2 * m, o = nb.at(-SX[k0], -SY[k0], -SZ[k0]);
            if constexpr (PAIR) {
                hraw[k0] = *reinterpret_cast<const TS*>(src + h_at<TS>(K, k0, pos + o));
                hraw[k0 + 1] = *reinterpret_cast<const TS*>(src + h_at<TS>(K, k0 + 1, pos + o));
            } else {
                const vec2<TS> v = *reinterpret_cast<const vec2<TS>*>(src + h_at<TS>(K, k0, pos + o));
                hraw[k0] = v.x, hraw[k0 + 1] = v.y;
            }
        }
    };
    const double f_rest = ld<TS>(src, f_at<TS>(K, 0, pos)), g_rest = ld<TS>(src, g_at<TS>(K, 0, pos));
    Raw raw[2];
    issue(std::integral_constant<int, 1>{}, raw[1]);
    M.T00 = f_rest + fshift(K, 0);
    M.N0 = g_rest + gshift(K, 0);
    static_for<1>([&](auto ic) {
        constexpr int s = decltype(ic)::value;
        if constexpr (s <= 9) {
            if constexpr (s < 9)
                issue(std::integral_constant<int, s + 1>{}, raw[(s + 1) & 1]);
            else
                issue_h();
            Raw& r = raw[s & 1];
            arrive(ic, r);
            auto add = [&](auto qc, double f0, double fm1, double fm2, double fp1, double g0, double gm1, double gm2,
                           double gp1, double sx, double sy, double sz) {
                constexpr int i = decltype(qc)::value;
                const double lap = fma(-6.0, f0, sx + sy + sz);
                double bf, bg;
                const double fa = advect<double, double>(f0, fm1, fm2, fp1, K.cour, K.slope, 1.0, bf);
                const double ga = advect<double, double>(g0, gm1, gm2, gp1, K.cour, K.slope, 1.0, bg);
                const double fv = fma(K.kv, lap, bf == bf ? fa : bf) + fshift(K, i);
                const double gv = (bg == bg ? ga : bg) + gshift(K, i);
                M.T00 += fv;
                M.N0 += gv;
                if (EX[i]) t0x += EX[i] * fv;
                if (EY[i]) t0y += EY[i] * fv;
                if (EZ[i]) t0z += EZ[i] * fv;
                if (EX[i]) txx += fv;
                if (EY[i]) tyy += fv;
                if (EZ[i]) tzz += fv;
                if (EX[i] * EY[i]) txy += (EX[i] * EY[i]) * fv;
                if (EX[i] * EZ[i]) txz += (EX[i] * EZ[i]) * fv;
                if (EY[i] * EZ[i]) tyz += (EY[i] * EZ[i]) * fv;
            };
            auto second = [](const Fs& v) { return (double)(PAIR ? v[1] : v[PAIR ? 1 : 2]); };
            add(std::integral_constant<int, 2 * s - 1>{}, r.c.x, r.m1.x, r.m2[0], r.p1.x, r.c.y, r.m1.y, r.m2[1],
                r.p1.y, (double)r.xp[0] + (double)r.xm[0], (double)r.yp[0] + (double)r.ym[0],
                (double)r.zp[0] + (double)r.zm[0]);
            add(std::integral_constant<int, 2 * s>{}, r.c.z, r.p1.z, r.p2[PAIR ? 0 : 2], r.m1.z, r.c.w, r.p1.w,
                r.p2[PAIR ? 1 : 3], r.m1.w, second(r.xp) + second(r.xm), second(r.yp) + second(r.ym),
                second(r.zp) + second(r.zm));
            pin(M.T00), pin(M.N0);  // the slot's arithmetic stays here
        }
    });
    M.T0[0] = KAPPA * t0x;
    M.T0[1] = KAPPA * t0y;
    M.T0[2] = KAPPA * t0z;
    M.Tab[0] = KAPPA2 * txx;
    M.Tab[1] = KAPPA2 * tyy;
    M.Tab[2] = KAPPA2 * tzz;
    M.Tab[3] = KAPPA2 * txy;
    M.Tab[4] = KAPPA2 * txz;
    M.Tab[5] = KAPPA2 * tyz;

    // previous E and its Gauss charge
    auto Ea = [&](int a, int o) { return ld<TE>(src, e_at<TS>(K, a, pos + o)); };
    M.Ep[0] = Ea(0, 0);
    M.Ep[1] = Ea(1, 0);
    M.Ep[2] = Ea(2, 0);
    M.rho_g = K.eps0 * K.inv_2dx *
              ((Ea(0, nb.at(1, 0, 0)) - Ea(0, nb.at(-1, 0, 0))) + (Ea(1, nb.at(0, 1, 0)) - Ea(1, nb.at(0, -1, 0))) +
               (Ea(2, nb.at(0, 0, 1)) - Ea(2, nb.at(0, 0, -1))));

    // stream h (Eq. LB_Maxwell): h_k(x) = h*_k(x - v_k dt)
    double ehx = 0, ehy = 0, ehz = 0, bx = 0, by = 0, bz = 0, hs = 0;
#pragma unroll
    for (int k = 0; k < QH; ++k) {
        const double h = (double)hraw[k];
        hs += h;
        if (EHX[k]) ehx += EHX[k] * h;
        if (EHY[k]) ehy += EHY[k] * h;
        if (EHZ[k]) ehz += EHZ[k] * h;
        if (BHX[k]) bx += BHX[k] * h;
        if (BHY[k]) by += BHY[k] * h;
        if (BHZ[k]) bz += BHZ[k] * h;
    }
    const double ec = K.c * INV_SQRT2;  // |e_k| / |ehat_k|
    M.Epr[0] = ec * ehx;
    M.Epr[1] = ec * ehy;
    M.Epr[2] = ec * ehz;
    M.B[0] = bx;
    M.B[1] = by;
    M.B[2] = bz;
    M.rho = ld<TS>(src, h_at<TS>(K, QH, pos)) + hs;

    if (K.divb) apply_face_b(K, faceB, x, y, z, M.B);
    if (K.bprev) {
        double Bp[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) Bp[a] = Ea(3 + a, 0);
        solve_cell<GM>(K, M, Bp, gt);
    } else {
        solve_cell<GM>(K, M, M.B, gt);
    }
}

// The two lanes of a cell are l and l ^ 32 of a wavefront: each half of the
// wavefront then reads 32 consecutive values of one array, which the vector
// memory path coalesces (with the partner in the adjacent lane every
// instruction touched two arrays lane by lane and the texture units, not
// HBM, set the step time).
template <typename V>
__device__ __forceinline__ V pair_sum(V v) {
    return v + __shfl_xor(v, 32, 64);
}

// VR: the alternative readings, bit 0 the printed semi-implicit f collision
// of Eq. rlb, f' = (f + omega f_eq) / (1 + omega) (else explicit, Reading
// R4); bit 1 the limited Lax-Wendroff face values (else MUSCL, Reading R2);
// bit 2 the external force; bit 3 the previous step's B in the recovery and
// f_eq (else this step's, Reading R10), carried in the state.
template <bool NT, typename TS, typename TE, typename V, int GM, int VR, bool FLAT, bool SYNC>
__device__ __forceinline__ void pair_cell(const char* __restrict__ sd, char* __restrict__ dd,
                                          const double* __restrict__ faceB, const GuessTables* __restrict__ gt,
                                          const Consts& K, int cell, const Nbr& nb, int h, int x, int y, int z,
                                          bool active, double& bmax, bool& gate) {
    using L = Lay<TS>;
    const V sgn = h ? V(-1) : V(1);
    const int pos = (int)K.g0 + cell;
    // Byte offset of this lane's records at a stencil point, the lane's choice
    // between the two arrays of a pair included (the arrays of a pair are
    // neighbours in the chunk); what is left per array is a constant.
    const int h16 = h ? CHUNK * 16 : 0, h8 = h ? CHUNK * 8 : 0;
    auto rec = [&](int o) { return lane_off<16>(K, pos + o) + h16; };
    auto mrec = [&](int o) { return lane_off<8>(K, pos + o) + h8; };
    const int64_t c16 = lane_off<16>(K, pos), c8 = lane_off<8>(K, pos);
    constexpr int CM = VR & 1;
    const V cour = (V)K.cour, kv = (V)K.kv, slope = (VR & 2) ? (V)K.slope : V(0.5);
    V Fv[10], Gv[10], Hv[13];
    V t00 = 0, t0x = 0, t0y = 0, t0z = 0, txx = 0, tyy = 0, tzz = 0, txy = 0, txz = 0, tyz = 0, n0 = 0;
    uint64_t lost = 0;  // lanes with a NaN in a downwind neighbour: their energy, and with it the cell, becomes one
    // slot 0: f_0, g_0 (lane 0) and h_rest (lane 1)
    {
        const vec2<V> fg0 = ldv2<V, TS>(sd, c16);
        const V hr = ldv_once<V, TS>(sd, c8 + L::H + CHUNK * 8 * QH);
        Fv[0] = h ? V(0) : fg0.x;
        Gv[0] = h ? V(0) : fg0.y;
        Hv[12] = h ? hr : V(0);
        t00 = Fv[0];
        n0 = Gv[0];
    }
    const int64_t cc = c16 + h16;
    const int64_t lap_xp = rec(nb.at(1, 0, 0)), lap_xm = rec(nb.at(-1, 0, 0)), lap_yp = rec(nb.at(0, 1, 0)),
                  lap_ym = rec(nb.at(0, -1, 0)), lap_zp = rec(nb.at(0, 0, 1)), lap_zm = rec(nb.at(0, 0, -1));
    // The loads of a slot: its pairs at the centre and the link's points, its f at the Laplacian's.
    struct Raw {
        vec2<TS> c0, m2, m1, p1;
        TS xp, xm, yp, ym, zp, zm;
    };
    auto issue = [&](auto ic, Raw& r) {
        using K_ = Link<decltype(ic)::value, FLAT>;
        const char* __restrict__ fga = sd + CHUNK * 16 * (2 * decltype(ic)::value - 1);  // uniform base of the pairs
        auto pr = [&](int64_t o) { return *reinterpret_cast<const vec2<TS>*>(fga + o); };
        auto f = [&](int64_t o) { return *reinterpret_cast<const TS*>(fga + o); };
        r.c0 = pr(cc);
        if constexpr (K_::axes > 0) {
            r.m2 = pr(rec(h ? nb.at(2 * K_::x, 2 * K_::y, 2 * K_::z) : nb.at(-2 * K_::x, -2 * K_::y, -2 * K_::z)));
            r.m1 = pr(rec(h ? nb.at(K_::x, K_::y, K_::z) : nb.at(-K_::x, -K_::y, -K_::z)));
            r.p1 = pr(rec(h ? nb.at(-K_::x, -K_::y, -K_::z) : nb.at(K_::x, K_::y, K_::z)));
        }
        if constexpr (K_::lap_x) r.xp = f(lap_xp), r.xm = f(lap_xm);
        if constexpr (K_::lap_y) r.yp = f(lap_yp), r.ym = f(lap_ym);
        if constexpr (K_::lap_z) r.zp = f(lap_zp), r.zm = f(lap_zm);
    };
    auto arrive = [&](auto ic, Raw& r) {
        using K_ = Link<decltype(ic)::value, FLAT>;
        pin(r.c0);
        if constexpr (K_::axes > 0)
            pin(r.m2), pin(r.m1), pin(r.p1);
        else
            r.m2 = r.m1 = r.p1 = r.c0;
        if constexpr (K_::lap_x) pin(r.xp), pin(r.xm);
        if constexpr (K_::lap_y) pin(r.yp), pin(r.ym);
        if constexpr (K_::lap_z) pin(r.zp), pin(r.zm);
        if constexpr (FLAT) r.zp = r.zm = r.c0.x;
    };
    TS hraw[12];
    auto issue_h = [&]() {
#pragma unroll
        for (int m = 0; m < 12; ++m) {
            const int k0 = 2 * m;
            hraw[m] = __builtin_nontemporal_load(reinterpret_cast<const TS*>(
                sd + L::H + CHUNK * 8 * k0 + mrec(nb.at(-SX[k0], -SY[k0], -SZ[k0]))));
        }
    };
    Raw raw[2];
    issue(std::integral_constant<int, 1>{}, raw[1]);
    static_for<1>([&](auto ic) {
        constexpr int s = decltype(ic)::value;
        if constexpr (s <= 9) {
            constexpr int i0 = 2 * s - 1;
            constexpr int ex = EX[i0], ey = EY[i0], ez = EZ[i0];
            using K_ = Link<s, FLAT>;
            if constexpr (SYNC) __builtin_amdgcn_s_barrier();
            // the next slot's loads (after the last slot, the Maxwell populations') are in flight while this
            // slot's arrive and are used
            if constexpr (s < 9)
                issue(std::integral_constant<int, s + 1>{}, raw[(s + 1) & 1]);
            else
                issue_h();
            Raw& r = raw[s & 1];
            arrive(ic, r);
            const V f0 = r.c0.x, fm1 = r.m1.x, fp1 = r.p1.x;
            const V up = h ? fm1 : fp1, dn = h ? fp1 : fm1;  // f at x + e_i0 and x - e_i0 (lane 1 walks -e)
            const V lxp = K_::lap_x ? r.xp : up, lxm = K_::lap_x ? r.xm : dn;
            const V lyp = K_::lap_y ? r.yp : up, lym = K_::lap_y ? r.ym : dn;
            const V lzp = K_::lap_z || FLAT ? r.zp : up, lzm = K_::lap_z || FLAT ? r.zm : dn;
            const V lap = (lxp + lxm) + (lyp + lym) + (lzp + lzm) - V(6) * f0;
            V bf, bg;
            const V fv = fma(kv, lap, advect<V, TS>(r.c0.x, r.m1.x, r.m2.x, r.p1.x, cour, slope, V(1), bf));
            const V gv = advect<V, TS>(r.c0.y, r.m1.y, r.m2.y, r.p1.y, cour, slope, V(1), bg);
            lost |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(bf, bg));
            pin_mask(lost);
            Fv[s] = fv;
            Gv[s] = gv;
            pin(Fv[s]), pin(Gv[s]);  // the slot's arithmetic stays here
            t00 += fv;
            n0 += gv;
            const V sf = sgn * fv;
            if (ex) t0x += ex * sf;
            if (ey) t0y += ey * sf;
            if (ez) t0z += ez * sf;
            if (ex) txx += fv;
            if (ey) tyy += fv;
            if (ez) tzz += fv;
            if (ex * ey) txy += (ex * ey) * fv;
            if (ex * ez) txz += (ex * ez) * fv;
            if (ey * ez) tyz += (ey * ez) * fv;
        }
    });
    // E of the last step, and the Gauss charge: lane 0 takes E_x(x+-1), E_y(y+1); lane 1 E_y(y-1), E_z(z+-1)
    auto Ea = [&](int a, int64_t off) { return ld<TE>(sd, off + L::E + CHUNK * 8 * a); };
    auto at8 = [&](int dx, int dy, int dz) { return lane_off<8>(K, pos + nb.at(dx, dy, dz)); };
    double Ep[3], ga, gb, gc;
#pragma unroll
    for (int a = 0; a < 3; ++a) Ep[a] = Ea(a, c8);
    ga = Ea(h ? 1 : 0, h ? at8(0, -1, 0) : at8(1, 0, 0));
    gb = Ea(h ? 2 : 0, h ? at8(0, 0, 1) : at8(-1, 0, 0));
    gc = Ea(h ? 2 : 1, h ? at8(0, 0, -1) : at8(0, 1, 0));
#pragma unroll
    for (int m = 0; m < 12; ++m) pin(hraw[m]);
    V ehx = 0, ehy = 0, ehz = 0, bx = 0, by = 0, bz = 0, hs = 0;
#pragma unroll
    for (int m = 0; m < 12; ++m) {
        const int k0 = 2 * m;
        const V v = hraw[m];
        Hv[m] = v;
        hs += v;
        const V sv = sgn * v;
        if (EHX[k0]) ehx += EHX[k0] * sv;
        if (EHY[k0]) ehy += EHY[k0] * sv;
        if (EHZ[k0]) ehz += EHZ[k0] * sv;
        if (BHX[k0]) bx += BHX[k0] * sv;
        if (BHY[k0]) by += BHY[k0] * sv;
        if (BHZ[k0]) bz += BHZ[k0] * sv;
    }
    CellSol M;
#pragma unroll
    for (int a = 0; a < 3; ++a) M.Ep[a] = Ep[a];
    const double gpart = ((h ? -ga : ga) + (h ? gb : -gb)) + (h ? -gc : gc);
    M.T00 = K.fs0 + (double)pair_sum(__builtin_amdgcn_inverse_ballot_w64(lost) ? V(__builtin_nan("")) : t00);
    M.N0 = K.gs0 + (double)pair_sum(n0);
    M.T0[0] = KAPPA * (double)pair_sum(t0x);
    M.T0[1] = KAPPA * (double)pair_sum(t0y);
    M.T0[2] = KAPPA * (double)pair_sum(t0z);
    M.Tab[0] = KAPPA2 * (K.fsaa + (double)pair_sum(txx));
    M.Tab[1] = KAPPA2 * (K.fsaa + (double)pair_sum(tyy));
    M.Tab[2] = KAPPA2 * (K.fsaa + (double)pair_sum(tzz));
    M.Tab[3] = KAPPA2 * (double)pair_sum(txy);
    M.Tab[4] = KAPPA2 * (double)pair_sum(txz);
    M.Tab[5] = KAPPA2 * (double)pair_sum(tyz);
    const double ec = K.c * INV_SQRT2;
    M.Epr[0] = ec * (double)pair_sum(ehx);
    M.Epr[1] = ec * (double)pair_sum(ehy);
    M.Epr[2] = ec * (double)pair_sum(ehz);
    M.B[0] = (double)pair_sum(bx);
    M.B[1] = (double)pair_sum(by);
    M.B[2] = (double)pair_sum(bz);
    // The Maxwell populations relax towards h_eq of the streamed B (an
    // adjusted face B enters only the fluid coupling): take its B part,
    // B . b_k / 8, into h* = 2 h_eq - h now, while the streamed B is at hand.
    {
        const V sb0 = (V)M.B[0], sb1 = (V)M.B[1], sb2 = (V)M.B[2];
#pragma unroll
        for (int m = 0; m < 12; ++m) {
            const int k0 = 2 * m;
            Hv[m] -= V(0.25) * sgn * (BHX[k0] * sb0 + BHY[k0] * sb1 + BHZ[k0] * sb2);
        }
    }
    M.rho = (double)pair_sum(Hv[12] + hs);
    M.rho_g = K.eps0 * K.inv_2dx * pair_sum(gpart);
    if (K.divb) apply_face_b(K, faceB, x, y, z, M.B);
    FeqCellT<V> fe;
    if constexpr ((VR & 8) != 0) {
        double Bp[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) Bp[a] = Ea(3 + a, c8);
        solve_cell<GM>(K, M, Bp, gt, &gate);
        fe.setup(M.eps, M.p, M.gam, M.beta, M.Ep, Bp, K.c, K.eps0);
    } else {
        solve_cell<GM>(K, M, M.B, gt, &gate);
        fe.setup(M.eps, M.p, M.gam, M.beta, M.Ep, M.B, K.c, K.eps0);
    }

    // collisions and stores (new deviations)
    const V rate = (V)(M.gam * K.inv_tau);
    const V wg = (V)K.wg, inv1wg = (V)K.inv1wg;
    const V ng = (V)(M.n * M.gam);
    const V gc1 = (V)K.gc1, gc2 = (V)K.gc2, gc3b2 = (V)(K.gc3 * norm2(M.beta));
    const V bx_ = (V)M.beta[0], by_ = (V)M.beta[1], bz_ = (V)M.beta[2];
    // External force (Reading R26): c dt F^a into T^{0a} through the moving
    // populations, (19/9) w_i (e_i . c dt F) / kappa each, and the work
    // c dt F . beta into T^00 through the rest population; on while the
    // previous step's largest |beta| is below the gate.
    double fw = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
    if constexpr ((VR & 4) != 0) {
        bmax = fmax(bmax, sqrt(M.beta[0] * M.beta[0] + M.beta[1] * M.beta[1] + M.beta[2] * M.beta[2]));
        if (!(K.fgate > 0.0) || *K.vmax_prev < K.fgate) {
            const double cdt = K.dx * INV_SQRT2;  // c dt
            fx = cdt * K.force[cell];
            fy = cdt * K.force[K.N + cell];
            fz = cdt * K.force[2 * K.N + cell];
            fw = fx * M.beta[0] + fy * M.beta[1] + fz * M.beta[2];
        }
    }
    if (h == 0) {
        const V q0 = (V)K.fsh[0] - fe.template eq<0>();
        const V geq0 = (V)K.wp[0] * ng * (V(1) - gc3b2);
        V f0n = CM == 0 ? Fv[0] - rate * (Fv[0] + q0) : (Fv[0] - rate * q0) / (V(1) + rate);
        if constexpr ((VR & 4) != 0) f0n += (V)fw;
        if (active) st2<NT, TS>(dd, c16, f0n, (Gv[0] + wg * (geq0 - (V)K.gsh[0])) * inv1wg);
    } else {
        if (active) st<NT, TS>(dd, c8 + L::H + CHUNK * 8 * QH, (V)(2.0 * M.rho) - Hv[12]);
    }
    static_for<1>([&](auto ic) {
        constexpr int s = decltype(ic)::value;
        if constexpr (s <= 9) {
            constexpr int i0 = 2 * s - 1;
            constexpr int cls = i0 <= 6 ? 1 : 2;
            const V eb = sgn * (EX[i0] * bx_ + EY[i0] * by_ + EZ[i0] * bz_);
            const V om = rate * (V(1) - V(KAPPA) * eb);
            const V q = (V)K.fsh[cls] - feq_signed<i0>(fe, sgn);
            const V geq = (V)K.wp[cls] * ng * (V(1) + gc1 * eb + gc2 * eb * eb - gc3b2);
            V fn = CM == 0 ? Fv[s] - om * (Fv[s] + q) : (Fv[s] - om * q) / (V(1) + om);
            if constexpr ((VR & 4) != 0) {
                constexpr double wcls = cls == 1 ? 99.0 / 722.0 : 9.0 / 361.0;  // D3Q19 weights
                fn += (V)((19.0 / 9.0) * wcls / KAPPA * ((h ? -1.0 : 1.0) * (EX[i0] * fx + EY[i0] * fy + EZ[i0] * fz)));
            }
            if (active)
                st2<NT, TS>(dd, cc + CHUNK * 16 * i0, fn, (Gv[s] + wg * (geq - (V)K.gsh[cls])) * inv1wg);
        }
    });
    const V cj = (V)K.cj, cE = (V)K.ce;
    const V J0 = (V)M.J[0], J1 = (V)M.J[1], J2 = (V)M.J[2];
    const V E0 = (V)M.E[0], E1 = (V)M.E[1], E2 = (V)M.E[2];
#pragma unroll
    for (int m = 0; m < 12; ++m) {
        const int k0 = 2 * m;
        const V heq = cj * (SX[k0] * J0 + SY[k0] * J1 + SZ[k0] * J2) + sgn * cE * (EHX[k0] * E0 + EHY[k0] * E1 + EHZ[k0] * E2);
        if (active) st<NT, TS>(dd, c8 + h8 + L::H + CHUNK * 8 * k0, V(2) * heq - Hv[m]);
    }
    if (h == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
            if (active) st<NT, TE>(dd, c8 + L::E + CHUNK * 8 * a, M.E[a]);
    } else if constexpr ((VR & 8) != 0) {  // this step's coupling B is the next one's previous B
#pragma unroll
        for (int a = 0; a < 3; ++a)
            if (active) st<NT, TE>(dd, c8 + L::E + CHUNK * 8 * (3 + a), M.B[a]);
    }
}

// ---------------------------------------------------- one lane per cell

// 16 bytes of FP16 (two quads)
template <bool NT, typename T, typename V>
__device__ __forceinline__ void st8(char* __restrict__ d, int64_t o, const vec4<V>& lo, const vec4<V>& hi) {
    typedef T vec8 __attribute__((ext_vector_type(8)));
    vec8 v;
    v[0] = static_cast<T>(lo.x);
    v[1] = static_cast<T>(lo.y);
    v[2] = static_cast<T>(lo.z);
    v[3] = static_cast<T>(lo.w);
    v[4] = static_cast<T>(hi.x);
    v[5] = static_cast<T>(hi.y);
    v[6] = static_cast<T>(hi.z);
    v[7] = static_cast<T>(hi.w);
    put_raw<NT>(d, o, v);
}

// The fused step of one cell in one lane (FP32 storage, quad layout; FP16,
// double-quad layout, where one load at the centre and at each Laplacian
// point serves the two slots of a record):
// slot s = 1..9 carries the opposite directions i0 = 2s - 1 (+e) and
// i1 = 2s (-e), and one load per point of the link x - 2e .. x + 2e and of the
// Laplacian serves both; the Maxwell populations 2m, 2m + 1 come from one load
// of the cell they stream from.  The arithmetic per direction is that of
// pair_cell (the readings it implements are listed there); only the
// assignment of work to lanes and the order of the moment sums differ.
template <bool NT, typename TS, typename TE, typename V, int GM, int VR, bool FLAT, bool SYNC>
__device__ __forceinline__ void quad_cell(const char* __restrict__ sd, char* __restrict__ dd,
                                          const double* __restrict__ faceB, const GuessTables* __restrict__ gt,
                                          const Consts& K, int cell, const Nbr& nb, int x, int y, int z, bool active,
                                          double& bmax, bool& gate) {
    using L = Lay<TS>;
    const int pos = (int)K.g0 + cell;
    // byte offsets of this cell's records at a stencil point; what is left per array is a constant
    auto rec = [&](int o) { return lane_off<16>(K, pos + o); };
    const int64_t cc = lane_off<16>(K, pos), ch = lane_off<L::HREC>(K, pos), ce = lane_off<4>(K, pos);
    constexpr int CM = VR & 1;
    const V cour = (V)K.cour, kv = (V)K.kv, slope = (VR & 2) ? (V)K.slope : V(0.5);
    V Fv[Q], Gv[Q], Hv[QH + 1];
    V t00 = 0, t0x = 0, t0y = 0, t0z = 0, txx = 0, tyy = 0, tzz = 0, txy = 0, txz = 0, tyz = 0, n0 = 0;
    uint64_t lost = 0;  // lanes with a NaN in a downwind neighbour: their energy, and with it the cell, becomes one
    const int64_t lap_xp = rec(nb.at(1, 0, 0)), lap_xm = rec(nb.at(-1, 0, 0)), lap_yp = rec(nb.at(0, 1, 0)),
                  lap_ym = rec(nb.at(0, -1, 0)), lap_zp = rec(nb.at(0, 0, 1)), lap_zm = rec(nb.at(0, 0, -1));
    // Transport and moments of slot s from its quads at the link points x - 2e .. x + 2e and the
    // Laplacian's six neighbours.
    V one = V(1);  // not seen by the compiler: see sum_of
    if constexpr (sizeof(TS) != sizeof(V)) asm("" : "+s"(one));
    auto transport = [&](auto sc, const vec4<TS>& q0, const vec4<TS>& qm2, const vec4<TS>& qm1, const vec4<TS>& qp1,
                         const vec4<TS>& qp2, const vec4<TS>& lxp, const vec4<TS>& lxm, const vec4<TS>& lyp,
                         const vec4<TS>& lym, const vec4<TS>& lzp, const vec4<TS>& lzm) {
        constexpr int s = decltype(sc)::value;
        constexpr int i0 = 2 * s - 1, i1 = 2 * s;
        constexpr int ex = EX[i0], ey = EY[i0], ez = EZ[i0];
        // +e: upwind stencil x - 2e, x - e, x, x + e; -e: x + 2e, x + e, x, x - e
        auto laplacian = [&](TS f0, TS xp, TS xm, TS yp, TS ym, TS zp, TS zm) {
            return fma(V(-6), V(f0), sum_of<V>(xp, xm, one) + sum_of<V>(yp, ym, one) + sum_of<V>(zp, zm, one));
        };
        V bf0, bf1, bg0, bg1;
        const V fv0 = fma(kv, laplacian(q0.x, lxp.x, lxm.x, lyp.x, lym.x, lzp.x, lzm.x),
                          advect<V, TS>(q0.x, qm1.x, qm2.x, qp1.x, cour, slope, one, bf0));
        const V fv1 = fma(kv, laplacian(q0.z, lxp.z, lxm.z, lyp.z, lym.z, lzp.z, lzm.z),
                          advect<V, TS>(q0.z, qp1.z, qp2.z, qm1.z, cour, slope, one, bf1));
        const V gv0 = advect<V, TS>(q0.y, qm1.y, qm2.y, qp1.y, cour, slope, one, bg0);
        const V gv1 = advect<V, TS>(q0.w, qp1.w, qp2.w, qm1.w, cour, slope, one, bg1);
        lost |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(bf0, bf1)) |
                __builtin_amdgcn_ballot_w64(__builtin_isunordered(bg0, bg1));
        pin_mask(lost);
        Fv[i0] = fv0;
        Fv[i1] = fv1;
        Gv[i0] = gv0;
        Gv[i1] = gv1;
        const V sum = fv0 + fv1, dif = fv0 - fv1;
        t00 += sum;
        n0 += gv0 + gv1;
        if (ex) t0x += ex * dif;
        if (ey) t0y += ey * dif;
        if (ez) t0z += ez * dif;
        if (ex) txx += sum;
        if (ey) tyy += sum;
        if (ez) tzz += sum;
        if (ex * ey) txy += (ex * ey) * sum;
        if (ex * ez) txz += (ex * ez) * sum;
        if (ey * ez) tyz += (ey * ez) * sum;
    };
    // The loads of a record (FP32: one slot; FP16: two, the centre and the Laplacian's points in one load each
    // and the link's points in one per slot); the next record's are in flight while this one's arrive and are used.
    constexpr bool DQ = dquad_layout<TS>();
    using Rec = unsigned __attribute__((ext_vector_type(4)));   // 16 bytes: a quad (FP32), two quads (FP16)
    using Half = std::conditional_t<DQ, vec2<unsigned>, Rec>;   // one slot's quad
    struct Raw {
        Rec c, xp, xm, yp, ym, zp, zm;
        Half a[4], b[4];  // link points x - 2e, x + 2e, x - e, x + e of the record's slots
    };
    constexpr int RECS = DQ ? DQUAD_RECORDS : 9;
    auto rec16 = [&](const char* __restrict__ base, int64_t o) { return *reinterpret_cast<const Rec*>(base + o); };
    auto half8 = [&](const char* __restrict__ base, int64_t o) { return *reinterpret_cast<const Half*>(base + o); };
    auto issue_links = [&](auto sc, const char* __restrict__ base, Half (&q)[4]) {
        using K_ = Link<decltype(sc)::value, FLAT>;
        if constexpr (K_::axes > 0) {
            q[0] = half8(base, rec(nb.at(-2 * K_::x, -2 * K_::y, -2 * K_::z)));
            q[1] = half8(base, rec(nb.at(2 * K_::x, 2 * K_::y, 2 * K_::z)));
        }
        if constexpr (K_::axes > 1) {
            q[2] = half8(base, rec(nb.at(-K_::x, -K_::y, -K_::z)));
            q[3] = half8(base, rec(nb.at(K_::x, K_::y, K_::z)));
        }
    };
    auto pin_links = [&](auto sc, Half (&q)[4]) {
        using K_ = Link<decltype(sc)::value, FLAT>;
        if constexpr (K_::axes > 0) pin(q[0]), pin(q[1]);
        if constexpr (K_::axes > 1) pin(q[2]), pin(q[3]);
    };
    // record r: slots sa and (FP16) sb, 0 when the second quad is the rest one
    auto slot_a = [](auto rc) { return std::integral_constant<int, DQ ? 2 * decltype(rc)::value + 1 : decltype(rc)::value + 1>{}; };
    auto slot_b = [](auto rc) { return std::integral_constant<int, DQ && decltype(rc)::value < 4 ? 2 * decltype(rc)::value + 2 : 0>{}; };
    auto issue = [&](auto rc, Raw& q) {
        constexpr auto sa = slot_a(rc);
        constexpr auto sb = slot_b(rc);
        const char* __restrict__ base = sd + CHUNK * 16 * (DQ ? decltype(rc)::value : sa.value);
        q.c = rec16(base, cc);
        // an FP32 axis slot's points x -+ e also serve its Laplacian; an FP16 record's serve both slots
        q.xp = rec16(base, lap_xp), q.xm = rec16(base, lap_xm);
        q.yp = rec16(base, lap_yp), q.ym = rec16(base, lap_ym);
        if constexpr (!FLAT) q.zp = rec16(base, lap_zp), q.zm = rec16(base, lap_zm);
        issue_links(sa, base, q.a);
        if constexpr (sb.value != 0) issue_links(sb, base + 8, q.b);
    };
    auto arrive = [&](auto rc, Raw& q) {
        constexpr auto sa = slot_a(rc);
        constexpr auto sb = slot_b(rc);
        pin(q.c), pin(q.xp), pin(q.xm), pin(q.yp), pin(q.ym);
        if constexpr (!FLAT) pin(q.zp), pin(q.zm);
        pin_links(sa, q.a);
        if constexpr (sb.value != 0) pin_links(sb, q.b);
    };
    auto quad_of = [](const auto& w, int half) {  // the quad in a record or half record
        vec4<TS> r;
        if constexpr (sizeof(w) == 16 && !DQ) {
            r.x = __builtin_bit_cast(float, (unsigned)w[0]), r.y = __builtin_bit_cast(float, (unsigned)w[1]);
            r.z = __builtin_bit_cast(float, (unsigned)w[2]), r.w = __builtin_bit_cast(float, (unsigned)w[3]);
        } else {
            const int o = sizeof(w) == 16 ? 2 * half : 0;
            const vec2<_Float16> lo = __builtin_bit_cast(vec2<_Float16>, (unsigned)w[o]),
                                 hi = __builtin_bit_cast(vec2<_Float16>, (unsigned)w[o + 1]);
            r.x = lo.x, r.y = lo.y, r.z = hi.x, r.w = hi.y;
        }
        return r;
    };
    auto use = [&](auto sc, const Raw& q, int half, const Half (&lk)[4]) {
        constexpr int s = decltype(sc)::value;
        using K_ = Link<s, FLAT>;
        const vec4<TS> c = quad_of(q.c, half), xp = quad_of(q.xp, half), xm = quad_of(q.xm, half),
                      yp = quad_of(q.yp, half), ym = quad_of(q.ym, half), zp = FLAT ? c : quad_of(q.zp, half),
                      zm = FLAT ? c : quad_of(q.zm, half);
        const vec4<TS> m2 = K_::axes > 0 ? quad_of(lk[0], 0) : c, p2 = K_::axes > 0 ? quad_of(lk[1], 0) : c;
        vec4<TS> m1, p1;
        if constexpr (K_::axes == 0)
            m1 = p1 = c;
        else if constexpr (K_::axes > 1)
            m1 = quad_of(lk[2], 0), p1 = quad_of(lk[3], 0);
        else if constexpr (K_::x != 0)
            m1 = K_::x > 0 ? xm : xp, p1 = K_::x > 0 ? xp : xm;
        else if constexpr (K_::y != 0)
            m1 = K_::y > 0 ? ym : yp, p1 = K_::y > 0 ? yp : ym;
        else
            m1 = zm, p1 = zp;
        transport(sc, c, m2, m1, p1, p2, xp, xm, yp, ym, zp, zm);
        pin(Fv[2 * s - 1]), pin(Fv[2 * s]), pin(Gv[2 * s - 1]), pin(Gv[2 * s]);  // the slot's arithmetic stays here
    };
    using HRaw = std::conditional_t<DQ, unsigned, vec2<unsigned>>;
    HRaw hraw[12];
    auto issue_h = [&]() {
#pragma unroll
        for (int m = 0; m < 12; ++m) {
            const int k0 = 2 * m;
            hraw[m] = __builtin_nontemporal_load(reinterpret_cast<const HRaw*>(
                sd + L::H + CHUNK * L::HREC * m + lane_off<L::HREC>(K, pos + nb.at(-SX[k0], -SY[k0], -SZ[k0]))));
        }
    };
    Rec rest_raw = {0, 0, 0, 0};
    if constexpr (!DQ) rest_raw = rec16(sd, cc);
    Raw raw[2];
    issue(std::integral_constant<int, 0>{}, raw[0]);
    static_for<0>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        if constexpr (r < RECS) {
            if constexpr (SYNC && r % 2 == 0) __builtin_amdgcn_s_barrier();
            if constexpr (r + 1 < RECS)
                issue(std::integral_constant<int, r + 1>{}, raw[(r + 1) & 1]);
            else
                issue_h();
            Raw& q = raw[r & 1];
            arrive(rc, q);
            if constexpr (r == 0 && !DQ) {
                pin(rest_raw);
                const vec4<TS> fg0 = quad_of(rest_raw, 0);
                Fv[0] = fg0.x;
                Gv[0] = fg0.y;
                Hv[QH] = fg0.z;
                t00 = Fv[0];
                n0 = Gv[0];
            }
            use(slot_a(rc), q, 0, q.a);
            if constexpr (slot_b(rc).value != 0) {
                use(slot_b(rc), q, 1, q.b);
            } else if constexpr (DQ) {  // the rest quad
                const vec4<TS> fg0 = quad_of(q.c, 1);
                Fv[0] = fg0.x;
                Gv[0] = fg0.y;
                Hv[QH] = fg0.z;
                t00 += Fv[0];
                n0 += Gv[0];
            }
        }
    });
    // E of the last step and its neighbours for the Gauss charge
    auto Ea = [&](int a, int64_t off) { return ldv<V, TE>(sd, off + L::E + CHUNK * 4 * a); };
    auto at4 = [&](int dx, int dy, int dz) { return lane_off<4>(K, pos + nb.at(dx, dy, dz)); };
    V Ep[3], gE[6];
#pragma unroll
    for (int a = 0; a < 3; ++a) Ep[a] = Ea(a, ce);
    gE[0] = Ea(0, at4(1, 0, 0)), gE[1] = Ea(0, at4(-1, 0, 0)), gE[2] = Ea(1, at4(0, 1, 0));
    gE[3] = Ea(1, at4(0, -1, 0)), gE[4] = Ea(2, at4(0, 0, 1)), gE[5] = Ea(2, at4(0, 0, -1));
#pragma unroll
    for (int m = 0; m < 12; ++m) pin(hraw[m]);
    // stream h (Eq. LB_Maxwell): the pair 2m, 2m + 1 from its common source cell
    V ehx = 0, ehy = 0, ehz = 0, bx = 0, by = 0, bz = 0, hs = 0;
#pragma unroll
    for (int m = 0; m < 12; ++m) {
        const int k0 = 2 * m;
        vec2<V> v;
        if constexpr (DQ) {
            const vec2<_Float16> w = __builtin_bit_cast(vec2<_Float16>, hraw[m]);
            v.x = (V)w.x, v.y = (V)w.y;
        } else {
            v.x = __builtin_bit_cast(float, (unsigned)hraw[m][0]), v.y = __builtin_bit_cast(float, (unsigned)hraw[m][1]);
        }
        Hv[k0] = v.x;
        Hv[k0 + 1] = v.y;
        hs += v.x + v.y;
        const V d = v.x - v.y;  // population 2m + 1 has the opposite e and b
        if (EHX[k0]) ehx += EHX[k0] * d;
        if (EHY[k0]) ehy += EHY[k0] * d;
        if (EHZ[k0]) ehz += EHZ[k0] * d;
        if (BHX[k0]) bx += BHX[k0] * d;
        if (BHY[k0]) by += BHY[k0] * d;
        if (BHZ[k0]) bz += BHZ[k0] * d;
    }
    CellSol M;
#pragma unroll
    for (int a = 0; a < 3; ++a) M.Ep[a] = (double)Ep[a];
    {
        const double dv = (((double)gE[0] - (double)gE[1]) + ((double)gE[2] - (double)gE[3])) +
                          ((double)gE[4] - (double)gE[5]);
        M.rho_g = K.eps0 * K.inv_2dx * dv;
    }
    M.T00 = K.fs0 + (double)(__builtin_amdgcn_inverse_ballot_w64(lost) ? V(__builtin_nan("")) : t00);
    M.N0 = K.gs0 + (double)n0;
    M.T0[0] = KAPPA * (double)t0x;
    M.T0[1] = KAPPA * (double)t0y;
    M.T0[2] = KAPPA * (double)t0z;
    M.Tab[0] = KAPPA2 * (K.fsaa + (double)txx);
    M.Tab[1] = KAPPA2 * (K.fsaa + (double)tyy);
    M.Tab[2] = KAPPA2 * (K.fsaa + (double)tzz);
    M.Tab[3] = KAPPA2 * (double)txy;
    M.Tab[4] = KAPPA2 * (double)txz;
    M.Tab[5] = KAPPA2 * (double)tyz;
    const double ec = K.c * INV_SQRT2;
    M.Epr[0] = ec * (double)ehx;
    M.Epr[1] = ec * (double)ehy;
    M.Epr[2] = ec * (double)ehz;
    M.B[0] = (double)bx;
    M.B[1] = (double)by;
    M.B[2] = (double)bz;
    // h* = 2 h_eq - h: the B part of h_eq (of the streamed B) now
    {
        const V sb0 = (V)M.B[0], sb1 = (V)M.B[1], sb2 = (V)M.B[2];
#pragma unroll
        for (int m = 0; m < 12; ++m) {
            const int k0 = 2 * m;
            const V bb = V(0.25) * (BHX[k0] * sb0 + BHY[k0] * sb1 + BHZ[k0] * sb2);
            Hv[k0] -= bb;
            Hv[k0 + 1] += bb;
        }
    }
    M.rho = (double)(Hv[QH] + hs);
    if (K.divb) apply_face_b(K, faceB, x, y, z, M.B);
    FeqCellT<V> fe;
    if constexpr ((VR & 8) != 0) {
        double Bp[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) Bp[a] = Ea(3 + a, ce);
        solve_cell<GM>(K, M, Bp, gt, &gate);
        fe.setup(M.eps, M.p, M.gam, M.beta, M.Ep, Bp, K.c, K.eps0);
    } else {
        solve_cell<GM>(K, M, M.B, gt, &gate);
        fe.setup(M.eps, M.p, M.gam, M.beta, M.Ep, M.B, K.c, K.eps0);
    }

    // collisions and stores (new deviations)
    const V rate = (V)(M.gam * K.inv_tau);
    const V wg = (V)K.wg, inv1wg = (V)K.inv1wg;
    const V ng = (V)(M.n * M.gam);
    const V gc1 = (V)K.gc1, gc2 = (V)K.gc2, gc3b2 = (V)(K.gc3 * norm2(M.beta));
    const V bx_ = (V)M.beta[0], by_ = (V)M.beta[1], bz_ = (V)M.beta[2];
    double fw = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
    if constexpr ((VR & 4) != 0) {
        bmax = fmax(bmax, sqrt(M.beta[0] * M.beta[0] + M.beta[1] * M.beta[1] + M.beta[2] * M.beta[2]));
        if (!(K.fgate > 0.0) || *K.vmax_prev < K.fgate) {
            const double cdt = K.dx * INV_SQRT2;  // c dt
            fx = cdt * K.force[cell];
            fy = cdt * K.force[K.N + cell];
            fz = cdt * K.force[2 * K.N + cell];
            fw = fx * M.beta[0] + fy * M.beta[1] + fz * M.beta[2];
        }
    }
    vec4<V> rest;  // new (f_0, g_0, h_rest, 0)
    {
        const V q0 = (V)K.fsh[0] - fe.template eq<0>();
        const V geq0 = (V)K.wp[0] * ng * (V(1) - gc3b2);
        V f0n = CM == 0 ? Fv[0] - rate * (Fv[0] + q0) : (Fv[0] - rate * q0) / (V(1) + rate);
        if constexpr ((VR & 4) != 0) f0n += (V)fw;
        rest.x = f0n;
        rest.y = (Gv[0] + wg * (geq0 - (V)K.gsh[0])) * inv1wg;
        rest.z = (V)(2.0 * M.rho) - Hv[QH];
        rest.w = V(0);
        if constexpr (!dquad_layout<TS>())
            if (active) st4<NT, TS>(dd, cc, rest);
    }
    // the new quad (f, g, f-bar, g-bar) of slot s
    auto collide = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int i0 = 2 * s - 1, i1 = 2 * s;
        constexpr int cls = i0 <= 6 ? 1 : 2;
        const V eb = EX[i0] * bx_ + EY[i0] * by_ + EZ[i0] * bz_;  // e_i0 . beta; -eb for i1
        const V q_0 = (V)K.fsh[cls] - feq_signed<i0>(fe, V(1));
        const V q_1 = (V)K.fsh[cls] - feq_signed<i0>(fe, V(-1));
        const V om0 = rate * (V(1) - V(KAPPA) * eb), om1 = rate * (V(1) + V(KAPPA) * eb);
        const V ebb = gc2 * eb * eb - gc3b2;
        const V geq_0 = (V)K.wp[cls] * ng * (V(1) + gc1 * eb + ebb);
        const V geq_1 = (V)K.wp[cls] * ng * (V(1) - gc1 * eb + ebb);
        V fn0 = CM == 0 ? Fv[i0] - om0 * (Fv[i0] + q_0) : (Fv[i0] - om0 * q_0) / (V(1) + om0);
        V fn1 = CM == 0 ? Fv[i1] - om1 * (Fv[i1] + q_1) : (Fv[i1] - om1 * q_1) / (V(1) + om1);
        if constexpr ((VR & 4) != 0) {
            constexpr double wcls = cls == 1 ? 99.0 / 722.0 : 9.0 / 361.0;  // D3Q19 weights
            const double fe_ = (19.0 / 9.0) * wcls / KAPPA * (EX[i0] * fx + EY[i0] * fy + EZ[i0] * fz);
            fn0 += (V)fe_;
            fn1 += (V)(-fe_);
        }
        vec4<V> q;
        q.x = fn0;
        q.y = (Gv[i0] + wg * (geq_0 - (V)K.gsh[cls])) * inv1wg;
        q.z = fn1;
        q.w = (Gv[i1] + wg * (geq_1 - (V)K.gsh[cls])) * inv1wg;
        return q;
    };
    if constexpr (!dquad_layout<TS>()) {
        static_for<1>([&](auto ic) {
            constexpr int s = decltype(ic)::value;
            if constexpr (s <= 9) {
                const vec4<V> q = collide(ic);
                if (active) st4<NT, TS>(dd, cc + CHUNK * 16 * s, q);
            }
        });
    } else {
        static_for<0>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            if constexpr (r < DQUAD_RECORDS) {
                const vec4<V> a = collide(std::integral_constant<int, 2 * r + 1>{});
                if constexpr (r < 4) {
                    const vec4<V> b = collide(std::integral_constant<int, 2 * r + 2>{});
                    if (active) st8<NT, TS>(dd, cc + CHUNK * 16 * r, a, b);
                } else {
                    if (active) st8<NT, TS>(dd, cc + CHUNK * 16 * r, a, rest);
                }
            }
        });
    }
    const V cj = (V)K.cj, cE = (V)K.ce;
    const V J0 = (V)M.J[0], J1 = (V)M.J[1], J2 = (V)M.J[2];
    const V E0 = (V)M.E[0], E1 = (V)M.E[1], E2 = (V)M.E[2];
#pragma unroll
    for (int m = 0; m < 12; ++m) {
        const int k0 = 2 * m;
        const V hj = cj * (SX[k0] * J0 + SY[k0] * J1 + SZ[k0] * J2);
        const V he = cE * (EHX[k0] * E0 + EHY[k0] * E1 + EHZ[k0] * E2);
        if (active)
            st2<NT, TS>(dd, ch + L::H + CHUNK * L::HREC * m, V(2) * (hj + he) - Hv[k0], V(2) * (hj - he) - Hv[k0 + 1]);
    }
    if (active) {
#pragma unroll
        for (int a = 0; a < 3; ++a) st<NT, TE>(dd, ce + L::E + CHUNK * 4 * a, M.E[a]);
        if constexpr ((VR & 8) != 0) {
#pragma unroll
            for (int a = 0; a < 3; ++a) st<NT, TE>(dd, ce + L::E + CHUNK * 4 * (3 + a), M.B[a]);
        }
    }
}

// ------------------------------------------------------------------ kernels

// Whether the wavefronts of a block keep in step through the slots (a barrier
// per slot in FP64, per two in FP32).  What bounds the three-dimensional step
// in these forms is the lines that a CU's L1 has under way to L2 (about 70 of
// 128 bytes, at 700 cycles each): in step, the wavefronts of a tile find each
// other's rows and planes in L1.  256x256x512 with tiles of two planes, ms per
// step free / in step: FP64 10.0 / 9.36, FP32 5.0 / 4.75; FP16, which is bound
// by arithmetic, 3.42 / 3.48, and slabs lose 2-4 %.  Batches of boxes and tiles
// of one plane gain too: 16 boxes of 64x64x64 FP64 1.22 / 1.14, FP32 0.598 /
// 0.585; 256x256x64 in FP64's 64-wide tiles with the printed collision 1.27 /
// 1.21, Lax-Wendroff faces 1.27 / 1.20, the previous-B reading 1.31 / 1.25.
// A wavefront that has no
// rows left ends, and the barrier then waits for the others only.  Not in the
// persistent kernel, whose blocks meet at barriers of their own.
template <typename TS, bool FLAT>
constexpr bool in_step() {
    return !FLAT && sizeof(TS) >= 4;
}

// The step's constants in memory that it never writes (its kernel arguments,
// or a batch's table).  reread() hides from the compiler that they do not
// change, so that a plane takes them anew by scalar loads: kept across the
// walk they outgrow the scalar registers, and every spilled one costs a lane
// move (and its wait state) where it is used.
typedef const __attribute__((address_space(4))) Consts* ConstsPtr;
__device__ __forceinline__ const Consts& reread(ConstsPtr kp) {
    asm volatile("" : "+s"(kp));
    return *(const Consts*)kp;
}
// Likewise the state's base pointers (uniform, in global memory), so that the
// bases of its arrays are added up at their use and not kept across the walk:
// a step of 4096 cells takes 10.75 us instead of 11.04, 512 x 512 cells 69.0
// instead of 71.0.
template <typename T>
__device__ __forceinline__ T* again(T* p) {
    const uint64_t v = (uint64_t)p;
    uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)v) |
                 (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32;
    asm volatile("" : "+s"(u));
    return (T*)(__attribute__((address_space(1))) T*)u;
}

// One block owns a row group of 128 (FP64, two lanes per cell) or 256 cells:
// ROWS = 128 / PXT or 256 / PXT rows of PXT cells (a power of two), PYT of them along y in each
// of ZT neighbouring planes (step_walk), yw such groups stacked along y.  It
// walks zb z-planes, the yw groups of its planes one after another.  A chunk
// of zg * zb planes is shared by zg blocks per column, which take its planes
// (ZT at a time) in turn, so that the zg blocks of a column run at
// neighbouring planes at the same time and the z-neighbour planes of the
// stencil are fetched once into L2 for all of them (zg = 1: one block walks zb
// consecutive planes).  Blocks are numbered column-fastest within a chunk, the
// zg blocks of a column next to each other, and XCD k receives the contiguous
// block range [k P, (k + 1) P): the columns one XCD runs at the same time are
// neighbours marching through the same planes, so the y-halo meets in that
// XCD's L2 as well.
// With the learned guess the network runs on whole wavefronts, so lanes past
// a ragged edge stay and compute a copy of the edge cell without storing it.
template <bool NT, typename TS, typename TE, typename V, int GM, int PXT, int VR, bool FLAT, bool SYNC>
__device__ __forceinline__ void fused_block(const char* __restrict__ sd, char* __restrict__ dd,
                                            const double* __restrict__ faceB, const GuessTables* __restrict__ gt,
                                            ConstsPtr kp, int tiles_x, int ncol, int zb, int zt, int zg, int yw, int b) {
    const Consts& K = *(const Consts*)kp;
    // pair layout (FP64): 128 cells per row group, two lanes each; quad and double-quad layouts (FP32,
    // FP16): 256 cells, one lane each
    constexpr bool ONE = quad_layout<TS>();
    constexpr int ROWS = cells_per_block(sizeof(TS)) / PXT, MOST = most_planes(sizeof(TS), PXT, FLAT);
    constexpr int LG_ROWS = __builtin_ctz(ROWS);
    const int ZT = MOST == 1 ? 1 : zt, lg = LG_ROWS + 1 - ZT, PYT = 1 << lg;  // ZT is 1 or 2
    const int per = ncol * zg, zc = b / per, r = b % per;
    const int col = r / zg, zoff = r % zg;
    const int tx = col % tiles_x, ty = col / tiles_x;
    // pair layout: cell c of a row group is lane c % 32 (h = 0) and lane c % 32 + 32 (h = 1) of
    // wavefront c / 32; quad layout: cell c is thread c
    const int lane = threadIdx.x & 63;
    const int c = ONE ? (int)threadIdx.x : (int)(threadIdx.x >> 6) * 32 + (lane & 31), h = ONE ? 0 : lane >> 5;
    const int xr = tx * PXT + (c % PXT);
    int x = xr;
    const int ybase = (ty * yw << lg) + (c / PXT & (PYT - 1));
    // plane of the tile this wavefront works on (its rows share it)
    const int zl = MOST == 1 ? 0 : __builtin_amdgcn_readfirstlane(c / PXT >= PYT);
    // with the force every lane stays (the wavefront's largest |beta| is
    // reduced over all 64 lanes)
    constexpr bool all_lanes = GM == GUESS_PAIR || GM == GUESS_SINGLE || (VR & 4) != 0;
    // row groups of this lane that lie inside the grid (the later groups are further along y)
    int ng = yw;
    if (ybase >= K.ny) ng = 0;
    else if (ybase + (yw - 1) * PYT >= K.ny) ng = ((K.ny - 1 - ybase) >> lg) + 1;
    if constexpr (!all_lanes) {
        if (x >= K.nx || ng == 0) return;  // both lanes of a pair leave together
    } else {
        x = min(x, K.nx - 1);
    }
    const int z0 = zc * zb * zg, z1 = min(K.nz, z0 + zb * zg);
    double bmax = 0.0;
    bool gate = false;  // a cell of the walk lay above the guess's gate (uniform over the wavefront)
    // The lane's coordinates are made opaque at every plane, so that the x- and
    // y-parts of the neighbour table are recomputed per plane (a few integer
    // operations) instead of being kept across the walk (FP16 1 % slower then).
    const int groups = all_lanes ? yw : ng;
    for (int zp = z0 + zoff * ZT; zp < z1; zp += zg * ZT) {
        // the last planes of a chunk may be fewer than the tile's
        const bool inside = zp + zl < z1;
        if (!all_lanes && !inside) break;
        const int z = all_lanes ? min(zp + zl, z1 - 1) : zp + zl;
        for (int j = 0; j < groups; ++j) {
            const int yj = ybase + j * PYT;
            const bool active = xr < K.nx && yj < K.ny && inside;
            int xp = x, yp = all_lanes ? min(yj, K.ny - 1) : yj, hp = h;
            asm volatile("" : "+v"(xp), "+v"(yp), "+v"(hp));
            const Consts& Kp = reread(kp);
            const char* sp = again(sd);
            char* dp = again(dd);
            const int cell = xp + Kp.nx * (yp + Kp.ny * z);
            const Nbr nb = make_nbr<true, FLAT>(Kp, xp, yp, z);
            if constexpr (ONE)
                quad_cell<NT, TS, TE, V, GM, VR, FLAT, SYNC>(sp, dp, faceB, gt, Kp, cell, nb, xp, yp, z,
                                                 all_lanes ? active : true, bmax, gate);
            else
                pair_cell<NT, TS, TE, V, GM, VR, FLAT, SYNC>(sp, dp, faceB, gt, Kp, cell, nb, hp, xp, yp, z,
                                                 all_lanes ? active : true, bmax, gate);
        }
    }
    if constexpr (GM != GUESS_NONE) open_gate(K, gate);
    if constexpr ((VR & 4) != 0) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) bmax = fmax(bmax, __shfl_xor(bmax, o, 64));
        if (lane == 0) K.vmax_part[(int64_t)b * (PTPB / 64) + (threadIdx.x >> 6)] = bmax;
    }
}

constexpr int STEP_CONSTS_AT = 4 * sizeof(void*);  // K among k_fused_step's arguments: after four pointers
static_assert(alignof(Consts) == sizeof(void*), "K follows the pointers without padding");
template <bool NT, typename TS, typename TE, typename V, int GM, int PXT, int VR, bool FLAT>
__global__ __launch_bounds__(PTPB, FUSED_WAVES) void k_fused_step(const char* __restrict__ sd,
                                                        char* __restrict__ dd, const double* __restrict__ faceB,
                                                        const GuessTables* __restrict__ gt, Consts K,
                                                        int tiles_x, int ncol, int zb, int zt, int zg, int yw, int nblk) {
    const int b = tile_of_block(nblk);
    if (b >= nblk) return;  // uniform over the block
    // With the guess enabled every step launches the network kernel and the monitor kernel (its own
    // instantiation, so that it carries none of the network's registers); the one the gate does not
    // select leaves at once (uniform over the grid).
    if constexpr (GM == GUESS_MONITOR) {
        if (*K.gflag_rd == K.gstep - 1) return;
    } else if constexpr (GM != GUESS_NONE) {
        if (*K.gflag_rd != K.gstep - 1) return;
        if (blockIdx.x == 0 && threadIdx.x == 0 && K.gcount) *K.gcount += 1;  // one writer per step
    }
    const ConstsPtr kp = (ConstsPtr)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                                     STEP_CONSTS_AT);
    fused_block<NT, TS, TE, V, GM, PXT, VR, FLAT, in_step<TS, FLAT>()>(sd, dd, faceB, gt, kp, tiles_x, ncol, zb, zt, zg, yw, b);
}

// Index of the instance whose range [first[i], first[i + 1]) holds v (first
// is ascending with first[0] = 0); uniform over the block.
template <typename Get>
__device__ __forceinline__ int find_instance(int ninst, int64_t v, Get first) {
    int lo = 0, hi = ninst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first(mid) <= v)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Batched step: the blocks of every instance in one launch.  Block b is
// mapped XCD-aware over the whole batch, then to its instance by the prefix
// table of block counts, so neighbouring tiles of one instance still share
// an XCD.  parity selects which of each instance's buffers is read.  WV:
// waves per SIMD the kernel is compiled for (the occupancy the batch tuner
// sweeps).
template <bool NT, typename TS, typename TE, typename V, int PXT, int WV, bool FLAT>
__global__ __launch_bounds__(PTPB, WV) void k_fused_batch(const BatchInst* __restrict__ I, int ninst, int total,
                                                          int parity) {
    const int b = tile_of_block(total);
    if (b >= total) return;
    const int i = find_instance(ninst, b, [&](int j) { return I[j].blk0; });
    const BatchInst& B = I[i];
    fused_block<NT, TS, TE, V, GUESS_NONE, PXT, 0, FLAT, in_step<TS, FLAT>()>(
        B.buf[parity], B.buf[1 - parity], B.faceB, nullptr, (ConstsPtr)(uintptr_t)&B.K, B.tiles_x, B.ncol, B.zb, B.zt, 1, B.yw, (int)(b - B.blk0));
}

// B of Eq. Cal_B at a cell from the streamed h (population order, FP64).
template <typename TS>
__device__ __forceinline__ double streamed_B(const char* __restrict__ src, const Consts& K, int comp, int x, int y,
                                             int z) {
    const Nbr nb = make_nbr<true>(K, x, y, z);
    const int pos = (int)K.g0 + x + K.nx * (y + K.ny * z);
    double b = 0.0;
#pragma unroll
    for (int k = 0; k < QH; ++k) {
        const int bk = comp == 0 ? BHX[k] : (comp == 1 ? BHY[k] : BHZ[k]);
        if (bk) b += bk * ld<TS>(src, h_at<TS>(K, k, pos + nb.at(-SX[k], -SY[k], -SZ[k])));
    }
    return b;
}

// Normal B of the open-face cells for this step (Sec. IV, KH set-up): in a
// cell on an open face of axis a (not an edge or corner cell) the discrete
// divergence is made zero with
// the streamed B of the inner neighbour and the tangential derivatives of
// the streamed B:  low face  B_a = B_a(x + e_a) + dx sum_{b != a} d_b B_b,
//                  high face B_a = B_a(x - e_a) - dx sum_{b != a} d_b B_b.
// One thread per face cell over the six faces; inactive faces return.
template <typename TS>
__device__ __forceinline__ void face_b_cell(const char* __restrict__ src, const Consts& K, double* __restrict__ faceB,
                                            int64_t i) {
    if (i >= K.fo[6]) return;
    int f = 0;
    while (f < 5 && i >= K.fo[f + 1]) ++f;
    const int a = f >> 1, high = f & 1;
    if (!(high ? K.open_hi[a] : K.open_lo[a])) return;
    const int64_t j = i - K.fo[f];
    int x, y, z;
    if (a == 0) {
        y = (int)(j % K.ny);
        z = (int)(j / K.ny);
        x = high ? K.nx - 1 : 0;
    } else if (a == 1) {
        x = (int)(j % K.nx);
        z = (int)(j / K.nx);
        y = high ? K.ny - 1 : 0;
    } else {
        x = (int)(j % K.nx);
        y = (int)(j / K.nx);
        z = high ? K.nz - 1 : 0;
    }
    if (on_other_face(K, a, x, y, z)) return;  // edge and corner cells keep the streamed B
    double dsum = 0.0;
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if (b != a)
            dsum += axis_derivative(K, b, x, y, z, [&](int xx, int yy, int zz) { return streamed_B<TS>(src, K, b, xx, yy, zz); });
    const int s = high ? -1 : 1;
    const double inner = streamed_B<TS>(src, K, a, x + s * (a == 0), y + s * (a == 1), z + s * (a == 2));
    faceB[i] = high ? inner - K.dx * dsum : inner + K.dx * dsum;
}

template <typename TS>
__global__ __launch_bounds__(256) void k_face_b(const char* __restrict__ src, Consts K, double* __restrict__ faceB) {
    face_b_cell<TS>(src, K, faceB, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// The face pass of every instance of a batch in one launch.
template <typename TS>
__global__ __launch_bounds__(256) void k_face_b_batch(const BatchInst* __restrict__ I, int ninst, int64_t total,
                                                      int parity) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= total) return;
    const int i = find_instance(ninst, g, [&](int j) { return I[j].face0; });
    const BatchInst& B = I[i];
    if (!B.K.divb) return;
    face_b_cell<TS>(B.buf[parity], B.K, B.faceB, g - B.face0);
}

// Persistent batched run: nsteps steps in one cooperative launch whose grid
// (a multiple of 8) is no larger than the blocks resident at once.  The tiles
// of a step are dealt as k_fused_batch deals its blocks: XCD x (blocks g with
// g % 8 == x, as the hardware deals blocks to XCDs) runs the contiguous tile
// range [x P, (x + 1) P), and its blocks take the next tile of that range
// from a counter, in order and as they become free (each block takes its
// next one while its current one runs), so that the tiles in flight
// together stay neighbours.  next holds two sets of 8 counters, zero
// at launch: step k counts in set k % 2, and the first block of each group
// clears its counter of the other set (last used in step k - 1, whose fetches
// all ended before the barrier).  All blocks meet at a grid barrier after
// each step (the next one reads what it wrote).  No face pass: batches with
// the open-face adjustment are stepped by graph replays.  Every block reaches
// every barrier: no thread leaves the kernel early, and a fetch loop ends
// once its counter passes P.
template <bool NT, typename TS, typename TE, typename V, int PXT, int WV, bool FLAT>
__global__ __launch_bounds__(PTPB, WV) void k_fused_batch_persistent(const BatchInst* __restrict__ I, int ninst,
                                                                     int total, int parity0, int nsteps,
                                                                     int* __restrict__ next) {
    cooperative_groups::grid_group grid = cooperative_groups::this_grid();
    __shared__ int tile_sh;
    const int P = (total + 7) / 8;
    const int x = blockIdx.x % 8;
    for (int k = 0; k < nsteps; ++k) {
        const int parity = (parity0 + k) & 1;
        int* cnt = next + (k & 1) * 8 + x;
        if (blockIdx.x < 8 && threadIdx.x == 0) atomicExch(next + ((k + 1) & 1) * 8 + x, 0);
        // the next tile is taken while the current one runs, so the counter's round trip is hidden
        if (threadIdx.x == 0) tile_sh = atomicAdd(cnt, 1);
        __syncthreads();
        int j = tile_sh;
        __syncthreads();
        while (j < P) {  // j is uniform over the block
            int nj = 0;
            if (threadIdx.x == 0) nj = atomicAdd(cnt, 1);
            const int b = __builtin_amdgcn_readfirstlane(x * P + j);
            if (b < total) {
                const int i = find_instance(ninst, b, [&](int jj) { return I[jj].blk0; });
                const BatchInst& B = I[i];
                fused_block<NT, TS, TE, V, GUESS_NONE, PXT, 0, FLAT, false>(
                    B.buf[parity], B.buf[1 - parity], B.faceB, nullptr, (ConstsPtr)(uintptr_t)&B.K, B.tiles_x, B.ncol, B.zb, B.zt, 1, B.yw,
                    (int)(b - B.blk0));
            }
            if (threadIdx.x == 0) tile_sh = nj;
            __syncthreads();
            j = tile_sh;
            __syncthreads();
        }
        grid.sync();
    }
}

// Deterministic (key, index) minimum, ties to the lower index; NaN keys never win.
__device__ __forceinline__ void argmin_merge(double& k, double& i, double k2, double i2) {
    if (k2 < k || (k2 == k && i2 < i)) {
        k = k2;
        i = i2;
    }
}

__device__ __forceinline__ void block_argmin(double k, double i, double* __restrict__ out) {
    __shared__ double shk[RED_WAVES], shi[RED_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) argmin_merge(k, i, __shfl_xor(k, o, 64), __shfl_xor(i, o, 64));
    if (lane == 0) {
        shk[wave] = k;
        shi[wave] = i;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double bk = shk[0], bi = shi[0];
        for (int w = 1; w < RED_WAVES; ++w) argmin_merge(bk, bi, shk[w], shi[w]);
        out[0] = bk;
        out[1] = bi;
    }
}

constexpr double NO_INDEX = 9.0e15;  // larger than any cell index, exact in FP64

// Primitives of the current state and per-block partial diagnostics:
// part[blk * NPART + j], j = T00, N0, T0x, T0y, T0z, em energy, rho, iters,
// failed, then 16 Newton-iteration bins, then learned-guess fallbacks;
// null-search partials (least B_x^2 + B_y^2 in the band and its cell) in
// nullp[2 blk ..]; B and E^z of every cell into scratch (4 arrays of N).
// Every thread runs the cell pass (on the edge cell when past a ragged edge,
// so that the network sees whole wavefronts); only real cells write.
template <typename TS, typename TE, int GM>
__global__ __launch_bounds__(TPB, 2) void k_moments(const char* __restrict__ src, const double* __restrict__ faceB,
                                                 const GuessTables* __restrict__ gt, Consts K, int tiles_x,
                                                 int tiles_y, int ntiles, OutPtrs out, double* __restrict__ scratch,
                                                 double* __restrict__ part, double* __restrict__ nullp) {
    const int tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;  // uniform over the block
    const int tx = tile % tiles_x, rest = tile / tiles_x;
    const int ty = rest % tiles_y, z = rest / tiles_y;
    const int x0 = tx * TX + (threadIdx.x % TX), y0 = ty * TY + (threadIdx.x / TX);
    const bool active = x0 < K.nx && y0 < K.ny;
    const int x = min(x0, K.nx - 1), y = min(y0, K.ny - 1);
    double v[NPART] = {0};
    double key = __builtin_inf(), idx = NO_INDEX;
    const int cell = x + K.nx * (y + K.ny * z);
    const Nbr nb = make_nbr<true>(K, x, y, z);
    CellSol M;
    if constexpr (GM == GUESS_NONE)
        macroscopic<GM, TS, TE>(src, faceB, gt, K, cell, nb, x, y, z, M);
    else if (*K.gflag_rd == K.gstep - 1)  // the guess the next step would take
        macroscopic<GM, TS, TE>(src, faceB, gt, K, cell, nb, x, y, z, M);
    else
        macroscopic<GUESS_MONITOR, TS, TE>(src, faceB, gt, K, cell, nb, x, y, z, M);
    if (active) {
        const double c = K.c;
        if (out.n) out.n[cell] = M.n;
        if (out.p) out.p[cell] = M.p;
        if (out.eps) out.eps[cell] = M.eps;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (out.u[a]) out.u[a][cell] = c * M.beta[a];
            if (out.E[a]) out.E[a][cell] = M.E[a];
            if (out.B[a]) out.B[a][cell] = M.B[a];
            if (out.J[a]) out.J[a][cell] = M.J[a];
            scratch[(int64_t)a * K.N + cell] = M.B[a];
        }
        scratch[3 * K.N + cell] = M.E[2];
        if (out.rho_c) out.rho_c[cell] = M.rho;
        v[0] = M.T00;
        v[1] = M.N0;
        v[2] = M.T0[0];
        v[3] = M.T0[1];
        v[4] = M.T0[2];
        const double E2 = M.E[0] * M.E[0] + M.E[1] * M.E[1] + M.E[2] * M.E[2];
        const double B2 = M.B[0] * M.B[0] + M.B[1] * M.B[1] + M.B[2] * M.B[2];
        v[5] = 0.5 * K.eps0 * (E2 + c * c * B2);
        v[6] = M.rho;
        v[7] = M.iters;
        v[8] = M.ok ? 0.0 : 1.0;
        const int bin = M.iters < 15 ? (M.iters > 0 ? M.iters : 0) : 15;
#pragma unroll
        for (int k = 0; k < 16; ++k) v[9 + k] = bin == k ? 1.0 : 0.0;
        v[25] = M.fallback;
        // |y_j| <= band with cell centres y_j = j + 1/2 - ny/2
        const int dy = 2 * y + 1 - K.ny;
        if ((dy < 0 ? -dy : dy) <= 2 * K.band) {
            const double kb = fma(M.B[0], M.B[0], M.B[1] * M.B[1]);
            if (kb == kb) {
                key = kb;
                idx = (double)cell;
            }
        }
    }
    block_sum<NPART>(v, part + (int64_t)tile * NPART);
    block_argmin(key, idx, nullp + 2 * (int64_t)tile);
}

// max |div B| per block from the B written by k_moments (the derivative
// operator of the normal-B adjustment).
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_divb(const double* __restrict__ Bs, Consts K, int tiles_x, int tiles_y,
                                              int ntiles, double* __restrict__ part) {
    const int tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;
    const int tx = tile % tiles_x, rest = tile / tiles_x;
    const int ty = rest % tiles_y, z = rest / tiles_y;
    const int x = tx * TX + (threadIdx.x % TX), y = ty * TY + (threadIdx.x / TX);
    double v[1] = {0.0};
    if (x < K.nx && y < K.ny) {
        double dv = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double* Ba = Bs + (int64_t)a * K.N;
            dv += axis_derivative(K, a, x, y, z, [&](int xx, int yy, int zz) { return Ba[xx + K.nx * (yy + K.ny * zz)]; });
        }
        v[0] = fabs(dv);
    }
    block_max1(v[0], part + tile);
}

// Null point over the per-block partials, then R = (E^z - E^z_0) / B0 there.
// out[0] = R, out[1] = null cell (-1: none), out[2] = B0.
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_null_reduce(const double* __restrict__ nullp, int nblk,
                                                     const double* __restrict__ ez, const double* __restrict__ ez0,
                                                     const double* __restrict__ b0, double* __restrict__ out) {
    __shared__ double res[2];
    double k = __builtin_inf(), i = NO_INDEX;
    int b = threadIdx.x;
    for (; b + 7 * TPB < nblk; b += 8 * TPB) {  // 8 candidates of a thread in flight
        vec2<double> v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const vec2<double>*>(nullp + 2 * (int64_t)(b + u * TPB));
#pragma unroll
        for (int u = 0; u < 8; ++u) argmin_merge(k, i, v[u].x, v[u].y);
    }
    for (; b < nblk; b += TPB) argmin_merge(k, i, nullp[2 * (int64_t)b], nullp[2 * (int64_t)b + 1]);
    block_argmin(k, i, res);
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool found = res[1] < NO_INDEX;
        const int64_t c = found ? (int64_t)res[1] : -1;
        out[0] = found ? (ez[c] - ez0[c]) / b0[0] : __builtin_nan("");
        out[1] = (double)c;
        out[2] = b0[0];
    }
}

// Largest |beta| of a forced step from its per-wavefront partials (which are
// cleared for the next step); one block.
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_vmax_reduce(double* __restrict__ part, int64_t n, double* __restrict__ out) {
    double m = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 15 * TPB < n; i += 16 * TPB) {  // 16 partials of a thread in flight
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = part[i + u * TPB];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            m = fmax(m, v[u]);
            part[i + u * TPB] = 0.0;
        }
    }
    for (; i < n; i += TPB) {
        m = fmax(m, part[i]);
        part[i] = 0.0;
    }
    __shared__ double sh[TPB / 64];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = sh[0];
        for (int w = 1; w < TPB / 64; ++w) r = fmax(r, sh[w]);
        *out = r;
    }
}

// Fixed-order reduction of the per-block partials, one column of them per block.
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_reduce(const double* __restrict__ part, int nblk, int width,
                                                                        int is_max, double* __restrict__ out) {
    const int j = blockIdx.x;  // one column per block; 16 rows of a thread in flight, added in order
    double acc = 0.0;
    int b = threadIdx.x;
    for (; b + 15 * TPB < nblk; b += 16 * TPB) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)(b + u * TPB) * width + j];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc = is_max ? fmax(acc, v[u]) : acc + v[u];
    }
    for (; b < nblk; b += TPB) {
        const double v = part[(int64_t)b * width + j];
        acc = is_max ? fmax(acc, v) : acc + v;
    }
    const double r = is_max ? block_max_value(acc) : block_sum_value(acc);
    if (threadIdx.x == 0) out[j] = is_max == 2 ? sqrt(r) : r;
}

// Sums of eps = n c^2 + p / (Gamma - 1) and n over the initial fields (the
// references of the stored deviations).
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_init_ref(InPtrs in, Consts K, double* __restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    double v[2] = {0.0, 0.0};
    if (i < K.N) {
        v[0] = in.n[i] * K.c * K.c + in.p[i] / K.gm1;
        v[1] = in.n[i];
    }
    block_sum<2>(v, part + (int64_t)blockIdx.x * 2);
}

// Face cells with |u| >= c, n <= 0 or p < 0, per block.
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_face_check(FacePtrs in, Consts K, double* __restrict__ part) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    double bad[1] = {0.0};
    if (i < (int64_t)K.nx * K.ny) {
        const double u2 = in.u[0][i] * in.u[0][i] + in.u[1][i] * in.u[1][i] + in.u[2][i] * in.u[2][i];
        bad[0] = (u2 < K.c * K.c && in.n[i] > 0.0 && in.p[i] >= 0.0) ? 0.0 : 1.0;
    }
    block_sum<1>(bad, part + blockIdx.x);
}

// Ghost planes of a driven low-z face: the post-collision state of a fully
// relaxed cell with the prescribed fields -- f_eq and g_eq of (n, p, u,
// E = -u x B, B) (stored minus their shifts), h* = h_eq of (J, E + q J, B)
// with J of Eq. Ohm at zero charge (h* = h_eq is the fixed point of the
// tau_h = 1/2 collision), rest h* = 0 and E_prev = E; both planes the same.
// The planes sit just below cell 0 of the state buffer.
template <typename TS, typename TE>
__global__ __launch_bounds__(TPB) void k_init_ghost(FacePtrs in, Consts K, char* __restrict__ dd) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    const int64_t plane = (int64_t)K.nx * K.ny;
    if (i >= plane) return;
    const double c = K.c, c2 = c * c;
    double u[3], Bv[3], beta[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        u[a] = in.u[a][i];
        Bv[a] = in.B[a][i];
        beta[a] = u[a] / c;
    }
    const double E[3] = {-(u[1] * Bv[2] - u[2] * Bv[1]), -(u[2] * Bv[0] - u[0] * Bv[2]), -(u[0] * Bv[1] - u[1] * Bv[0])};
    const double n = in.n[i], p = in.p[i];
    const double b2 = beta[0] * beta[0] + beta[1] * beta[1] + beta[2] * beta[2];
    const double gam = 1.0 / sqrt(1.0 - b2);
    const double eps = n * c2 + p / K.gm1;
    const double uxB[3] = {u[1] * Bv[2] - u[2] * Bv[1], u[2] * Bv[0] - u[0] * Bv[2], u[0] * Bv[1] - u[1] * Bv[0]};
    const double Eu = (E[0] * u[0] + E[1] * u[1] + E[2] * u[2]) / c2;
    double J[3], Epr[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        J[a] = K.sigma * gam * (E[a] + uxB[a] - Eu * u[a]);
        Epr[a] = E[a] + K.q * J[a];
    }
    FeqCell fe;
    fe.setup(eps, p, gam, beta, E, Bv, c, K.eps0);
    const double cj = 1.0 / (16.0 * 1.4142135623730951 * c), ce = 1.0 / (8.0 * 1.4142135623730951 * c);
    for (int layer = 1; layer <= 2; ++layer) {
        const int g = (int)K.g0 + (int)(i - layer * plane);  // position of the ghost cell
        static_for<0>([&](auto ic) {
            constexpr int q = decltype(ic)::value;
            const double eb = EX[q] * beta[0] + EY[q] * beta[1] + EZ[q] * beta[2];
            const double wpi = q == 0 ? K.wp[0] : (q <= 6 ? K.wp[1] : K.wp[2]);
            st2<false, TS>(dd, f_at<TS>(K, q, g), fe.template eq<q>() - fshift(K, q),
                           wpi * n * gam * (1.0 + K.gc1 * eb + K.gc2 * eb * eb - K.gc3 * b2) - gshift(K, q));
        });
#pragma unroll
        for (int k = 0; k < QH; ++k) {
            const double heq = cj * (SX[k] * J[0] + SY[k] * J[1] + SZ[k] * J[2]) +
                               ce * (EHX[k] * Epr[0] + EHY[k] * Epr[1] + EHZ[k] * Epr[2]) +
                               0.125 * (BHX[k] * Bv[0] + BHY[k] * Bv[1] + BHZ[k] * Bv[2]);
            st<false, TS>(dd, h_at<TS>(K, k, g), heq);
        }
        st<false, TS>(dd, h_at<TS>(K, QH, g), 0.0);
#pragma unroll
        for (int a = 0; a < 3; ++a) st<false, TE>(dd, e_at<TS>(K, a, g), E[a]);
        if (K.bprev)
#pragma unroll
            for (int a = 0; a < 3; ++a) st<false, TE>(dd, e_at<TS>(K, 3 + a, g), Bv[a]);
    }
}

// Initial state, pass 1: J0 from Eq. Ohm with the Gauss charge of E0, and
// E'0 = E0 + (dt/2) mu0 c^2 J0 (Reading of the initial h), into scratch.
// Also the references of the reconnection rate: E^z_0, and the largest B^2 per
// tile (as fma(B_x, B_x, fma(B_y, B_y, B_z B_z))).
[[maybe_unused]] static __global__ __launch_bounds__(TPB) void k_init_current(InPtrs in, Consts K, int tiles_x, int tiles_y, int ntiles,
                                                      double* __restrict__ scr, double* __restrict__ ez0,
                                                      double* __restrict__ part) {
    const int tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;
    const int tx = tile % tiles_x, rest = tile / tiles_x;
    const int ty = rest % tiles_y, z = rest / tiles_y;
    const int x = tx * TX + (threadIdx.x % TX), y = ty * TY + (threadIdx.x / TX);
    double b2max = 0.0;
    if (x < K.nx && y < K.ny) {
        const int cell = x + K.nx * (y + K.ny * z);
        const Nbr nb = make_nbr<false>(K, x, y, z);
        const double c = K.c, c2 = c * c;
        double u[3], E[3], B[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u[a] = in.u[a][cell];
            E[a] = in.E[a][cell];
            B[a] = in.B[a][cell];
        }
        const double rg = K.eps0 * K.inv_2dx *
                          ((in.E[0][cell + nb.at(1, 0, 0)] - in.E[0][cell + nb.at(-1, 0, 0)]) +
                           (in.E[1][cell + nb.at(0, 1, 0)] - in.E[1][cell + nb.at(0, -1, 0)]) +
                           (in.E[2][cell + nb.at(0, 0, 1)] - in.E[2][cell + nb.at(0, 0, -1)]));
        const double gam = 1.0 / sqrt(1.0 - (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]) / c2);
        const double uxB[3] = {u[1] * B[2] - u[2] * B[1], u[2] * B[0] - u[0] * B[2], u[0] * B[1] - u[1] * B[0]};
        const double Eu = (E[0] * u[0] + E[1] * u[1] + E[2] * u[2]) / c2;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double J = K.sigma * gam * (E[a] + uxB[a] - Eu * u[a]) + rg * u[a];
            scr[(int64_t)a * K.N + cell] = J;
            scr[(int64_t)(3 + a) * K.N + cell] = E[a] + K.q * J;
        }
        ez0[cell] = E[2];
        b2max = fma(B[0], B[0], fma(B[1], B[1], B[2] * B[2]));
    }
    block_max1(b2max, part + tile);
}

// Initial state, pass 2: f* = f_eq, g* = g_eq (stored minus their shifts),
// h*_k(x) = h_eq-form at x + s_k, h*_rest = rho_c, E_prev = E0.
template <typename TS, typename TE>
__global__ __launch_bounds__(TPB) void k_init_state(InPtrs in, Consts K, int tiles_x, int tiles_y, int ntiles,
                                                    const double* __restrict__ scr, char* __restrict__ dst) {
    const int tile = tile_of_block(ntiles);
    if (tile >= ntiles) return;
    const int tx = tile % tiles_x, rest = tile / tiles_x;
    const int ty = rest % tiles_y, z = rest / tiles_y;
    const int x = tx * TX + (threadIdx.x % TX), y = ty * TY + (threadIdx.x / TX);
    if (x >= K.nx || y >= K.ny) return;
    const int cell = x + K.nx * (y + K.ny * z);
    const Nbr nb = make_nbr<false>(K, x, y, z);
    const double c = K.c, c2 = c * c;
    double u[3], Ep[3], Bv[3], beta[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        u[a] = in.u[a][cell];
        Ep[a] = in.E[a][cell];
        Bv[a] = in.B[a][cell];
        beta[a] = u[a] / c;
    }
    const int pos = (int)K.g0 + cell;
    const double n = in.n[cell], p = in.p[cell];
    const double b2 = beta[0] * beta[0] + beta[1] * beta[1] + beta[2] * beta[2];
    const double gam = 1.0 / sqrt(1.0 - b2);
    const double eps = n * c2 + p / K.gm1;
    FeqCell fe;
    fe.setup(eps, p, gam, beta, Ep, Bv, c, K.eps0);
    // rest value of h*, written with the rest pair in the quad layouts
    double rho;
    if (in.rho_c) {
        rho = in.rho_c[cell];
    } else {
        rho = K.eps0 * K.inv_2dx *
              ((in.E[0][cell + nb.at(1, 0, 0)] - in.E[0][cell + nb.at(-1, 0, 0)]) +
               (in.E[1][cell + nb.at(0, 1, 0)] - in.E[1][cell + nb.at(0, -1, 0)]) +
               (in.E[2][cell + nb.at(0, 0, 1)] - in.E[2][cell + nb.at(0, 0, -1)]));
    }
    auto fg = [&](auto ic, double& f, double& g) {
        constexpr int i = decltype(ic)::value;
        const double eb = EX[i] * beta[0] + EY[i] * beta[1] + EZ[i] * beta[2];
        const double wpi = i == 0 ? K.wp[0] : (i <= 6 ? K.wp[1] : K.wp[2]);
        f = fe.template eq<i>() - fshift(K, i);
        g = wpi * n * gam * (1.0 + K.gc1 * eb + K.gc2 * eb * eb - K.gc3 * b2) - gshift(K, i);
    };
    static_for<0>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (!quad_layout<TS>()) {
            double f, g;
            fg(ic, f, g);
            st2<true, TS>(dst, f_at<TS>(K, i, pos), f, g);
        } else if constexpr (i == 0 || (i & 1)) {  // the record half of directions i, i + 1 (or the rest quad)
            vec4<double> v;
            double f, g;
            fg(ic, f, g);
            v.x = f, v.y = g;
            if constexpr (i == 0) {
                v.z = rho, v.w = 0.0;
            } else {
                fg(std::integral_constant<int, i + 1>{}, f, g);
                v.z = f, v.w = g;
            }
            st4<true, TS>(dst, f_at<TS>(K, i, pos), v);
        }
    });
    const double cj = 1.0 / (16.0 * 1.4142135623730951 * c), ce = 1.0 / (8.0 * 1.4142135623730951 * c);
    // the populations 2m and 2m + 1 go to the same cell
#pragma unroll
    for (int m = 0; m < QH / 2; ++m) {
        const int t = cell + nb.at(SX[2 * m], SY[2 * m], SZ[2 * m]);
        const double J0 = scr[t], J1 = scr[K.N + t], J2 = scr[2 * K.N + t];
        const double P0 = scr[3 * K.N + t], P1 = scr[4 * K.N + t], P2 = scr[5 * K.N + t];
        const double B0 = in.B[0][t], B1 = in.B[1][t], B2 = in.B[2][t];
        double heq[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int k = 2 * m + j;
            heq[j] = cj * (SX[k] * J0 + SY[k] * J1 + SZ[k] * J2) + ce * (EHX[k] * P0 + EHY[k] * P1 + EHZ[k] * P2) +
                     0.125 * (BHX[k] * B0 + BHY[k] * B1 + BHZ[k] * B2);
        }
        if constexpr (quad_layout<TS>()) {
            st2<true, TS>(dst, h_at<TS>(K, 2 * m, pos), heq[0], heq[1]);
        } else {
            st<true, TS>(dst, h_at<TS>(K, 2 * m, pos), heq[0]);
            st<true, TS>(dst, h_at<TS>(K, 2 * m + 1, pos), heq[1]);
        }
    }
    if constexpr (!quad_layout<TS>()) st<true, TS>(dst, h_at<TS>(K, QH, pos), rho);
#pragma unroll
    for (int a = 0; a < 3; ++a) st<true, TE>(dst, e_at<TS>(K, a, pos), Ep[a]);
    if (K.bprev)
#pragma unroll
        for (int a = 0; a < 3; ++a) st<true, TE>(dst, e_at<TS>(K, 3 + a, pos), Bv[a]);
}

// Raw state conversion to / from the FP64 interface layout (shifts added
// back) by whole records of a cell, so every line of the state is touched once
// (with one thread per value each f-g record was visited twice, and export and
// import of 256x256x64 cells in FP64 took 1.07 and 1.66 ms; so 0.80 and 0.76).
// Record r of a cell: the f-g records, then the Maxwell ones, then E_prev
// (and B_prev) value by value.
template <typename TS>
constexpr int FG_RECORDS = quad_layout<TS>() ? 10 : Q;
template <typename TS>
__host__ __device__ inline int state_records(const Consts& K) {
    return FG_RECORDS<TS> + Lay<TS>::HRECORDS + state_arrays(K) - OFF_E;
}
template <typename TS, typename TE, typename Put>
__device__ __forceinline__ void export_record(const char* __restrict__ s, const Consts& K, int r, int pos, Put&& put) {
    constexpr int NF = FG_RECORDS<TS>, NH = Lay<TS>::HRECORDS;
    auto put_fg = [&](int i, double f, double g) {
        put(OFF_F + i, f + fshift(K, i));
        put(OFF_G + i, g + gshift(K, i));
    };
    if (r < NF) {
        if constexpr (quad_layout<TS>()) {
            const int i0 = r == 0 ? 0 : 2 * r - 1;
            const vec4<double> v = ldv4<double, TS>(s, f_at<TS>(K, i0, pos));
            put_fg(i0, v.x, v.y);
            if (r == 0)
                put(OFF_H + QH, v.z);
            else
                put_fg(i0 + 1, v.z, v.w);
        } else {
            const vec2<double> v = ldv2<double, TS>(s, f_at<TS>(K, r, pos));
            put_fg(r, v.x, v.y);
        }
    } else if (r < NF + NH) {
        if constexpr (quad_layout<TS>()) {
            const int k = 2 * (r - NF);
            const vec2<double> v = ldv2<double, TS>(s, h_at<TS>(K, k, pos));
            put(OFF_H + k, v.x);
            put(OFF_H + k + 1, v.y);
        } else {
            put(OFF_H + r - NF, ld<TS>(s, h_at<TS>(K, r - NF, pos)));
        }
    } else {
        put(OFF_E + r - NF - NH, ld<TE>(s, e_at<TS>(K, r - NF - NH, pos)));
    }
}
template <typename TS, typename TE, typename Get>
__device__ __forceinline__ void import_record(char* __restrict__ d, const Consts& K, int r, int pos, Get&& get) {
    constexpr int NF = FG_RECORDS<TS>, NH = Lay<TS>::HRECORDS;
    auto get_f = [&](int i) { return get(OFF_F + i) - fshift(K, i); };
    auto get_g = [&](int i) { return get(OFF_G + i) - gshift(K, i); };
    if (r < NF) {
        if constexpr (quad_layout<TS>()) {
            const int i0 = r == 0 ? 0 : 2 * r - 1;
            vec4<double> v;
            v.x = get_f(i0);
            v.y = get_g(i0);
            v.z = r == 0 ? get(OFF_H + QH) : get_f(i0 + 1);
            v.w = r == 0 ? 0.0 : get_g(i0 + 1);
            st4<true, TS>(d, f_at<TS>(K, i0, pos), v);
        } else {
            st2<true, TS>(d, f_at<TS>(K, r, pos), get_f(r), get_g(r));
        }
    } else if (r < NF + NH) {
        if constexpr (quad_layout<TS>()) {
            const int k = 2 * (r - NF);
            st2<true, TS>(d, h_at<TS>(K, k, pos), get(OFF_H + k), get(OFF_H + k + 1));
        } else {
            st<true, TS>(d, h_at<TS>(K, r - NF, pos), get(OFF_H + r - NF));
        }
    } else {
        st<true, TE>(d, e_at<TS>(K, r - NF - NH, pos), get(OFF_E + r - NF - NH));
    }
}
// One thread per cell, or (EACH) per record of a cell, record blockIdx.y: see record_threads.
template <typename TS, typename TE, bool EACH>
__global__ __launch_bounds__(256) void k_export(const char* __restrict__ s, double* __restrict__ d, Consts K) {
    const int64_t cell = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (cell >= K.N) return;
    const int pos = (int)K.g0 + (int)cell;
    auto put = [&](int a, double v) { __builtin_nontemporal_store(v, d + a * K.N + cell); };
    if constexpr (EACH) {
        export_record<TS, TE>(s, K, blockIdx.y, pos, put);
    } else {
        constexpr int N = FG_RECORDS<TS> + Lay<TS>::HRECORDS + 3;
#pragma unroll
        for (int r = 0; r < N; ++r) export_record<TS, TE>(s, K, r, pos, put);
        for (int r = N; r < state_records<TS>(K); ++r) export_record<TS, TE>(s, K, r, pos, put);
    }
}

template <typename TS, typename TE, bool EACH>
__global__ __launch_bounds__(256) void k_import(const double* __restrict__ s, char* __restrict__ d, Consts K) {
    const int64_t cell = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (cell >= K.N) return;
    const int pos = (int)K.g0 + (int)cell;
    auto get = [&](int a) { return __builtin_nontemporal_load(s + a * K.N + cell); };
    if constexpr (EACH) {
        import_record<TS, TE>(d, K, blockIdx.y, pos, get);
    } else {
        constexpr int N = FG_RECORDS<TS> + Lay<TS>::HRECORDS + 3;
#pragma unroll
        for (int r = 0; r < N; ++r) import_record<TS, TE>(d, K, r, pos, get);
        for (int r = N; r < state_records<TS>(K); ++r) import_record<TS, TE>(d, K, r, pos, get);
    }
}

// (features, targets) of sampled cells of the current state with the plain
// recovery: cell floor(i N / ns) for sample i.  F: ns x 6, T: ns x 2 (FP64).
// Per-block partial sums of F, F^2, T, T^2 and failed cells into part (17 per block).

template <typename TS, typename TE>
__global__ __launch_bounds__(256) void k_guess_samples(const char* __restrict__ src,
                                                       const double* __restrict__ faceB, Consts K, int ns,
                                                       double* __restrict__ F, double* __restrict__ T,
                                                       double* __restrict__ part) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    double acc[SAMPLE_SUMS] = {0};
    if (i < ns) {
        const int64_t cell = (int64_t)i * K.N / ns;
        const int x = (int)(cell % K.nx), y = (int)((cell / K.nx) % K.ny), z = (int)(cell / ((int64_t)K.nx * K.ny));
        const Nbr nb = make_nbr<true>(K, x, y, z);
        CellSol M;
        macroscopic<GUESS_NONE, TS, TE>(src, faceB, nullptr, K, (int)cell, nb, x, y, z, M);
        double Ef, S[3], Pi[6];
        fluid_tensor(K, M, M.B, Ef, S, Pi);  // the guess is not offered with the previous-B reading
        double f[6], sn;
        f[0] = flow_ratio(Ef, S, sn);
        mlp_features(Ef, S, Pi, M.N0, sn, f);
        const double t0 = M.eps / Ef;
        const double t1 = sqrt(M.beta[0] * M.beta[0] + M.beta[1] * M.beta[1] + M.beta[2] * M.beta[2]);
        if (M.ok) {
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                F[(int64_t)i * 6 + j] = f[j];
                acc[j] = f[j];
                acc[6 + j] = f[j] * f[j];
            }
            T[(int64_t)i * 2] = t0;
            T[(int64_t)i * 2 + 1] = t1;
            acc[12] = t0;
            acc[13] = t1;
            acc[14] = t0 * t0;
            acc[15] = t1 * t1;
        } else {
            acc[16] = 1.0;
        }
    }
    block_sum<SAMPLE_SUMS>(acc, part + (int64_t)blockIdx.x * SAMPLE_SUMS);
}

// Plain copy of n 16-byte words, four per lane in flight, with the non-temporal
// hints of the step's streamed loads and stores (the reference rate of HBM).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
[[maybe_unused]] static __global__ __launch_bounds__(256) void k_copy16(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int64_t n) {
    const int64_t base = (int64_t)blockIdx.x * (256 * 4) + threadIdx.x;
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = base + (int64_t)u * 256;
        if (i < n) v[u] = __builtin_nontemporal_load(src + i);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = base + (int64_t)u * 256;
        if (i < n) __builtin_nontemporal_store(v[u], dst + i);
    }
}

// ------------------------------------------------------------ host launchers

#if RMHDLB_FORM == 64  // what depends on no storage form is built once
hipError_t launch_copy16(const void* src, void* dst, int64_t n16, hipStream_t s) {
    const int64_t blocks = (n16 + 1023) / 1024;
    if (blocks > 0)
        hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, s, (const u32x4*)src, (u32x4*)dst, n16);
    return hipGetLastError();
}
#endif

static inline void grid_of(const Consts& K, int& tiles_x, int& tiles_y, int& ntiles, int& nblocks) {
    tiles_x = (K.nx + TX - 1) / TX;
    tiles_y = (K.ny + TY - 1) / TY;
    ntiles = tiles_x * tiles_y * K.nz;
    nblocks = ((ntiles + 7) / 8) * 8;
}

#if RMHDLB_FORM == 64  // what depends on no storage form is built once
int num_tiles(const Consts& K) {
    int a, b, n, nb;
    grid_of(K, a, b, n, nb);
    return n;
}
#endif

template <typename TS>
hipError_t launch_face_b(const char* src, const Consts& K, double* faceB, hipStream_t s) {
    if (!K.divb) return hipSuccess;
    const int64_t blocks = (K.fo[6] + 255) / 256;
    hipLaunchKernelGGL((k_face_b<TS>), dim3((unsigned)blocks), dim3(256), 0, s, src, K, faceB);
    return hipGetLastError();
}

#if RMHDLB_FORM == 64  // what depends on no storage form is built once
void step_geometry(const Consts& K, int px, const StepWalk& w, int zg, int yw, int elem, int& tiles_x, int& ncol,
                   int& nblk) {
    const int py = cells_per_block(elem) / px / w.zt * yw;
    tiles_x = (K.nx + px - 1) / px;
    ncol = tiles_x * ((K.ny + py - 1) / py);
    nblk = ncol * zg * ((K.nz + zg * w.zb - 1) / (zg * w.zb));
}
#endif

template <typename TS, int GM, int PXT, int VR = 0>
static void launch_fused(const char* sd, char* dd, double* faceB, const GuessTables* gt, const Consts& K, int zb, int zg, int yw, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    using V = typename StoreTypes<TS>::V;
    int tx, ncol, nblk;
    const StepWalk w = step_walk(K, PXT, zb, sizeof(TS), flat_grid(K), plane_blocks(K, PXT, yw, sizeof(TS)));
    step_geometry(K, PXT, w, zg, yw, sizeof(TS), tx, ncol, nblk);
    const int grid = ((nblk + 7) / 8) * 8;
    if (flat_grid(K))
        hipLaunchKernelGGL((k_fused_step<true, TS, TE, V, GM, PXT, VR, true>), dim3(grid), dim3(PTPB), 0, s, sd, dd,
                           (const double*)faceB, gt, K, tx, ncol, w.zb, w.zt, zg, yw, nblk);
    else
        hipLaunchKernelGGL((k_fused_step<true, TS, TE, V, GM, PXT, VR, false>), dim3(grid), dim3(PTPB), 0, s, sd, dd,
                           (const double*)faceB, gt, K, tx, ncol, w.zb, w.zt, zg, yw, nblk);
}

template <typename TS>
hipError_t launch_step(const char* src, char* dst, const Consts& K, const StepTuning& tune,
                       double* faceB, const GuessTables* gt, hipStream_t s) {
    hipError_t e = launch_face_b<TS>(src, K, faceB, s);
    if (e != hipSuccess) return e;
    const int zb = tune.zb;
    // interleaved walks: zg blocks per column and chunk (the force path keeps
    // zg = 1, the geometry its per-wavefront maxima are sized for)
    const int zg = (tune.zg > 1 && !K.forced) ? tune.zg : 1;
    const int vr = (K.coll ? 1 : 0) | (K.flux ? 2 : 0);
    const int yw = tune.yw > 1 && !K.forced ? tune.yw : 1;  // the force's partial maxima are sized for yw = 1
    if (K.bprev) {  // the previous-B reading: 64-wide tiles, default collision and faces, no guess or force
        if (gt || vr || K.forced) return hipErrorNotSupported;
        launch_fused<TS, GUESS_NONE, 64, 8>(src, dst, faceB, gt, K, zb, zg, yw, s);
    } else if (K.forced) {  // the external force: 64-wide tiles, MUSCL faces, no guess
        if (gt || K.flux) return hipErrorNotSupported;
        if (K.coll)
            launch_fused<TS, GUESS_NONE, 64, 5>(src, dst, faceB, gt, K, zb, 1, 1, s);
        else
            launch_fused<TS, GUESS_NONE, 64, 4>(src, dst, faceB, gt, K, zb, 1, 1, s);
        int tx, ncol, nblk;
        const StepWalk w = step_walk(K, 64, zb, sizeof(TS), flat_grid(K), plane_blocks(K, 64, 1, sizeof(TS)));
        step_geometry(K, 64, w, 1, 1, sizeof(TS), tx, ncol, nblk);
        hipLaunchKernelGGL(k_vmax_reduce, dim3(1), dim3(TPB), 0, s, K.vmax_part, (int64_t)nblk * (PTPB / 64),
                           const_cast<double*>(K.vmax_prev));
    } else if (vr) {  // the alternative readings: 64-wide tiles, no guess
        if (gt) return hipErrorNotSupported;
        if (vr == 1)
            launch_fused<TS, GUESS_NONE, 64, 1>(src, dst, faceB, gt, K, zb, zg, yw, s);
        else if (vr == 2)
            launch_fused<TS, GUESS_NONE, 64, 2>(src, dst, faceB, gt, K, zb, zg, yw, s);
        else
            launch_fused<TS, GUESS_NONE, 64, 3>(src, dst, faceB, gt, K, zb, zg, yw, s);
    } else if (gt) {  // the guess path is built for 64-wide tiles only; one cell per lane in the quad layout
        if constexpr (quad_layout<TS>())
            launch_fused<TS, GUESS_SINGLE, 64>(src, dst, faceB, gt, K, zb, zg, yw, s);
        else
            launch_fused<TS, GUESS_PAIR, 64>(src, dst, faceB, gt, K, zb, zg, yw, s);
        launch_fused<TS, GUESS_MONITOR, 64>(src, dst, faceB, gt, K, zb, zg, yw, s);
    }
    else if (tune.px == 32)
        launch_fused<TS, GUESS_NONE, 32>(src, dst, faceB, gt, K, zb, zg, yw, s);
    else if (tune.px == 16)
        launch_fused<TS, GUESS_NONE, 16>(src, dst, faceB, gt, K, zb, zg, yw, s);
    else
        launch_fused<TS, GUESS_NONE, 64>(src, dst, faceB, gt, K, zb, zg, yw, s);
    return hipGetLastError();
}

template <typename TS, int PXT, int WV>
static void launch_batch_fused(const BatchInst* dev, int ninst, int total_blocks, bool flat, int parity,
                               hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    using V = typename StoreTypes<TS>::V;
    const int grid = ((total_blocks + 7) / 8) * 8;
    if (flat)
        hipLaunchKernelGGL((k_fused_batch<true, TS, TE, V, PXT, WV, true>), dim3(grid), dim3(PTPB), 0, s, dev, ninst,
                           total_blocks, parity);
    else
        hipLaunchKernelGGL((k_fused_batch<true, TS, TE, V, PXT, WV, false>), dim3(grid), dim3(PTPB), 0, s, dev, ninst,
                           total_blocks, parity);
}

template <typename TS, int WV>
static void launch_batch_px(const BatchInst* dev, int ninst, int total_blocks, bool flat, int px, int parity,
                            hipStream_t s) {
    if (px == 128)
        launch_batch_fused<TS, 128, WV>(dev, ninst, total_blocks, flat, parity, s);
    else if (px == 32)
        launch_batch_fused<TS, 32, WV>(dev, ninst, total_blocks, flat, parity, s);
    else if (px == 16)
        launch_batch_fused<TS, 16, WV>(dev, ninst, total_blocks, flat, parity, s);
    else
        launch_batch_fused<TS, 64, WV>(dev, ninst, total_blocks, flat, parity, s);
}

template <typename TS>
hipError_t launch_batch(const BatchInst* dev, int ninst, int total_blocks, int64_t total_face, bool flat, int px,
                        int waves, int parity, hipStream_t s) {
    if (total_face > 0)
        hipLaunchKernelGGL((k_face_b_batch<TS>), dim3((unsigned)((total_face + 255) / 256)), dim3(256), 0, s, dev,
                           ninst, total_face, parity);
    // FP32 storage (the sweep's) is built for two and three waves per SIMD;
    // FP64 and FP16 for their single-instance counts
    if constexpr (sizeof(TS) == 4) {
        if (waves == 3)
            launch_batch_px<TS, 3>(dev, ninst, total_blocks, flat, px, parity, s);
        else
            launch_batch_px<TS, 2>(dev, ninst, total_blocks, flat, px, parity, s);
    } else {
        launch_batch_px<TS, FUSED_WAVES>(dev, ninst, total_blocks, flat, px, parity, s);
    }
    return hipGetLastError();
}

// Clears the persistent run's 16 tile counters (a kernel, not a memset node,
// should a caller capture the step).
[[maybe_unused]] static __global__ void k_zero16(int* __restrict__ p) {
    if (threadIdx.x < 16) p[threadIdx.x] = 0;
}

// The persistent run's grid: the blocks resident at once (occupancy of this
// instantiation times the compute units), rounded down to a multiple of 8 and
// at most the rounded tile range.  The cooperative launch refuses a grid that
// cannot be resident as a whole, so the grid barriers always complete.
template <typename TS, int PXT, int WV>
static hipError_t launch_persistent_fused(const BatchInst* dev, int ninst, int total_blocks, bool flat, int parity,
                                          int nsteps, int* next, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    using V = typename StoreTypes<TS>::V;
    const void* kern = flat ? reinterpret_cast<const void*>(&k_fused_batch_persistent<true, TS, TE, V, PXT, WV, true>)
                            : reinterpret_cast<const void*>(&k_fused_batch_persistent<true, TS, TE, V, PXT, WV, false>);
    int dev_id = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev_id);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev_id);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, PTPB, 0);
    if (e != hipSuccess) return e;
    const int range = (total_blocks + 7) / 8 * 8;
    const int resident = per_cu * cus / 8 * 8;
    const int grid = resident < range ? resident : range;
    if (grid < 8) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_zero16, dim3(1), dim3(64), 0, s, next);
    void* args[] = {(void*)&dev, (void*)&ninst, (void*)&total_blocks, (void*)&parity, (void*)&nsteps,
                    (void*)&next};
    return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(PTPB), args, 0, s);
}

template <typename TS, int WV>
static hipError_t launch_persistent_px(const BatchInst* dev, int ninst, int total_blocks, bool flat, int px,
                                       int parity, int nsteps, int* next, hipStream_t s) {
    if (px == 128)
        return launch_persistent_fused<TS, 128, WV>(dev, ninst, total_blocks, flat, parity, nsteps, next, s);
    if (px == 32)
        return launch_persistent_fused<TS, 32, WV>(dev, ninst, total_blocks, flat, parity, nsteps, next, s);
    if (px == 16)
        return launch_persistent_fused<TS, 16, WV>(dev, ninst, total_blocks, flat, parity, nsteps, next, s);
    return launch_persistent_fused<TS, 64, WV>(dev, ninst, total_blocks, flat, parity, nsteps, next, s);
}

template <typename TS>
hipError_t launch_batch_persistent(const BatchInst* dev, int ninst, int total_blocks, bool flat, int px, int waves,
                                   int parity, int nsteps, int* next, hipStream_t s) {
    if constexpr (sizeof(TS) == 4) {
        if (waves == 3)
            return launch_persistent_px<TS, 3>(dev, ninst, total_blocks, flat, px, parity, nsteps, next, s);
        return launch_persistent_px<TS, 2>(dev, ninst, total_blocks, flat, px, parity, nsteps, next, s);
    } else {
        return launch_persistent_px<TS, FUSED_WAVES>(dev, ninst, total_blocks, flat, px, parity, nsteps, next, s);
    }
}

template <typename TS>
hipError_t launch_moments(const char* src, const Consts& K, const OutPtrs& out, const DiagBufs& D,
                          const GuessTables* gt, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    int tx, ty, nt, nb;
    grid_of(K, tx, ty, nt, nb);
    hipError_t e = launch_face_b<TS>(src, K, D.faceB, s);
    if (e != hipSuccess) return e;
    if (gt)
        hipLaunchKernelGGL((k_moments<TS, TE, GUESS_SINGLE>), dim3(nb), dim3(TPB), 0, s, src,
                           (const double*)D.faceB, gt, K, tx, ty, nt, out, D.scratch, D.part,
                           D.nullp);
    else
        hipLaunchKernelGGL((k_moments<TS, TE, GUESS_NONE>), dim3(nb), dim3(TPB), 0, s, src,
                           (const double*)D.faceB, gt, K, tx, ty, nt, out, D.scratch, D.part,
                           D.nullp);
    hipLaunchKernelGGL(k_divb, dim3(nb), dim3(TPB), 0, s, (const double*)D.scratch, K, tx, ty, nt, D.part2);
    hipLaunchKernelGGL(k_reduce, dim3(NPART), dim3(TPB), 0, s, (const double*)D.part, nt, NPART, 0, D.result);
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(TPB), 0, s, (const double*)D.part2, nt, 1, 1, D.result + NPART);
    hipLaunchKernelGGL(k_null_reduce, dim3(1), dim3(TPB), 0, s, (const double*)D.nullp, nt,
                       (const double*)(D.scratch + 3 * K.N), (const double*)D.ez0, (const double*)D.b0,
                       D.result + NPART + 1);
    return hipGetLastError();
}

#if RMHDLB_FORM == 64  // what depends on no storage form is built once
hipError_t launch_face_check(const FacePtrs& in, const Consts& K, double* part, double* result, hipStream_t s) {
    const int nblk = (int)(((int64_t)K.nx * K.ny + TPB - 1) / TPB);
    hipLaunchKernelGGL(k_face_check, dim3(nblk), dim3(TPB), 0, s, in, K, part);
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(TPB), 0, s, (const double*)part, nblk, 1, 0, result);
    return hipGetLastError();
}
#endif

template <typename TS>
hipError_t launch_ghost(const FacePtrs& in, const Consts& K, char* dst, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    const int nblk = (int)(((int64_t)K.nx * K.ny + TPB - 1) / TPB);
    hipLaunchKernelGGL((k_init_ghost<TS, TE>), dim3(nblk), dim3(TPB), 0, s, in, K, dst);
    return hipGetLastError();
}

#if RMHDLB_FORM == 64  // what depends on no storage form is built once
hipError_t launch_init_ref(const InPtrs& in, const Consts& K, double* part, double* result, hipStream_t s) {
    const int nblk = (int)((K.N + TPB - 1) / TPB);
    hipLaunchKernelGGL(k_init_ref, dim3(nblk), dim3(TPB), 0, s, in, K, part);
    hipLaunchKernelGGL(k_reduce, dim3(2), dim3(TPB), 0, s, (const double*)part, nblk, 2, 0, result);
    return hipGetLastError();
}
#endif

template <typename TS>
hipError_t launch_init(const InPtrs& in, const Consts& K, double* scr, char* dst, double* ez0, double* part,
                       double* b0, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    int tx, ty, nt, nb;
    grid_of(K, tx, ty, nt, nb);
    hipLaunchKernelGGL(k_init_current, dim3(nb), dim3(TPB), 0, s, in, K, tx, ty, nt, scr, ez0, part);
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(TPB), 0, s, (const double*)part, nt, 1, 2, b0);
    hipLaunchKernelGGL((k_init_state<TS, TE>), dim3(nb), dim3(TPB), 0, s, in, K, tx, ty, nt, (const double*)scr, dst);
    return hipGetLastError();
}

// Whether export and import take a thread per record: below a block of 256 cells
// for every CU a thread per cell leaves most of the chip idle while it goes
// through its 25 (FP32, FP16) to 47 records.  A set_state call of 4096 cells, a thread per cell / per
// record, us: FP64 18.0 / 15.0, FP32 17.1 / 14.9, FP16 21.0 / 15.4; of 65536
// cells 25.0 / 25.5, 21.6 / 20.9, 25.8 / 21.6; of 4194304 772 / 801, 568 / 622,
// 528 / 713.
static inline bool record_threads(const Consts& K) { return K.N < 256 * 256; }

template <typename TS>
hipError_t launch_export(const char* src, double* dst, const Consts& K, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    const unsigned blocks = (unsigned)((K.N + 255) / 256);
    if (record_threads(K))
        hipLaunchKernelGGL((k_export<TS, TE, true>), dim3(blocks, state_records<TS>(K)), dim3(256), 0, s, src, dst, K);
    else
        hipLaunchKernelGGL((k_export<TS, TE, false>), dim3(blocks), dim3(256), 0, s, src, dst, K);
    return hipGetLastError();
}

template <typename TS>
hipError_t launch_import(const double* src, char* dst, const Consts& K, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    const unsigned blocks = (unsigned)((K.N + 255) / 256);
    if (record_threads(K))
        hipLaunchKernelGGL((k_import<TS, TE, true>), dim3(blocks, state_records<TS>(K)), dim3(256), 0, s, src, dst, K);
    else
        hipLaunchKernelGGL((k_import<TS, TE, false>), dim3(blocks), dim3(256), 0, s, src, dst, K);
    return hipGetLastError();
}

template <typename TS>
hipError_t launch_guess_samples(const char* src, const Consts& K, double* faceB, int ns, double* F, double* T,
                                double* part, double* result, hipStream_t s) {
    using TE = typename StoreTypes<TS>::E;
    hipError_t e = launch_face_b<TS>(src, K, faceB, s);
    if (e != hipSuccess) return e;
    const int nblk = (ns + 255) / 256;
    hipLaunchKernelGGL((k_guess_samples<TS, TE>), dim3(nblk), dim3(256), 0, s, src, (const double*)faceB, K, ns, F, T, part);
    hipLaunchKernelGGL(k_reduce, dim3(SAMPLE_SUMS), dim3(256), 0, s, (const double*)part, nblk, SAMPLE_SUMS, 0, result);
    return hipGetLastError();
}

#define RMHD_INSTANTIATE(TS)                                                                                          \
    template hipError_t launch_step<TS>(const char*, char*, const Consts&, const StepTuning&, double*,                \
                                        const GuessTables*, hipStream_t);                                             \
    template hipError_t launch_moments<TS>(const char*, const Consts&, const OutPtrs&, const DiagBufs&,               \
                                           const GuessTables*, hipStream_t);                                          \
    template hipError_t launch_init<TS>(const InPtrs&, const Consts&, double*, char*, double*, double*, double*,       \
                                         hipStream_t);                                                          \
    template hipError_t launch_ghost<TS>(const FacePtrs&, const Consts&, char*, hipStream_t);                         \
    template hipError_t launch_batch<TS>(const BatchInst*, int, int, int64_t, bool, int, int, int, hipStream_t);      \
    template hipError_t launch_batch_persistent<TS>(const BatchInst*, int, int, bool, int, int, int, int, int*,       \
                                                    hipStream_t);                                                     \
    template hipError_t launch_guess_samples<TS>(const char*, const Consts&, double*, int, double*, double*,          \
                                                 double*, double*, hipStream_t);                                      \
    template hipError_t launch_export<TS>(const char*, double*, const Consts&, hipStream_t);                          \
    template hipError_t launch_import<TS>(const double*, char*, const Consts&, hipStream_t);

// One storage form per object, so that the forms compile side by side.
#if RMHDLB_FORM == 64
RMHD_INSTANTIATE(double)
#elif RMHDLB_FORM == 32
RMHD_INSTANTIATE(float)
#else
RMHD_INSTANTIATE(_Float16)
#endif

}  // namespace rmhd
