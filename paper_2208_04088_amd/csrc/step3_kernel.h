// Device code of the three-dimensional (D3Q19) solid lattice-Boltzmann step.
//
// The paper's method (sections 2-4) is two-dimensional; its rules are local
// to a link, and this is their D3Q19 form: the same moments (eq:moments),
// source term (eq:sourceterm), equilibrium with the populations' own second
// moment (eq:fieq) and forced BGK collision (eq:coll), with c_s^2 = 1/3 and
// weights 1/3, 1/18, 1/36.  Boundaries: either two planes normal to x that
// cut the links leaving the material at a fraction q (y and z periodic), or
// (GEO) a general geometry periodic on every axis -- a material mask and cut
// links, each with its own q, outward normal and group (cavities, cracks).
// The Dirichlet rule is eq:bbcon / eq:bbnoncon, the Neumann rule eq:abbcon /
// eq:abbnoncon with the boundary stress
// sigma* = Pi sigma_b Pi + n t* + t* n - (t*.n) n n (Pi = I - n n).
//
// State: shifted post-collision populations g = f - r (r the rest state),
// SoA planes g[i][z][y][x], site offset (z ny + y) nx + x; consecutive planes
// are `stride` elements apart, a little more than a plane, so that the 19
// streams of a pull do not all start on the same HBM channel.  A step of a
// large box is one launch, k3_march (march_of has the rule); of a small one two:
// k3_density (delta-rho of the pulled state, needed by the gradient stencil of
// every neighbour) and k3_step (pull with the rules, moments, source term,
// collision, U, store; with a general geometry also the next step's rule
// values at the cut links), and with extrapolating Neumann links k3_links_ext
// before them.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace slbm3_dev {

// D3Q19: rest; +x -x +y -y +z -z; (1,1,0) (-1,-1,0) (1,-1,0) (-1,1,0);
// (1,0,1) (-1,0,-1) (1,0,-1) (-1,0,1); (0,1,1) (0,-1,-1) (0,1,-1) (0,-1,1).
// Opposite directions are adjacent: opp(i) = i + 1 for odd i.
constexpr int kQ = 19;

// A site update is flagged as diverged when |drho| + |j| (lattice units,
// rest density 1) reaches this bound -- a density deviation as large as the
// rest density itself, far outside linear elasticity -- or is not finite.
constexpr double kDivergeBound = 1.0;
constexpr int kCX[kQ] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr int kCY[kQ] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr int kCZ[kQ] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
__host__ __device__ constexpr int opp3(int i) { return i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1); }
__host__ __device__ constexpr double w3(int i) { return i == 0 ? 1.0 / 3.0 : (i <= 6 ? 1.0 / 18.0 : 1.0 / 36.0); }
__host__ __device__ constexpr int c2_3(int i) { return kCX[i] * kCX[i] + kCY[i] * kCY[i] + kCZ[i] * kCZ[i]; }

enum { kWallNone = 0, kWallDirichlet = 1, kWallNeumann = 2 };

// Site flags of a box with cut links (general geometry): bit i - 1 set when
// link i of the site is cut, kVoid3 for a void site.
constexpr uint32_t kVoid3 = 0x80000000u;
constexpr uint32_t kCutMask3 = 0x3FFFFu;

// One cut link (x, i) of a general geometry, in lattice units, with the
// rule's constants folded on the host.  Dirichlet (eq:bbcon / eq:bbnoncon):
//   g_ib = g_i + kappa (g_i(x - c_i) - g_ib) - rho(x) a c0,  c0 = beta 6 w_i c_i.v*.
// Neumann (eq:abbcon / eq:abbnoncon): g_ib = -g_i - kappa (g_i(x - c_i) + g_ib)
// + 2 beta e, with e = g_eq,i(rho_bd, 0, P*) the shifted equilibrium at the
// boundary stress sigma* = Pi sigma_b Pi + n t* + t* n - (t*.n) n n.  With
// A = c_i c_i - I/3 and sigma_b = -P_b - (lambda - mu) drho_bd I this is
// linear in the site's (or the extrapolated) drho_bd and P_b:
//   e = c0 drho_bd + sum_k B_k P_b,k - a K,
//   c0 = w_i [5/2 - 3/2 |c_i|^2 + 9/2 (lambda - mu)(tr(Pi A Pi) - |c_i|^2 + 1)],
//   B  = 9/2 w_i Pi A Pi (xx yy zz, then xy xz yz doubled),
//   K  = 9/2 w_i [2 n.A.t* - (t*.n) n.A.n].
// a is the time profile of the link's group (1, or a ramp: slot s of the
// launch's factor tables).  kappa and beta are 0 and 1 when the opposite link
// is cut too (no site behind); ext: Neumann with rho_bd and sigma_b
// extrapolated along the link, (1 + q) X(x) - q X(x - c_i).
template <typename real>
struct Link3 {
    real kap, bet2, q1, q;         // kappa, 2 beta, 1 + q, q
    real c0;
    real B[6];
    real K;
    uint32_t meta;                 // link3_meta
    int32_t site;                  // (z ny + y) nx + x of the material site x
};
// meta: direction k (5 bits), opposite (5), kind (2), ext (1), c + 1 per axis
// (2 each), time-profile slot (4)
constexpr int kProfileSlots3 = 16;          // slot 0: constant; 1..15: ramps
__host__ __device__ constexpr uint32_t link3_meta(int k, int kb, int kind, int ext, int cx, int cy, int cz, int slot)
{
    return (uint32_t)k | (uint32_t)kb << 5 | (uint32_t)kind << 10 | (uint32_t)ext << 12 |
           (uint32_t)(cx + 1) << 13 | (uint32_t)(cy + 1) << 15 | (uint32_t)(cz + 1) << 17 | (uint32_t)slot << 19;
}

template <typename real>
struct Step3Args {
    const real* src;           // post-collision state (pulled), or the populations themselves (local)
    real* dst;
    double* U;                 // [3] planes
    real* dens;                // delta-rho of the pulled state (written by k3_density)
    unsigned int* diverged;
    long long plane;           // sites per plane
    long long stride;          // elements from one plane of src, dst or U to the next (>= plane)
    int nx, ny, nz;
    int px;                    // periodic in x (else walls)
    int local;                 // src holds the populations at the sites themselves
    int ntiles;                // 64-site row chunks
    int back;                  // k3_step, k3_readout: from the box's end to its beginning
    int wkind[2];              // walls crossing the first and the last site's x links
    real wval[2][3];           // lattice units: wall velocity (Dirichlet) or traction (Neumann)
    // per wall, from its q: kappa = (1 - 2q)/(1 + 2q), beta = 2/(1 + 2q)
    // (0 and 1 with no site behind, nx = 1); wext: Neumann with rho_bd and
    // the tangential stress extrapolated along the link, weights 1 + q, -q
    real wkap[2], wbeta[2], wq1[2], wq[2];
    int wext[2];
    // general geometry (periodic on every axis): site flags, each cut site's
    // first link record, the records (sorted by site and direction)
    const uint32_t* flags;
    const int32_t* bidx;
    const Link3<real>* links;
    real* lval;                // per record: (A, s_kappa), see cut_links3
    real* lval_next;           // the same, written by k3_march for the next step
    const int32_t* rowrec;     // per 64-site chunk of a row: its first record (one more: the count)
    const int32_t* wrec;       // per workgroup of k3_step: its first record (one more: the count)
    // the groups' time profiles per slot, at the time of the state the pulls
    // read (pf_pull) and of the state the step produces (pf_next)
    real pf_pull[kProfileSlots3], pf_next[kProfileSlots3];
    // k3_march: its tiles (rows, planes, how many of each, 64-site chunks), the
    // walls' returned parts it reads and writes (see wall_parts3) and the
    // walls' values at the time of the state it produces
    int rows, depth, nyt, nch, mtiles, xgroup, nlinks;
    const real* wsrc;
    real* wdst;
    real wskap[2], wval_next[2][3];
    real omega, omega_h;       // 1/tau, 1 - 1/(2 tau)
    real ml, lm;               // mu - lambda, lambda - mu (lattice units)
    real F[3];
};

// Shifted equilibrium g_eq,i = f_eq,i - r_i of eq:fieq, drho = rho - 1:
// w_i [drho (5/2 - 3|c|^2/2) + 3 c.j + 9/2 (P : (c c - I/3))].
template <int i, typename real>
__device__ __forceinline__ real geq3(real dr, const real j[3], const real P[6])
{
    constexpr int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
    constexpr double w = w3(i);
    constexpr double a0 = w * (2.5 - 1.5 * c2_3(i));
    real v = real(a0) * dr;
    if (cx != 0) v += real(3.0 * w * cx) * j[0];
    if (cy != 0) v += real(3.0 * w * cy) * j[1];
    if (cz != 0) v += real(3.0 * w * cz) * j[2];
    v += real(4.5 * w * (cx * cx - 1.0 / 3.0)) * P[0];
    v += real(4.5 * w * (cy * cy - 1.0 / 3.0)) * P[1];
    v += real(4.5 * w * (cz * cz - 1.0 / 3.0)) * P[2];
    if (cx * cy != 0) v += real(9.0 * w * cx * cy) * P[3];
    if (cx * cz != 0) v += real(9.0 * w * cx * cz) * P[4];
    if (cy * cz != 0) v += real(9.0 * w * cy * cz) * P[5];
    return v;
}

// ------------------------------------------------------ ghost moments
//
// The collision of eq:coll leaves rho and P unchanged and adds S to j (the
// equilibrium carries the populations' own second moment).  It is applied as
//   g_i <- g_i + T_i(S) + sum_k a_k n_k,i
// with T(S) = (S_a/2)(e_{+a} - e_{-a}) on the axis links, whose zeroth,
// first and second moments are exactly 0, S and 0 in floating point, and nine
// integer ghost vectors n_k orthogonal to 1, c and c c (an orthogonal D3Q19
// moment basis: epsilon, q_x, q_y, q_z, 3 pi_xx, pi_ww, m_x, m_y, m_z).  The
// coefficients a_k are the projections of the BGK change onto the n_k:
//   a_k = [omega (E_k - m_k) + (1 - omega/2) Psi_k - tau_k] / N_k,
// m_k = n_k.g, E_k = n_k.g_eq, Psi_k = n_k.psi, tau_k = n_k.T, N_k = n_k.n_k.
// In exact arithmetic this is the BGK update; in floating point the conserved
// moments change only by unbiased rounding, whereas rounded equilibrium
// weights would scale them by (1 + omega eps) every step.
__host__ __device__ constexpr int ghost3(int k, int i)
{
    const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
    const int c2 = cx * cx + cy * cy + cz * cz;
    switch (k) {
    case 0: return (21 * c2 * c2 - 53 * c2 + 24) / 2;             // epsilon
    case 1: return (5 * c2 - 9) * cx;                             // q_x
    case 2: return (5 * c2 - 9) * cy;                             // q_y
    case 3: return (5 * c2 - 9) * cz;                             // q_z
    case 4: return (3 * c2 - 5) * (3 * cx * cx - c2);             // 3 pi_xx
    case 5: return (3 * c2 - 5) * (cy * cy - cz * cz);            // pi_ww
    case 6: return cx * (cy * cy - cz * cz);                      // m_x
    case 7: return cy * (cz * cz - cx * cx);                      // m_y
    default: return cz * (cx * cx - cy * cy);                     // m_z
    }
}
constexpr int kGhosts3 = 9;

// sum_i n_k,i f(i) for the lattice tables, at compile time
__host__ __device__ constexpr int ghost_dot_poly(int k, int px, int py, int pz)
{
    int s = 0;
    for (int i = 0; i < kQ; ++i) {
        int m = 1;
        for (int e = 0; e < px; ++e) m *= kCX[i];
        for (int e = 0; e < py; ++e) m *= kCY[i];
        for (int e = 0; e < pz; ++e) m *= kCZ[i];
        s += ghost3(k, i) * m;
    }
    return s;
}
__host__ __device__ constexpr bool ghosts_orthogonal()
{
    for (int k = 0; k < kGhosts3; ++k)
        for (int px = 0; px <= 2; ++px)
            for (int py = 0; py <= 2 - px; ++py)
                for (int pz = 0; pz <= 2 - px - py; ++pz)
                    if (ghost_dot_poly(k, px, py, pz) != 0) return false;
    for (int k = 0; k < kGhosts3; ++k)
        for (int l = 0; l < k; ++l) {
            int s = 0;
            for (int i = 0; i < kQ; ++i) s += ghost3(k, i) * ghost3(l, i);
            if (s != 0) return false;
        }
    return true;
}
static_assert(ghosts_orthogonal(), "ghost vectors must be orthogonal to 1, c, c c and to each other");

__host__ __device__ constexpr double ghost_norm(int k)
{
    double s = 0;
    for (int i = 0; i < kQ; ++i) s += double(ghost3(k, i)) * ghost3(k, i);
    return s;
}
// E_k = n_k.g_eq = er(k) drho + sum_a ej(k, a) j_a + sum_c ep(k, c) P_c (c: xx yy zz xy xz yz)
__host__ __device__ constexpr double ghost_er(int k)
{
    double s = 0;
    for (int i = 0; i < kQ; ++i) s += ghost3(k, i) * w3(i) * (2.5 - 1.5 * c2_3(i));
    return s;
}
__host__ __device__ constexpr double ghost_ej(int k, int a)      // also Psi_k per S_a
{
    double s = 0;
    for (int i = 0; i < kQ; ++i) s += ghost3(k, i) * 3.0 * w3(i) * (a == 0 ? kCX[i] : (a == 1 ? kCY[i] : kCZ[i]));
    return s;
}
__host__ __device__ constexpr double ghost_ep(int k, int c)
{
    double s = 0;
    for (int i = 0; i < kQ; ++i) {
        const int cx = kCX[i], cy = kCY[i], cz = kCZ[i];
        double t = 0;
        switch (c) {
        case 0: t = cx * cx - 1.0 / 3.0; break;
        case 1: t = cy * cy - 1.0 / 3.0; break;
        case 2: t = cz * cz - 1.0 / 3.0; break;
        case 3: t = 2.0 * cx * cy; break;
        case 4: t = 2.0 * cx * cz; break;
        default: t = 2.0 * cy * cz; break;
        }
        s += ghost3(k, i) * 4.5 * w3(i) * t;
    }
    return s;
}
// tau_k per S_a: T puts +S_a/2 on link +a (1, 3, 5) and -S_a/2 on -a (2, 4, 6)
__host__ __device__ constexpr double ghost_et(int k, int a) { return 0.5 * (ghost3(k, 1 + 2 * a) - ghost3(k, 2 + 2 * a)); }

// delta-rho of a site: its 19 populations added as a binary tree (i with
// i + 16, then 8, 4, 2, 1 apart), the order in which the lanes of half a wave
// add them when each holds one (row_sum3).
template <typename real>
__device__ __forceinline__ real sum3(const real g[kQ])
{
    real t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i] = i + 16 < kQ ? g[i] + g[i + 16] : g[i];
#pragma unroll
    for (int h = 8; h >= 1; h >>= 1)
#pragma unroll
        for (int i = 0; i < h; ++i) t[i] = t[i] + t[i + h];
    return t[0];
}

// a b + c, rounded once.
__device__ __forceinline__ float fma3(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma3(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Moments, source and collision of one site: j on return is with S/2, o the
// post-collision populations; S = F + c grad.
//
// Opposite links i, i + 1 (odd i) enter the even ghosts (epsilon, pi_xx,
// pi_ww) and P through their sum and the odd ones (q, m) and j through their
// difference, so each site forms the nine sums and differences once and gives
// the change back as even +- odd: about 240 operations, where summing each
// ghost over all 19 populations takes about 700.
template <typename real>
__device__ __forceinline__ void collide_pairs3(const real g[kQ], real dr, const real grad[3], real c, const real F[3],
                                               real omega, real omega_h, real j[3], real o[kQ])
{
    real s[9], d[9];
#pragma unroll
    for (int p = 0; p < 9; ++p) {
        s[p] = g[2 * p + 1] + g[2 * p + 2];
        d[p] = g[2 * p + 1] - g[2 * p + 2];
    }
    // links: 0-2 the axes; 3 (1,1,0) 4 (1,-1,0) 5 (1,0,1) 6 (1,0,-1) 7 (0,1,1) 8 (0,1,-1)
    const real sxy = s[3] + s[4], sxz = s[5] + s[6], syz = s[7] + s[8];
    const real dxy = d[3] + d[4], exy = d[3] - d[4];         // their x and y parts
    const real dxz = d[5] + d[6], exz = d[5] - d[6];         // x and z
    const real dyz = d[7] + d[8], eyz = d[7] - d[8];         // y and z
    const real bx = dxy + dxz, by = exy + dyz, bz = exz + eyz;
    real S[3], h[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        S[k] = fma3(c, grad[k], F[k]);
        h[k] = real(0.5) * S[k];
    }
    j[0] = (d[0] + bx) + h[0];
    j[1] = (d[1] + by) + h[1];
    j[2] = (d[2] + bz) + h[2];
    const real Pxx = s[0] + (sxy + sxz), Pyy = s[1] + (sxy + syz), Pzz = s[2] + (sxz + syz);
    // m_k = n_k.g and a_k N_k = omega (E_k - m_k) + (omega_h Psi_k - tau_k), with
    // E_k, Psi_k, tau_k of the lattice tables (q: E = ej j, Psi = ej S,
    // tau = -4 S; m: E = Psi = 0, tau = 0)
    const real a4 = s[0] + s[1] + s[2], b6 = sxy + sxz + syz;
    real ak[kGhosts3];
    {
        const real m = fma3(real(12), g[0], fma3(real(-4), a4, b6));
        const real e = fma3(real(ghost_er(0)), dr, real(ghost_ep(0, 0)) * (Pxx + Pyy + Pzz));
        ak[0] = omega * (e - m) * real(1.0 / ghost_norm(0));
    }
    {
        const real m = fma3(real(-4), s[0], fma3(real(2), s[1] + s[2], (sxy + sxz))) - real(2) * syz;
        const real e = fma3(real(ghost_ep(4, 0)), Pxx, real(ghost_ep(4, 1)) * (Pyy + Pzz));
        ak[4] = omega * (e - m) * real(1.0 / ghost_norm(4));
    }
    {
        const real m = fma3(real(2), s[2] - s[1], sxy - sxz);
        const real e = real(ghost_ep(5, 1)) * (Pyy - Pzz);
        ak[5] = omega * (e - m) * real(1.0 / ghost_norm(5));
    }
    const real bq[3] = {bx, by, bz};
    const real k_src = omega_h * real(ghost_ej(1, 0)) - real(ghost_et(1, 0));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const real m = fma3(real(-4), d[k], bq[k]);
        const real e = real(ghost_ej(1, 0)) * j[k];
        ak[1 + k] = fma3(omega, e - m, k_src * S[k]) * real(1.0 / ghost_norm(1));
    }
    const real om_m = -omega * real(1.0 / ghost_norm(6));
    ak[6] = om_m * (dxy - dxz);
    ak[7] = om_m * (dyz - exy);
    ak[8] = om_m * (exz - eyz);
    // even and odd parts of the change, per pair
    const real m4a0 = real(-4) * ak[0], a05 = ak[0] + ak[4];
    const real ev[6] = {fma3(real(-4), ak[4], m4a0), fma3(real(2), ak[4] - ak[5], m4a0), fma3(real(2), ak[4] + ak[5], m4a0),
                        a05 + ak[5], a05 - ak[5], fma3(real(-2), ak[4], ak[0])};
    real od[9];
#pragma unroll
    for (int k = 0; k < 3; ++k) od[k] = fma3(real(-4), ak[1 + k], h[k]);
    od[3] = (ak[1] + ak[2]) + (ak[6] - ak[7]);
    od[4] = (ak[1] - ak[2]) + (ak[6] + ak[7]);
    od[5] = (ak[1] + ak[3]) - (ak[6] - ak[8]);
    od[6] = (ak[1] - ak[3]) - (ak[6] + ak[8]);
    od[7] = (ak[2] + ak[3]) + (ak[7] - ak[8]);
    od[8] = (ak[2] - ak[3]) + (ak[7] + ak[8]);
    o[0] = fma3(real(12), ak[0], g[0]);
#pragma unroll
    for (int p = 0; p < 9; ++p) {
        const real e = ev[p < 3 ? p : 3 + (p - 3) / 2];
        o[2 * p + 1] = g[2 * p + 1] + (e + od[p]);
        o[2 * p + 2] = g[2 * p + 2] + (e - od[p]);
    }
}
// delta-rho, j and P (xx yy zz xy xz yz) of shifted populations.
template <typename real>
__device__ __forceinline__ void moments3(const real g[kQ], real& dr, real j[3], real P[6])
{
    dr = real(0);
    j[0] = j[1] = j[2] = real(0);
    for (int k = 0; k < 6; ++k) P[k] = real(0);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        dr += g[i];
        if (kCX[i]) j[0] += kCX[i] > 0 ? g[i] : -g[i];
        if (kCY[i]) j[1] += kCY[i] > 0 ? g[i] : -g[i];
        if (kCZ[i]) j[2] += kCZ[i] > 0 ? g[i] : -g[i];
        if (kCX[i]) P[0] += g[i];
        if (kCY[i]) P[1] += g[i];
        if (kCZ[i]) P[2] += g[i];
        if (kCX[i] * kCY[i]) P[3] += kCX[i] * kCY[i] > 0 ? g[i] : -g[i];
        if (kCX[i] * kCZ[i]) P[4] += kCX[i] * kCZ[i] > 0 ? g[i] : -g[i];
        if (kCY[i] * kCZ[i]) P[5] += kCY[i] * kCZ[i] > 0 ? g[i] : -g[i];
    }
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Site (x, y, z) of a 64-site row chunk: tile t -> (chunk, y, z), chunks
// fastest; lanes past nx are outside.
struct Site3 {
    int x, y, z;
    bool in;
};

__device__ __forceinline__ Site3 site_of(int tile, int lane, int nx, int ny)
{
    const int chunks = (nx + 63) >> 6;
    const int c = tile % chunks, r = tile / chunks;
    Site3 s;
    s.x = (c << 6) + lane;
    s.y = r % ny;
    s.z = r / ny;
    s.in = s.x < nx;
    if (!s.in) s.x = nx - 1;                   // keep addresses in the grid
    return s;
}

__device__ __forceinline__ unsigned sidx3(int x, int y, int z, int nx, int ny)
{
    return ((unsigned)z * (unsigned)ny + (unsigned)y) * (unsigned)nx + (unsigned)x;
}

// The populations of the step at a site: pulled from the neighbours'
// post-collision values along uncut links; on a link cut by a wall the
// returning population comes from the wall rule, from the site's own
// post-collision populations (rho and P are those of the previous step,
// conserved by the collision).
// The rules of section 4 at the cut links of a general geometry.  The value
// a cut link (x, i) returns to x in direction ibar is A + s_kappa g_i(x - c_i):
// A takes only the post-collision state at x, s_kappa is kappa (Dirichlet) or
// -kappa (Neumann), and g_i(x - c_i) is the population the pull of direction
// i brings to x anyway (a thin link has kappa = 0 and needs none).  k3_step
// evaluates A at every cut link of its workgroup's sites as soon as it has
// their post-collision populations (one thread per link, through LDS), so
// the rules take no pass of their own over the state.  A link whose Neumann
// data are extrapolated along it (ext) needs the state at x - c_i as well:
// k3_links_ext evaluates its whole value, with s_kappa = 0.  lval holds
// (A, s_kappa) per record; s_kappa is set on the host.
//
// A from the record's folded constants (its own q, normal and group), g_i
// and g_ib at x, drho and (or, ext, rho_bd and P_b) at x.
template <typename real>
__device__ __forceinline__ real link_part3(const Link3<real>& L, real hi, real hib, real dr, real drb, const real Pb[6],
                                           real at)
{
    if (((L.meta >> 10) & 3u) == kWallDirichlet) return hi - L.kap * hib - (real(1) + dr) * (at * L.c0);
    const real e = L.c0 * drb + (L.B[0] * Pb[0] + L.B[1] * Pb[1] + L.B[2] * Pb[2]) +
                   (L.B[3] * Pb[3] + L.B[4] * Pb[4] + L.B[5] * Pb[5]) - at * L.K;
    return -hi - L.kap * hib + L.bet2 * e;
}

// The whole value of each ext link from the post-collision state, one thread
// per link (elink: the records' indices).
template <typename real>
__global__ __launch_bounds__(256) void k3_links_ext(Step3Args<real> a, const int32_t* elink, int n_ext)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n_ext) return;
    const int l = elink[t];
    const Link3<real> L = a.links[l];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned s = (unsigned)L.site;
    const int x = (int)(s % (unsigned)nx), y = (int)((s / (unsigned)nx) % (unsigned)ny),
              z = (int)(s / ((unsigned)nx * (unsigned)ny));
    const int i = (int)(L.meta & 31u), ib = (int)((L.meta >> 5) & 31u);
    const int cx = (int)((L.meta >> 13) & 3u) - 1, cy = (int)((L.meta >> 15) & 3u) - 1, cz = (int)((L.meta >> 17) & 3u) - 1;
    // the site behind x along the link, x - c_i (periodic axes)
    const unsigned sb = sidx3(wrap(x - cx, nx), wrap(y - cy, ny), wrap(z - cz, nz), nx, ny);
    real h[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) h[k] = a.src[k * a.stride + s];
    real dr, j[3], P[6];
    moments3(h, dr, j, P);
    const real hi = a.src[i * a.stride + s], hib = a.src[ib * a.stride + s], hy = a.src[i * a.stride + sb];
#pragma unroll
    for (int k = 0; k < kQ; ++k) h[k] = a.src[k * a.stride + sb];
    real dry, Py[6];
    moments3(h, dry, j, Py);
    const real drb = L.q1 * dr - L.q * dry;
#pragma unroll
    for (int c = 0; c < 6; ++c) P[c] = L.q1 * P[c] - L.q * Py[c];
    a.lval[2 * l] = link_part3(L, hi, hib, dr, drb, P, a.pf_pull[(L.meta >> 19) & 15u]) - L.kap * hy;
}

// A cut site's pulls along its cut links (the site's records are consecutive,
// in direction order, from bidx): A + s_kappa g_i(x - c_i), every value
// formed from the pulled populations before any is replaced.
template <typename real>
__device__ __forceinline__ void cut_links3(const Step3Args<real>& a, unsigned s, uint32_t fl, real g[kQ])
{
    const int li = a.bidx[s];
    const uint32_t m = fl & kCutMask3;
    real v[kQ];
#pragma unroll
    for (int k = 1; k < kQ; ++k)
        if ((m >> (k - 1)) & 1u) {
            const int l = li + __builtin_popcount(m & ((1u << (k - 1)) - 1u));
            v[k] = a.lval[2 * l] + a.lval[2 * l + 1] * g[k];
        }
#pragma unroll
    for (int k = 1; k < kQ; ++k)
        if ((m >> (k - 1)) & 1u) g[opp3(k)] = v[k];
}

// The walls' parts: link k of the five that leave through a wall returns
// A_k + s g, g the population that the pull along the leaving direction brings
// to the site (f_i at x - c_i) and s = kappa (Dirichlet) or -kappa (Neumann);
// A takes the post-collision state of the site only, so the step that
// produces the state leaves it behind ([side][5][nz][ny]).
__host__ __device__ constexpr int wall_pair3(int m) { return m == 0 ? 1 : 5 + 2 * m; }   // 1 7 9 11 13: link with c_x = 1

template <typename real>
__device__ __forceinline__ void wall_parts3(const Step3Args<real>& a, int side, const real vs[3], const real o[kQ],
                                            real A[5])
{
    real dr, j[3], P[6];
    moments3(o, dr, j, P);
    real kap = a.wkap[side], bet = a.wbeta[side], lm = a.lm, v[3] = {vs[0], vs[1], vs[2]};
    // formed anew at each use: products of these held across k3_march's loop
    // would spill
    asm volatile("" : "+s"(kap), "+s"(bet), "+s"(lm), "+s"(v[0]), "+s"(v[1]), "+s"(v[2]));
    const real n = side == 0 ? real(-1) : real(1);
    const real Ps[6] = {-(n * v[0]) - lm * dr, P[1], P[2], -(n * v[1]), -(n * v[2]), P[5]};
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        // i leaves, i1 = the pair's link with c_x = 1: c_i = n c_i1
        const int i1 = wall_pair3(m);
        const real oi = side == 0 ? o[i1 + 1] : o[i1], ob = side == 0 ? o[i1] : o[i1 + 1];
        if (a.wkind[side] == kWallDirichlet) {
            const real cv = n * (v[0] + real(kCY[i1]) * v[1] + real(kCZ[i1]) * v[2]);
            A[m] = oi - kap * ob - bet * (real(6.0 * w3(i1)) * (real(1) + dr) * cv);
        } else {
            real e = real(w3(i1) * (2.5 - 1.5 * c2_3(i1))) * dr;
            e += real(4.5 * w3(i1) * (2.0 / 3.0)) * Ps[0];
            e += real(4.5 * w3(i1) * (kCY[i1] * kCY[i1] - 1.0 / 3.0)) * Ps[1];
            e += real(4.5 * w3(i1) * (kCZ[i1] * kCZ[i1] - 1.0 / 3.0)) * Ps[2];
            if (kCY[i1]) e += real(9.0 * w3(i1) * kCY[i1]) * Ps[3];
            if (kCZ[i1]) e += real(9.0 * w3(i1) * kCZ[i1]) * Ps[4];
            A[m] = -oi - kap * ob + bet * (real(2) * e);
        }
    }
}

// The five populations that a Neumann wall returns with its boundary data
// extrapolated along the link: eq:abbnoncon, f_ib = -f_i - kappa (f_i(x - c_i)
// + f_ib) + beta 2 f_eq,i(rho_bd, 0, P*); shifted: g_eq in place of f_eq.  The
// boundary Poisson stress P* = -sigma* - (lambda - mu) drho_bd I with
// sigma = -P - (lambda - mu) drho I takes its normal row from the traction,
// rho_bd and its tangential block as (1 + q) X(x) - q X(x - c_i).
template <typename real>
__device__ __forceinline__ void ext_wall3(const Step3Args<real>& a, const Site3& st, int side, const real h[kQ], real dr,
                                          const real P[6], real g[kQ])
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const real n = side == 0 ? real(-1) : real(1);
    const real* v = a.wval[side];
    const real kap = a.wkap[side], bet = a.wbeta[side];
    const int bx = side == 0 ? st.x + 1 : st.x - 1;         // the next site inward (nx > 1)
    const real jz[3] = {real(0), real(0), real(0)};
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
        // link i leaves through this wall; its opposite returns
        if (kCX[i] != (side == 0 ? -1 : 1)) continue;
        const unsigned sb = sidx3(bx, wrap(st.y - kCY[i], ny), wrap(st.z - kCZ[i], nz), nx, ny);
        const real hy = a.src[i * a.stride + sb];           // f_i at x - c_i
        real hb[kQ];
#pragma unroll
        for (int k = 0; k < kQ; ++k) hb[k] = a.src[k * a.stride + sb];
        real dry, jy[3], Py[6];
        moments3(hb, dry, jy, Py);
        const real w1 = a.wq1[side], w2 = a.wq[side];
        const real drb = w1 * dr - w2 * dry;
        const real Ps[6] = {-(n * v[0]) - a.lm * drb, w1 * P[1] - w2 * Py[1], w1 * P[2] - w2 * Py[2], -(n * v[1]),
                            -(n * v[2]), w1 * P[5] - w2 * Py[5]};
        real e;
        switch (i) {
#define SLBM3_GEQ(k) case k: e = geq3<k, real>(drb, jz, Ps); break;
            SLBM3_GEQ(1) SLBM3_GEQ(2) SLBM3_GEQ(3) SLBM3_GEQ(4) SLBM3_GEQ(5) SLBM3_GEQ(6)
            SLBM3_GEQ(7) SLBM3_GEQ(8) SLBM3_GEQ(9) SLBM3_GEQ(10) SLBM3_GEQ(11) SLBM3_GEQ(12)
            SLBM3_GEQ(13) SLBM3_GEQ(14) SLBM3_GEQ(15) SLBM3_GEQ(16) SLBM3_GEQ(17) SLBM3_GEQ(18)
#undef SLBM3_GEQ
            default: e = real(0);
        }
        g[opp3(i)] = -h[i] - kap * (hy + h[opp3(i)]) + bet * (real(2) * e);
    }
}

template <typename real, bool PX, bool GEO = false>
__device__ __forceinline__ void pull3(const Step3Args<real>& a, const Site3& st, real g[kQ], uint32_t& fl)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned s = sidx3(st.x, st.y, st.z, nx, ny);
    fl = GEO ? a.flags[s] : 0u;
    if (a.local) {
#pragma unroll
        for (int i = 0; i < kQ; ++i) g[i] = a.src[i * a.stride + s];
        if (GEO && (fl & kVoid3)) {
#pragma unroll
            for (int i = 0; i < kQ; ++i) g[i] = real(0);
        }
        return;
    }
    const int ym = wrap(st.y - 1, ny), yp = wrap(st.y + 1, ny);
    const int zm = wrap(st.z - 1, nz), zp = wrap(st.z + 1, nz);
    int xm = st.x - 1, xp = st.x + 1;
    if (PX) {
        xm = wrap(xm, nx);
        xp = wrap(xp, nx);
    } else {
        xm = xm < 0 ? 0 : xm;                  // cut links: replaced below
        xp = xp >= nx ? nx - 1 : xp;
    }
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
        const int xx = kCX[i] > 0 ? xm : (kCX[i] < 0 ? xp : st.x);
        const int yy = kCY[i] > 0 ? ym : (kCY[i] < 0 ? yp : st.y);
        const int zz = kCZ[i] > 0 ? zm : (kCZ[i] < 0 ? zp : st.z);
        g[i] = a.src[i * a.stride + sidx3(xx, yy, zz, nx, ny)];
    }
    if constexpr (GEO) {
        // the pulls above are issued for every lane (in-grid addresses), so
        // that they do not wait for the flags
        if (fl & kVoid3) {                      // void: nothing to pull
#pragma unroll
            for (int i = 0; i < kQ; ++i) g[i] = real(0);
        } else if ((fl & kCutMask3) != 0u) {
            cut_links3<real>(a, s, fl, g);
        }
        return;
    }
    if (!PX && (st.x == 0 || st.x == nx - 1)) {
        real h[kQ];
#pragma unroll
        for (int i = 0; i < kQ; ++i) h[i] = a.src[i * a.stride + s];
        real dr = real(0), j[3], P[6];
        if (a.wext[0] || a.wext[1]) moments3(h, dr, j, P);
        // both walls when nx == 1: what either returns is formed from the pulls
        // before any is replaced (kappa = 0 then)
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (side == 0 ? st.x != 0 : st.x != nx - 1) continue;
            if (a.wext[side]) {
                ext_wall3(a, st, side, h, dr, P, g);
                continue;
            }
            real A[5];
            wall_parts3(a, side, a.wval[side], h, A);
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                const int i1 = wall_pair3(m);               // c_x = 1: returned by side 0, leaves through side 1
                const real gl = nx == 1 ? real(0) : (side == 0 ? g[i1 + 1] : g[i1]);
                (side == 0 ? g[i1] : g[i1 + 1]) = A[m] + a.wskap[side] * gl;
            }
        }
    }
}

// Density gradient of eq:sourceterm, isotropic D3Q19 stencil
// grad = 3 sum_i w_i c_i rho(x + c_i); across a cut link the neighbour is
// 2 rho(x) - rho(x - c_i) (rho(x) if that is cut too).  It is added up plane by
// plane in z, so that k3_march can carry a plane's share to the next one:
// what plane p gives the gradient of the sites above and below it (sx, sy to
// the x and y components, tz to z), and in its own plane (gx, gy).
template <typename real>
struct PlaneTerms3 {
    real sx, sy, tz, gx, gy;
};

// From delta-rho of the 3 x 3 sites around a site (C its own; E, W at x +- 1,
// N, S at y +- 1).  side: the wall that cuts the site's x links (0 at x = 0, 1
// at x = nx - 1, -1 none): there the difference to the opposite neighbour
// doubles the inner one's (less 2 rho(x), which wall_grad3 takes off), and the
// sum that enters the other axes' terms doubles it too.
template <typename real>
__device__ __forceinline__ PlaneTerms3<real> plane_terms3(real C, real E, real W, real N, real S, real NE, real NW, real SE,
                                                          real SW, int side)
{
    real Ed = E, Wd = W, NEd = NE, NWd = NW, SEd = SE, SWd = SW;
    if (side == 0) { W = E; NW = NE; SW = SE; Wd = -E; NWd = -NE; SWd = -SE; }
    if (side == 1) { E = W; NE = NW; SE = SW; Ed = -W; NEd = -NW; SEd = -SW; }
    PlaneTerms3<real> t;
    t.sx = Ed - Wd;
    t.sy = N - S;
    t.tz = fma3(real(1.0 / 6.0), C, real(1.0 / 12.0) * ((E + W) + (N + S)));
    t.gx = fma3(real(1.0 / 6.0), t.sx, real(1.0 / 12.0) * ((NEd - NWd) + (SEd - SWd)));
    t.gy = fma3(real(1.0 / 6.0), t.sy, real(1.0 / 12.0) * ((NE - SE) + (NW - SW)));
    return t;
}
// The in-plane part with the share of the plane below, then with that above.
template <typename real>
__device__ __forceinline__ real with_share3(real g, real s)
{
    return fma3(real(1.0 / 12.0), s, g);
}
template <typename real>
__device__ __forceinline__ real wall_grad3(int side, real dr)
{
    return side == 0 ? -dr : (side == 1 ? dr : real(0));
}

// The gradient from the densities of all 18 neighbours (CUTS: across a cut
// link of fl the neighbour is extrapolated).
template <bool CUTS, typename real>
__device__ __forceinline__ void grad_nb3(real nb[kQ], real dr, uint32_t fl, int side, real grad[3])
{
    if (CUTS && (fl & kCutMask3) != 0u) {
        real sub[kQ];
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
            const bool ci = (fl >> (i - 1)) & 1u, co = (fl >> (opp3(i) - 1)) & 1u;
            sub[i] = ci ? (co ? dr : real(2) * dr - nb[opp3(i)]) : nb[i];
        }
#pragma unroll
        for (int i = 1; i < kQ; ++i) nb[i] = sub[i];
    }
    // planes z - 1, z, z + 1 (only the terms that enter are used)
    const real o = real(0);
    const PlaneTerms3<real> lo = plane_terms3(nb[6], nb[13], nb[12], nb[17], nb[16], o, o, o, o, side);
    const PlaneTerms3<real> in = plane_terms3(dr, nb[1], nb[2], nb[3], nb[4], nb[7], nb[10], nb[9], nb[8], side);
    const PlaneTerms3<real> hi = plane_terms3(nb[5], nb[11], nb[14], nb[15], nb[18], o, o, o, o, side);
    grad[0] = with_share3(with_share3(in.gx, lo.sx), hi.sx);
    if (side >= 0) grad[0] += wall_grad3(side, dr);
    grad[1] = with_share3(with_share3(in.gy, lo.sy), hi.sy);
    grad[2] = hi.tz - lo.tz;
}

// The gradient from the delta-rho buffer.
template <typename real, bool PX, bool GEO = false>
__device__ __forceinline__ void grad3(const Step3Args<real>& a, const Site3& st, real dr, real grad[3],
                                      uint32_t fl = 0u)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const real* d = a.dens;
    const int ym = wrap(st.y - 1, ny), yp = wrap(st.y + 1, ny);
    const int zm = wrap(st.z - 1, nz), zp = wrap(st.z + 1, nz);
    const bool cutm = !PX && st.x == 0, cutp = !PX && st.x == nx - 1;
    const int xm = PX ? wrap(st.x - 1, nx) : (cutm ? st.x : st.x - 1);
    const int xp = PX ? wrap(st.x + 1, nx) : (cutp ? st.x : st.x + 1);
    real nb[kQ];
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
        const int xx = kCX[i] > 0 ? xp : (kCX[i] < 0 ? xm : st.x);
        const int yy = kCY[i] > 0 ? yp : (kCY[i] < 0 ? ym : st.y);
        const int zz = kCZ[i] > 0 ? zp : (kCZ[i] < 0 ? zm : st.z);
        nb[i] = d[sidx3(xx, yy, zz, nx, ny)];
    }
    if (cutm && cutp) {                                     // both x neighbours are across a wall
#pragma unroll
        for (int i = 1; i < kQ; ++i)
            if (kCX[i]) nb[i] = dr;
    }
    const int side = cutm == cutp ? -1 : (cutm ? 0 : 1);
    grad_nb3<GEO>(nb, dr, fl, side, grad);
}

// Workgroups are dealt round-robin to the 8 XCDs.  Each XCD takes groups of
// kXcdGroup consecutive workgroups, and the groups of the 8 XCDs interleave:
// the chip streams through one region of the box at a time (one set of 19
// plane streams rather than one per XCD), while rows that share neighbours
// stay in one L2.  The grid size is a multiple of 8 groups, which makes the
// map a permutation of the workgroup indices.  Groups of 16 suit the plane
// walls; a general geometry runs best with groups of 64 (its flags, link
// records and rule values stay longer in one L2: 0.98 against 1.09 ms per
// step on the 256^3 porous solid, while the slab is the same within 0.2 %).
__host__ __device__ constexpr int xcd_group_size3(bool geo) { return geo ? 64 : 16; }
template <bool GEO>
__device__ __forceinline__ int xcd_group3(int b)
{
    constexpr int G = xcd_group_size3(GEO);
    const int x = b & 7, l = b >> 3;
    return ((l / G) * 8 + x) * G + l % G;
}

// delta-rho of the pulled state at every site.
template <typename real, bool PX, bool GEO = false>
__global__ __launch_bounds__(256) void k3_density(Step3Args<real> a)
{
    const int tile = xcd_group3<GEO>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (tile >= a.ntiles) return;
    const Site3 st = site_of(tile, threadIdx.x & 63, a.nx, a.ny);
    real g[kQ];
    uint32_t fl;
    pull3<real, PX, GEO>(a, st, g, fl);
    real dr = sum3(g);
    if (GEO && (fl & kVoid3)) dr = real(0);               // void: never read
    if (st.in) a.dens[sidx3(st.x, st.y, st.z, a.nx, a.ny)] = dr;
}

// 1/x: the hardware reciprocal in single precision, a division in double.
__device__ __forceinline__ float recip3(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip3(double x) { return 1.0 / x; }

// One time step at every site: pull (with the wall rules), moments, source
// term, eq:coll, U += j/rho, store.  With `back` it goes through the box
// backwards, as does k3_readout: the density pass before it ends on the sites
// that it begins with, and it ends on those the next density pass reads first,
// while they are still in the caches (make_args3 has the rule).
template <typename real, bool PX, bool GEO = false>
__global__ __launch_bounds__(256) void k3_step(Step3Args<real> a)
{
    const int wg = xcd_group3<GEO>(turn(blockIdx.x, gridDim.x, a.back));
    int tile = wg * 4 + (threadIdx.x >> 6);
    if (wg * 4 >= a.ntiles) return;                     // uniform over the workgroup
    const bool tvalid = tile < a.ntiles;
    if (!tvalid) {
        if constexpr (!GEO) return;
        tile = a.ntiles - 1;                            // GEO: stays for the barrier, stores nothing
    }
    Site3 st = site_of(tile, threadIdx.x & 63, a.nx, a.ny);
    if (!tvalid) st.in = false;
    real g[kQ];
    uint32_t fl;
    pull3<real, PX, GEO>(a, st, g, fl);
    const bool live = st.in && !(GEO && (fl & kVoid3));  // void sites stay at rest
    const real dr = sum3(g);
    real grad[3];
    grad3<real, PX, GEO>(a, st, dr, grad, fl);
    const real ir = recip3(real(1) + dr);
    const unsigned s = sidx3(st.x, st.y, st.z, a.nx, a.ny);
    // eq:coll in ghost-moment form (exact conserved moments)
    real o[kQ], j[3];
    collide_pairs3(g, dr, grad, a.ml * ir, a.F, a.omega, a.omega_h, j, o);
    const bool bad = !(fabs(dr) + fabs(j[0]) + fabs(j[1]) + fabs(j[2]) < real(kDivergeBound));
    // void sites store the rest state (zeros) rather than nothing: whole
    // lines reach HBM, where a partly written line costs a read-modify-write
    if (st.in) {
#pragma unroll
        for (int i = 0; i < kQ; ++i) a.dst[i * a.stride + s] = live ? o[i] : real(0);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            a.U[k * a.stride + s] = live ? a.U[k * a.stride + s] + (double)(j[k] * ir) : 0.0;
    }
    if (__any(bad && live) && (threadIdx.x & 63) == 0 && *(volatile unsigned int*)a.diverged == 0u)
        atomicOr(a.diverged, 1u);
    if constexpr (GEO) {
        // A at the cut links of the workgroup's sites (a contiguous range of
        // at most 256 from the first site of its first tile), one thread per
        // record, from the post-collision populations staged in LDS
        const int r0 = a.wrec[wg], nrec = a.wrec[wg + 1] - r0;   // uniform over the workgroup
        if (nrec > 0) {
            __shared__ real lo[kQ][256];
            const Site3 b0 = site_of(wg * 4, 0, a.nx, a.ny);
            const unsigned base = sidx3(b0.x, b0.y, b0.z, a.nx, a.ny);
            if (live) {
#pragma unroll
                for (int i = 0; i < kQ; ++i) lo[i][s - base] = o[i];
            }
            __syncthreads();
            for (int r = threadIdx.x; r < nrec; r += 256) {
                const Link3<real> L = a.links[r0 + r];
                if ((L.meta >> 12) & 1u) continue;              // ext: k3_links_ext
                const int slot = (int)((unsigned)L.site - base);
                real h[kQ];
#pragma unroll
                for (int i = 0; i < kQ; ++i) h[i] = lo[i][slot];
                real hd, hj[3], hP[6];
                moments3(h, hd, hj, hP);
                const int k = (int)(L.meta & 31u), kb = (int)((L.meta >> 5) & 31u);
                a.lval[2 * (r0 + r)] =
                    link_part3(L, lo[k][slot], lo[kb][slot], hd, hd, hP, a.pf_next[(L.meta >> 19) & 15u]);
            }
        }
    }
}

// ------------------------------------------------ one launch per step
//
// k3_march takes the density pass and the step in one launch: a workgroup
// owns `rows` rows of a 64-site chunk and marches through `depth` planes.
// Wave w holds row y0 - 1 + w (the first and the last only supply density).
// When the pulls of plane p arrive it adds them up, leaves the density in LDS
// and the populations in LDS of its own, and sends the loads of plane p + 1
// off into the same registers; after one barrier the inner waves step plane
// p - 1 while those are in flight.  So a population is read from memory once
// per step where the density pass and the step read it twice; the halo rows
// (2 in 10) and planes (2 in depth + 2) come from L2.
//
// Cut links (GEO): the (A, s_kappa) of a row's links and of its two halo sites'
// links come with its pulls (their place in the list follows from the row's
// first record and the flags, so no load waits for another), and the parts for
// the next step go to a second buffer, as workgroups that share a halo row
// still read the first.
//
// Bound by HBM: 256^3 fp32 moves 3.25 GB a step (counters), the 200 B per
// site it cannot do without, at 4.9 TB/s: 669 us periodic, 683 us with walls,
// where the two launches move 4.8 GB in 901 and 905 us; fp64 1229 us against
// 1682; the porous solid 752 against 981 us (its critical path is a cut row's
// 700 further instructions, between two barriers).  What it took, 256^3 fp32:
// - waves of an exact 64-site chunk (62-column strips waste a fifth of a
//   256-site row), the two halo columns gathered by one more load a wave;
// - collide_pairs3 (300 vector instructions a site-step, two launches: 1050);
// - no wait but for the pulls themselves: loads without a branch, a fixed
//   number of stores behind them, LDS-only barriers, U added in memory
//   (atomics that return nothing) instead of loaded, and not one spill, whose
//   reload would wait for every load in flight (slab: 1500 us with 47 spilled
//   registers, 731 with none);
// - tiles dealt to the XCDs in groups of 16, so that the chip moves through one
//   region of the box (groups of 8 to 32 689 us, contiguous bands 722, 1 711);
// - stores past the caches, where the state is larger than they are (689 ->
//   669 us, porous solid 854 -> 800; launch3_march has the smaller ones);
// - 8 rows: 6 rows 780 us (their halo, and a last tile of 4 rows), 14 rows 765;
//   one or two workgroups on a CU make no difference.
// fp64: 8 waves, what the LDS of a CU holds of their populations (110 KB).
constexpr int kMarchWaves(int bytes) { return bytes == 4 ? 10 : 8; }     // waves of a workgroup at most
constexpr int kMarchOcc(int bytes, bool geo) { return bytes == 4 ? (geo ? 3 : 5) : 2; }   // waves per SIMD it is compiled for

// The parts from a state that no k3_march produced (a loaded one, or one that
// the two launches advanced).
template <typename real>
__global__ __launch_bounds__(256) void k3_wall_parts(Step3Args<real> a, real* out)
{
    const int n = a.ny * a.nz, side = blockIdx.y, r = blockIdx.x * 256 + threadIdx.x;   // r = z ny + y
    if (r >= n) return;
    const unsigned s = (unsigned)r * (unsigned)a.nx + (side ? a.nx - 1 : 0);
    real o[kQ], A[5];
#pragma unroll
    for (int i = 0; i < kQ; ++i) o[i] = a.src[i * a.stride + s];
    wall_parts3(a, side, a.wval[side], o, A);
#pragma unroll
    for (int m = 0; m < 5; ++m) out[(long long)(side * 5 + m) * n + r] = A[m];
}

template <typename T>
using gptr3 = __attribute__((address_space(1))) T*;

// Walks the planes of a population or displacement buffer: the base stays in
// scalar registers (the empty asm also keeps the compiler from holding all 19
// bases across the loop, more than it has), the byte offset in the plane in
// one vector register (below 2^32: at most 2^29 sites).
struct PlaneWalk {
    gptr3<char> base;
    unsigned long long step;
    template <typename T>
    __device__ __forceinline__ PlaneWalk(const T* p, long long stride)
        : base((gptr3<char>)p), step((unsigned long long)stride * sizeof(T))
    {
        asm volatile("" : "+s"(base));
    }
    __device__ __forceinline__ void next()
    {
        base += step;
        asm("" : "+s"(base));
    }
    // what only the next launch reads again; STREAM: past the caches
    template <bool STREAM, typename T>
    __device__ __forceinline__ void store(unsigned off, T v) const
    {
        if constexpr (STREAM) __builtin_nontemporal_store(v, (gptr3<T>)(base + off));
        else *(gptr3<T>)(base + off) = v;
    }
    // += in memory (one rounded sum, as a load, an add and a store)
    __device__ __forceinline__ void add(unsigned off, double v) const
    {
        (void)__builtin_amdgcn_global_atomic_fadd_f64((gptr3<double>)(base + off), v);
    }
};

// Barrier over LDS only: loads from global memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Adds what the 32 lanes of each half-wave hold in sum3's order (lanes from
// kQ on hold zero).
template <int N>
__device__ __forceinline__ float row_ror(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, false));
}
template <int N>
__device__ __forceinline__ double row_ror(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + N, 0xF, 0xF, false);
    return __longlong_as_double((long long)((unsigned long long)(unsigned)hi << 32 | (unsigned)lo));
}
template <typename real>
__device__ __forceinline__ real half_sum3(real v)
{
    v += __shfl_xor(v, 16);
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return v;
}

// The population a lane holds of its halo column (lanes from kQ on: none,
// they repeat population 0), its c + 1 per axis (2 bits each), and whether it
// is one that the x = nx - 1 wall returns to the right column.
__device__ __forceinline__ int halo_dir3(int lane) { return (lane & 31) < kQ ? (lane & 31) : 0; }
__host__ __device__ constexpr uint64_t halo_bits3(int axis, int sign)
{
    uint64_t b = 0;
    for (int i = 0; i < kQ; ++i) b |= (uint64_t)((axis == 0 ? kCX[i] : (axis == 1 ? kCY[i] : kCZ[i])) == sign) << i;
    return b;
}
__device__ __forceinline__ int halo_c3(int i)
{
    constexpr uint32_t xp = (uint32_t)halo_bits3(0, 1), xn = (uint32_t)halo_bits3(0, -1), yp = (uint32_t)halo_bits3(1, 1),
                       yn = (uint32_t)halo_bits3(1, -1), zp = (uint32_t)halo_bits3(2, 1), zn = (uint32_t)halo_bits3(2, -1);
    const int cx = 1 + (int)((xp >> i) & 1u) - (int)((xn >> i) & 1u), cy = 1 + (int)((yp >> i) & 1u) - (int)((yn >> i) & 1u),
              cz = 1 + (int)((zp >> i) & 1u) - (int)((zn >> i) & 1u);
    return cx | cy << 2 | cz << 4;
}
__device__ __forceinline__ bool halo_ret3(int lane)
{
    constexpr uint32_t xn = (uint32_t)halo_bits3(0, -1);
    return lane >= 32 && ((xn >> (lane & 31)) & 1u);
}

// Pulled populations of one plane: a row's, and the lane's share of the two
// halo columns (lane i: population i of column x0 - 1, lane 32 + i of column
// x0 + 64).
// GEO: also the flags of the lane's site and of its halo site, and (A, s_kappa)
// of the first 64 cut links of the wave's sites (lane l: link l) and of the
// links next to them (lanes 0..17: the 18 before, which end with the left halo
// site's; lanes 32..49: the 18 after, which begin with the right one's).
template <typename real, bool GEO>
struct Plane3 {
    real g[kQ];
    real halo;
};
template <typename real>
struct Plane3<real, true> {
    real g[kQ];
    real halo;
    uint32_t fl, hfl;
    real la, ls, ha, hs;
};
// The records of a row chunk, and where those of its left halo site end and
// those of its right one begin.
struct RowRec3 {
    int r0, r1, left, right;
};

template <typename real, bool PX, bool GEO, bool STREAM>
__global__ __launch_bounds__(64 * kMarchWaves(sizeof(real)), kMarchOcc(sizeof(real), GEO)) void k3_march(Step3Args<real> a)
{
    constexpr int NW = kMarchWaves(sizeof(real));
    constexpr int RING = GEO ? 4 : 2;                       // GEO: a cut site reads three planes
    __shared__ real dens[RING][NW][68];
    __shared__ real pairs[GEO ? NW : 1][GEO ? 64 : 1][2];
    // GEO, fp32: a cut row's post-collision populations, for its links' parts (in
    // double precision LDS has no room left; the lanes shuffle them)
    constexpr bool STAGE = GEO && sizeof(real) == 4;
    __shared__ real stage[STAGE ? NW : 1][STAGE ? kQ : 1][STAGE ? 64 : 1];
    __shared__ real profile[kProfileSlots3];                // the groups' factors, indexed by record
    if (GEO && threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kProfileSlots3; ++k) profile[k] = a.pf_next[k];
    }
    // a lane's own of the plane before: populations, and of grad its in-plane
    // part with the share of the plane below (x, y), minus that share (z), and
    // its own share of its neighbours' (x, y, z)
    __shared__ real park[NW][kQ + 6][64];
    const int bx = blockIdx.x & 7, bl = blockIdx.x >> 3;
    const int t = (bl / a.xgroup * 8 + bx) * a.xgroup + bl % a.xgroup;
    if (t >= a.mtiles) return;                              // uniform over the workgroup
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int ch = t % a.nch, yt = (t / a.nch) % a.nyt, seg = t / (a.nch * a.nyt);
    const int x0 = ch * 64, z0 = seg * a.depth, H = min(a.depth, nz - z0);
    const int yl = yt * a.rows - 1 + wave;
    const int y = __builtin_amdgcn_readfirstlane((yl + ny) % ny);
    const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
    const bool out = wave >= 1 && wave <= a.rows && yl < ny;      // uniform over the wave
    // lanes past the row's end repeat its last site in everything they load and
    // store, so that no store below is conditional: then the compiler knows how
    // many stores follow the loads in flight, and waits for the loads alone
    const int wd = min(64, nx - x0), col = min(lane, wd - 1), x = x0 + col;
    const bool first = !PX && x0 == 0, last = !PX && x0 + 64 >= nx;   // uniform
    const int wall_side = PX ? -1 : (x == 0 ? 0 : (x == nx - 1 ? 1 : -1));
    const long long nyz = (long long)ny * nz;
    // the lane's halo population (halo_dir3): where it comes from in its plane
    unsigned hsrc;
    {
        const int hi = halo_dir3(lane), hc = halo_c3(hi);
        int hx = lane < 32 ? x0 - 1 : x0 + wd;              // the halo column
        if (PX) hx = hx < 0 ? nx - 1 : (hx >= nx ? 0 : hx);
        else hx = hx < 0 ? 0 : (hx >= nx ? nx - 1 : hx);
        int hsx = hx - ((hc & 3) - 1);
        if (PX) hsx = hsx < 0 ? nx - 1 : (hsx >= nx ? 0 : hsx);
        else hsx = hsx < 0 ? 0 : (hsx >= nx ? nx - 1 : hsx);
        const int cy = ((hc >> 2) & 3) - 1;
        hsrc = (unsigned)(cy > 0 ? ym : (cy < 0 ? yp : y)) * (unsigned)nx + (unsigned)hsx;
    }
    // the right halo column is the wall's own when one site follows the chunk
    const bool hwall = !PX && x0 + 65 == nx;                // uniform

    // GEO: the records of plane p's row chunk
    auto row_recs = [&](int p) __attribute__((always_inline)) -> RowRec3 {
        RowRec3 r{0, 0, 0, 0};
        if constexpr (GEO) {
            const int z = p < 0 ? p + nz : (p >= nz ? p - nz : p);
            // never written by a kernel: scalar loads
            const auto* rec = (const __attribute__((address_space(4))) int32_t*)(uintptr_t)a.rowrec + (z * ny + y) * a.nch;
            r.r0 = rec[ch];
            r.r1 = rec[ch + 1];
            r.left = rec[ch == 0 ? a.nch : ch];
            r.right = rec[ch == a.nch - 1 ? 0 : ch + 1];
        }
        return r;
    };
    auto issue = [&](int p, Plane3<real, GEO>& q, const RowRec3& rr) __attribute__((always_inline)) {
        const int z = p < 0 ? p + nz : (p >= nz ? p - nz : p), zm = z == 0 ? nz - 1 : z - 1, zp = z == nz - 1 ? 0 : z + 1;
        // what follows from the lane is formed anew for every plane: held across
        // the loop it would cost the registers that let two workgroups share a CU
        int xv = x, lv = lane;
        asm volatile("" : "+v"(xv), "+v"(lv));
        const int xm = xv == 0 ? nx - 1 : xv - 1, xp = xv == nx - 1 ? 0 : xv + 1;
        PlaneWalk w(a.src, a.stride), w0(a.wsrc, nyz), w1(a.wsrc + (PX ? 0 : 5 * nyz), nyz);
        const unsigned wrow = (unsigned)(z * ny + y) * (unsigned)sizeof(real);
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            const int zz = kCZ[i] > 0 ? zm : (kCZ[i] < 0 ? zp : z), yy = kCY[i] > 0 ? ym : (kCY[i] < 0 ? yp : y);
            const unsigned r = (unsigned)(zz * ny + yy) * (unsigned)nx;      // uniform
            // between walls the neighbours of every lane that keeps them are next to
            // it (a wall site's outer one is the wall's part); a periodic row wraps
            const unsigned off = (r + (unsigned)(!PX || kCX[i] == 0 ? xv : (kCX[i] > 0 ? xm : xp))) * (unsigned)sizeof(real);
            const int next = PX ? 0 : -kCX[i] * (int)sizeof(real);
            if (!PX && kCX[i] != 0 && (kCX[i] > 0 ? first : last)) {         // uniform
                const bool ret = kCX[i] > 0 ? xv == 0 : xv == nx - 1;
                gptr3<char> src = ret ? (kCX[i] > 0 ? w0.base : w1.base) + wrow : w.base + off + next;
                q.g[i] = *(gptr3<const real>)src;
            } else {
                q.g[i] = *(gptr3<const real>)(w.base + off + next);
            }
            w.next();
            if (!PX && kCX[i] > 0) w0.next();
            if (!PX && kCX[i] < 0) w1.next();
        }
        const int hi = halo_dir3(lv), cz = (halo_c3(hi) >> 4) - 1;
        const real* hp = a.src + hi * a.stride + ((unsigned)((cz > 0 ? zm : (cz < 0 ? zp : z)) * ny) * (unsigned)nx + hsrc);
        if (!PX && hwall && halo_ret3(lv)) {
            const int hm = hi == 2 ? 0 : (hi - 6) / 2;      // 2 8 10 12 14 -> 0..4
            hp = a.wsrc + ((5 + hm) * nyz + ((long long)z * ny + y));
        }
        q.halo = *(gptr3<const real>)hp;
        if constexpr (GEO) {
            const unsigned r = (unsigned)(z * ny + y) * (unsigned)nx;
            q.fl = a.flags[r + (unsigned)xv];
            const unsigned hx = lv < 32 ? (x0 == 0 ? nx - 1 : x0 - 1) : (x0 + wd >= nx ? 0 : x0 + wd);
            q.hfl = a.flags[r + hx];
            // (A, s_kappa): one link a lane, repeating the first where there are fewer
            const int l = rr.r0 + lv < rr.r1 ? rr.r0 + lv : min(rr.r0, a.nlinks - 1);
            q.la = a.lval[2 * (long long)l];
            q.ls = a.lval[2 * (long long)l + 1];
            int hl = lv < 32 ? rr.left - 18 + min(lv, 17) : rr.right + min(lv - 32, 17);
            hl = max(0, min(hl, a.nlinks - 1));
            q.ha = a.lval[2 * (long long)hl];
            q.hs = a.lval[2 * (long long)hl + 1];
        }
    };
    // GEO: the cut links' returning populations of the row and of its halo sites
    // (cut_links3's arithmetic), nothing at void sites
    auto cut_pulls = [&](Plane3<real, GEO>& q, const RowRec3& rr) __attribute__((always_inline)) {
        if constexpr (GEO) {
            if (rr.r1 > rr.r0) {                            // uniform
                pairs[wave][lane][0] = q.la;
                pairs[wave][lane][1] = q.ls;
                const uint32_t m = q.fl & kCutMask3;
                // the links of the lanes before: the bits of every lane's count
                const uint32_t n = lane < wd ? (uint32_t)__builtin_popcount(m) : 0u;
                int before = 0;
#pragma unroll
                for (int b = 0; b < 5; ++b) {
                    const unsigned long long v = __ballot((n >> b) & 1u);
                    before += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)v, 0u)) << b;
                }
                before = __shfl(before, col);
                const bool many = rr.r1 - rr.r0 > 64;       // uniform
#pragma unroll
                for (int p = 0; p < 9; ++p) {
                    const int k = 2 * p + 1;
                    const uint32_t b = (m >> (k - 1)) & 3u;
                    const int l = before + __builtin_popcount(m & ((1u << (k - 1)) - 1u)), l1 = l + (int)(b & 1u);
                    real A = pairs[wave][l & 63][0], s = pairs[wave][l & 63][1];
                    real A1 = pairs[wave][l1 & 63][0], s1 = pairs[wave][l1 & 63][1];
                    if (many) {
                        const real* v = a.lval + 2 * (long long)(rr.r0 + l);
                        if ((b & 1u) && l >= 64) { A = v[0]; s = v[1]; }
                        const real* v1 = a.lval + 2 * (long long)(rr.r0 + l1);
                        if ((b & 2u) && l1 >= 64) { A1 = v1[0]; s1 = v1[1]; }
                    }
                    const real gk = q.g[k], gb = q.g[k + 1];
                    q.g[k + 1] = (b & 1u) ? A + s * gk : gb;
                    q.g[k] = (b & 2u) ? A1 + s1 * gb : gk;
                }
            }
            if (__any((q.fl & kVoid3) != 0u)) {
                const bool v = (q.fl & kVoid3) != 0u;
#pragma unroll
                for (int i = 0; i < kQ; ++i) q.g[i] = v ? real(0) : q.g[i];
            }
            const uint32_t hm = q.hfl & kCutMask3;
            if (__any(hm != 0u)) {
                // lane i (32 + i): population i returned by link k = opp(i)
                const int i = halo_dir3(lane), k = i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1);
                const int rank = __builtin_popcount(hm & (k > 0 ? (1u << (k - 1)) - 1u : 0u));
                const int from = lane < 32 ? 18 - __builtin_popcount(hm) + rank : 32 + rank;
                const real A = __shfl(q.ha, from & 63), s = __shfl(q.hs, from & 63);
                const real gk = __shfl(q.halo, (lane & 32) + k);
                if (k > 0 && ((hm >> (k - 1)) & 1u)) q.halo = A + s * gk;
            }
        }
    };
    // plane p (in q) has arrived: the walls' returning populations, its density
    // into LDS with the halo columns', the populations into `park` (inner
    // waves), then plane `next` on its way into q
    auto arrive = [&](Plane3<real, GEO>& q, int slot, int next, bool keep, const RowRec3& rr, const RowRec3& rn) __attribute__((always_inline)) -> real {
        if constexpr (GEO) {
            cut_pulls(q, rr);
        }
        if (!PX && first) {
            const real s = x == 0 ? a.wskap[0] : real(0);   // other lanes keep their pulls
#pragma unroll
            for (int m = 0; m < 5; ++m) q.g[wall_pair3(m)] += s * q.g[wall_pair3(m) + 1];
        }
        if (!PX && last) {
            const real s = x == nx - 1 ? a.wskap[1] : real(0);
#pragma unroll
            for (int m = 0; m < 5; ++m) q.g[wall_pair3(m) + 1] += s * q.g[wall_pair3(m)];
        }
        if (!PX && hwall) {
            const real gl = __shfl(q.halo, (lane - 1) & 63);
            if (halo_ret3(lane)) q.halo += a.wskap[1] * gl;
        }
        const real dr = sum3(q.g);
        const real hs = half_sum3((lane & 31) < kQ ? q.halo : real(0));
        if (keep) {
#pragma unroll
            for (int i = 0; i < kQ; ++i) park[wave][i][lane] = q.g[i];
        }
        issue(next, q, rn);
        __builtin_amdgcn_sched_barrier(0);
        dens[slot][wave][1 + col] = dr;
        if ((lane & 31) == 0) dens[slot][wave][lane ? 1 + wd : 0] = hs;
        lds_barrier();
        return dr;
    };

    Plane3<real, GEO> q;
    // the records of the plane that arrives, of the one whose loads go out then
    // and (rs) of the one that arrived before
    RowRec3 rr = row_recs(z0 - 1), rn = row_recs(z0), rs = rr;
    issue(z0 - 1, q, rr);
    auto next_recs = [&](int m) __attribute__((always_inline)) {
        rs = rr;
        rr = rn;
        rn = row_recs(z0 + min(m + 1, H));
    };
    if (!out) {
        // a row of halo: densities only; as many barriers as the others
        for (int m = 0; m <= H + 1; ++m) {
            arrive(q, m & (RING - 1), z0 + min(m, H), false, rr, rn);
            next_recs(m);
        }
        return;
    }
    uint32_t fl = 0u, flp = 0u;                             // flags of the stepped plane and of the arriving one
    bool bad = false;
    auto plane_grad = [&](int slot, real dr) __attribute__((always_inline)) {
        const real (*d)[68] = dens[slot];
        return plane_terms3(dr, d[wave][col + 2], d[wave][col], d[wave + 1][col + 1], d[wave - 1][col + 1],
                            d[wave + 1][col + 2], d[wave + 1][col], d[wave - 1][col + 2], d[wave - 1][col],
                            !PX && (first || last) ? wall_side : -1);
    };
    real (*own)[64] = park[wave];
    auto carry = [&](const PlaneTerms3<real>& t, real sx1, real sy1, real t1) __attribute__((always_inline)) {
        own[kQ][lane] = with_share3(t.gx, sx1);
        own[kQ + 1][lane] = with_share3(t.gy, sy1);
        own[kQ + 2][lane] = t1;
        own[kQ + 3][lane] = t.sx;
        own[kQ + 4][lane] = t.sy;
        own[kQ + 5][lane] = t.tz;
    };
    for (int m = 0; m < 2; ++m) {
        if constexpr (GEO) flp = q.fl;
        const PlaneTerms3<real> t = plane_grad(m, arrive(q, m, z0 + m, m == 1, rr, rn));
        next_recs(m);
        const bool below = m > 0;
        carry(t, below ? own[kQ + 3][lane] : real(0), below ? own[kQ + 4][lane] : real(0),
              below ? own[kQ + 5][lane] : real(0));
    }
    // plane z0 - 1 + m arrives, plane zc before it is stepped
    auto advance = [&](int m) __attribute__((always_inline)) {
        const int zc = z0 + m - 2;
        const unsigned s = (unsigned)(zc * ny + y) * (unsigned)nx + (unsigned)x;
        real cur[kQ];
#pragma unroll
        for (int i = 0; i < kQ; ++i) cur[i] = park[wave][i][lane];
        if constexpr (GEO) {
            fl = flp;
            flp = q.fl;
        }
        // the stepped row's records, the first 64 now: they arrive while the row
        // is stepped
        const int sr0 = rs.r0, sr1 = rs.r1;
        Link3<real> first64;
        if constexpr (GEO)
            if (sr1 > sr0) first64 = a.links[min(sr0 + lane, sr1 - 1)];
        const int slot = m & (RING - 1);
        const PlaneTerms3<real> t = plane_grad(slot, arrive(q, slot, z0 + min(m, H), true, rr, rn));
        next_recs(m);
        const int slot1 = (m - 1) & (RING - 1);
        const real dr1 = dens[slot1][wave][1 + col];        // the stepped plane's, left there one plane ago
        real grad[3];
        grad[0] = with_share3(own[kQ][lane], t.sx);
        if (!PX && (first || last)) grad[0] += wall_grad3(wall_side, dr1);
        grad[1] = with_share3(own[kQ + 1][lane], t.sy);
        grad[2] = t.tz - own[kQ + 2][lane];
        if constexpr (GEO) {
            if (__any((fl & kCutMask3) != 0u)) {
                const int slot2 = (m - 2) & (RING - 1);
                real nb[kQ], gc[3];
#pragma unroll
                for (int i = 1; i < kQ; ++i)
                    nb[i] = dens[kCZ[i] > 0 ? slot : (kCZ[i] < 0 ? slot2 : slot1)][wave + kCY[i]][1 + col + kCX[i]];
                grad_nb3<true>(nb, dr1, fl, -1, gc);
#pragma unroll
                for (int k = 0; k < 3; ++k) grad[k] = (fl & kCutMask3) ? gc[k] : grad[k];
            }
        }
        carry(t, own[kQ + 3][lane], own[kQ + 4][lane], own[kQ + 5][lane]);
        const real ir = recip3(real(1) + dr1);
        real o[kQ], j[3];
        collide_pairs3(cur, dr1, grad, a.ml * ir, a.F, a.omega, a.omega_h, j, o);
        const bool live = !GEO || !(fl & kVoid3);           // void sites stay at rest
        bad |= live && !(fabs(dr1) + fabs(j[0]) + fabs(j[1]) + fabs(j[2]) < real(kDivergeBound));
        PlaneWalk w(a.dst, a.stride);
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
            w.template store<STREAM>(s * (unsigned)sizeof(real), live ? o[i] : real(0));
            w.next();
        }
        PlaneWalk wu(a.U, a.stride);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (lane < wd && live) wu.add(s * 8u, (double)(j[k] * ir));
            wu.next();
        }
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (PX || !(side ? last : first)) continue;     // uniform
            if (wall_side != side) continue;
            real A[5];
            wall_parts3(a, side, a.wval_next[side], o, A);
            PlaneWalk ww(a.wdst + side * 5 * nyz, nyz);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                ww.template store<STREAM>((unsigned)(zc * ny + y) * (unsigned)sizeof(real), A[k]);
                ww.next();
            }
        }
        if constexpr (GEO) {
            // A of the row's cut links for the next step, one link a lane, from the
            // post-collision populations of its site's lane
            const unsigned base = (unsigned)(zc * ny + y) * (unsigned)nx + (unsigned)x0;
            if (STAGE && sr1 > sr0) {
#pragma unroll
                for (int i = 0; i < kQ; ++i) stage[wave][i][lane] = o[i];
            }
            for (int r = sr0; r < sr1; r += 64) {           // uniform
                const int l = min(r + lane, sr1 - 1);
                Link3<real> L = first64;
                if (r > sr0) L = a.links[l];
                const int from = (int)((unsigned)L.site - base);
                const int k = (int)(L.meta & 31u), kb = (int)((L.meta >> 5) & 31u);
                real h[kQ], hk = real(0), hb = real(0);
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    if constexpr (STAGE) {
                        h[i] = stage[wave][i][from];
                    } else {
                        h[i] = __shfl(o[i], from);
                        if (i == k) hk = h[i];
                        if (i == kb) hb = h[i];
                    }
                }
                if constexpr (STAGE) {
                    hk = stage[wave][k][from];
                    hb = stage[wave][kb][from];
                }
                real hd, hj[3], hP[6];
                moments3(h, hd, hj, hP);
                const real A = link_part3(L, hk, hb, hd, hd, hP, profile[(L.meta >> 19) & 15u]);
                const bool ext = (L.meta >> 12) & 1u;       // k3_links_ext's
                if (r + lane < sr1 && !ext) {
                    a.lval_next[2 * (long long)l] = A;
                    a.lval_next[2 * (long long)l + 1] = ((L.meta >> 10) & 3u) == kWallDirichlet ? L.kap : -L.kap;
                }
            }
        }
    };
    // the first one apart: in the loop the loads in flight always have a
    // plane's stores behind them
    advance(2);
    for (int m = 3; m <= H + 1; ++m) advance(m);
    if (__any(bad) && lane == 0 && *(volatile unsigned int*)a.diverged == 0u) atomicOr(a.diverged, 1u);
}

// Where a readout goes: arrays of the caller (null: not wanted), u [3][n]
// doubles, the moments T with their lattice-to-user scales.
template <typename T>
struct Readout3Dst {
    double* u;
    T *rho, *j, *P, *sigma;
    double s_rho, s_j, s_sigma;
};

// Readout at every site: rho, j (with S/2), P, the Cauchy stress
// sigma = -P - (lambda - mu) drho I and the displacement U + (j/rho)/2, what
// is wanted of them, scaled and stored where the caller wants it.  Needs
// k3_density of the same state first.  Void sites read zero.
// Bound by HBM: after the density pass it reads the pulls (and U for the
// displacement) once and writes each result once; the earlier chain wrote all
// 19 planes in double precision and scaled the wanted ones in a second pass.
// 256^3 slab, fp32, displacement: 0.44 ms against 1.00 (density pass apart);
// 256^3 porous solid, fp32 moments: 0.49 against 1.48.
template <typename real, bool PX, bool GEO, typename T>
__global__ __launch_bounds__(256) void k3_readout(Step3Args<real> a, Readout3Dst<T> d)
{
    const int tile = xcd_group3<GEO>(turn(blockIdx.x, gridDim.x, a.back)) * 4 + (threadIdx.x >> 6);
    if (tile >= a.ntiles) return;
    const Site3 st = site_of(tile, threadIdx.x & 63, a.nx, a.ny);
    real g[kQ];
    uint32_t fl;
    pull3<real, PX, GEO>(a, st, g, fl);
    real dr, j[3], P[6];
    moments3(g, dr, j, P);
    real grad[3];
    grad3<real, PX, GEO>(a, st, dr, grad, fl);
    const real rho = real(1) + dr;
    const real c = a.ml / rho;
    if (!st.in) return;
    const unsigned s = sidx3(st.x, st.y, st.z, a.nx, a.ny);
    const size_t n = (size_t)a.plane;
    const bool live = !(GEO && (fl & kVoid3));              // void sites report zeros (rho too)
    if (d.rho) d.rho[s] = (T)(live ? ((double)dr + 1.0) * d.s_rho : 0.0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double jk = (double)j[k] + 0.5 * ((double)a.F[k] + (double)c * (double)grad[k]);
        if (d.j) d.j[k * n + s] = (T)(live ? jk * d.s_j : 0.0);
        if (d.u) d.u[k * n + s] = live ? a.U[k * a.stride + s] + 0.5 * jk / (double)rho : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        if (d.P) d.P[k * n + s] = (T)(live ? (double)P[k] * d.s_sigma : 0.0);
        if (d.sigma)
            d.sigma[k * n + s] =
                (T)(live ? (-(double)P[k] - (k < 3 ? (double)a.lm * (double)dr : 0.0)) * d.s_sigma : 0.0);
    }
}

// delta-rho of the initial fields into the density buffer (k3_init's stencil).
template <typename real>
__global__ __launch_bounds__(256) void k3_set_dens(Step3Args<real> a, const double* in)
{
    const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < a.plane) a.dens[s] = (real)in[s];
}

// Initial state from fields (lattice units, double, planes of `in`): 0
// delta-rho, 1-3 j, 4-9 P, 10-12 u0; dens must hold delta-rho.  Populations
// g = g_eq(drho, j - S/2, P) at the sites themselves (the state is "local"),
// U = u0 - (j/rho)/2.
template <typename real, bool PX, bool GEO = false>
__global__ __launch_bounds__(256) void k3_init(Step3Args<real> a, const double* in)
{
    const int tile = xcd_group3<GEO>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (tile >= a.ntiles) return;
    const Site3 st = site_of(tile, threadIdx.x & 63, a.nx, a.ny);
    const unsigned s = sidx3(st.x, st.y, st.z, a.nx, a.ny);
    const long long n = a.plane;
    const uint32_t fl = GEO ? a.flags[s] : 0u;
    if (GEO && (fl & kVoid3)) {                             // void: the rest state, no displacement
        if (st.in) {
            for (int k = 0; k < kQ; ++k) a.dst[k * a.stride + s] = real(0);
            for (int k = 0; k < 3; ++k) a.U[k * a.stride + s] = 0.0;
        }
        return;
    }
    const real dr = (real)in[s];
    real grad[3];
    grad3<real, PX, GEO>(a, st, dr, grad, fl);
    const double rho = 1.0 + in[s];
    const real c = a.ml / (real)rho;
    real j[3], P[6];
    for (int k = 0; k < 3; ++k) j[k] = (real)(in[(1 + k) * n + s] - 0.5 * ((double)a.F[k] + (double)(c * grad[k])));
    for (int k = 0; k < 6; ++k) P[k] = (real)in[(4 + k) * n + s];
    if (!st.in) return;
    real* d = a.dst;
#define SLBM3_INIT(k) d[k * a.stride + s] = geq3<k, real>(dr, j, P);
    SLBM3_INIT(0) SLBM3_INIT(1) SLBM3_INIT(2) SLBM3_INIT(3) SLBM3_INIT(4) SLBM3_INIT(5) SLBM3_INIT(6)
    SLBM3_INIT(7) SLBM3_INIT(8) SLBM3_INIT(9) SLBM3_INIT(10) SLBM3_INIT(11) SLBM3_INIT(12)
    SLBM3_INIT(13) SLBM3_INIT(14) SLBM3_INIT(15) SLBM3_INIT(16) SLBM3_INIT(17) SLBM3_INIT(18)
#undef SLBM3_INIT
    for (int k = 0; k < 3; ++k) a.U[k * a.stride + s] = in[(10 + k) * n + s] - 0.5 * in[(1 + k) * n + s] / rho;
}

}  // namespace slbm3_dev
