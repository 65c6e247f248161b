// Adjoint (vector-Jacobian product) sums of the single- and double-layer
// kernels, float64, on the pair-sum skeleton of pairsum.hpp.
//
// Notation: a forward sum u_n = pref sum_m' K(x_n - y_m) q_m with q_m = w_m f_m
// (single layer, pref = c = 1/(8 pi mu)) or u_n = d sum_m' r (r.n_m)(r.q_m)/rho^5
// (double layer, d = 6/(8 pi)); g_n = dL/du_n.  The gradients are those of the
// definitions, differentiated by hand:
//   single layer, K(r;a,b) = [(r.b)a + (r.a)b - (a.b)r]/rho^3 - 3(r.a)(r.b)r/rho^5
//     dL/dx_n = c sum_m K(r_nm; g_n, q_m)
//     dL/df_m = c w_m sum_n S(r_nm) g_n          (S symmetric and even in r)
//     dL/dy_m = -c sum_n K(r_nm; g_n, q_m) = c sum_n K(r_mn; g_n, q_m)  (K odd)
//   double layer, G(r) = grad_r[(r.n)(r.q)(r.g)/rho^5]
//                      = [(r.q)(r.g)n + (r.n)(r.g)q + (r.n)(r.q)g]/rho^5 - 5(r.n)(r.q)(r.g) r/rho^7
//     dL/dx_n   = d sum_m G(r_nm)
//     dL/dphi_m = d w_m sum_n r_nm (r_nm.n_m)(r_nm.g_n)/rho^5
//     dL/dy_m   = -d sum_n G(r_nm)              (G even)
// Source-side gradients are transposed passes: the forward's sources act as
// targets and its targets (carrying g) as sources; when only the density
// gradient is asked for, a lighter pass skips the position terms.  The double
// layer's target side together with any of its source side is one sweep over the
// pairs (dl_both_main).  For a shared point set
// with one combined position gradient, a single fused pass gives
// dL/dx_p = c sum_m [K(r_pm; g_p, q_m) + K(r_pm; q_p, g_m)] and dL/df_p.
#include <algorithm>
#include <string>
#include <type_traits>

#include "../../include/stokes_mi355x.h"
#include "pairsum.hpp"
#include "vjp.hpp"

namespace stokes {
namespace {

using ps::PassArgs;
using ps::rinv;
using ps::rinv_masked;

__device__ __forceinline__ double dot3(double ax, double ay, double az, double bx, double by, double bz) {
    return __builtin_fma(ax, bx, __builtin_fma(ay, by, az * bz));
}

template <bool M>
__device__ __forceinline__ double ri_of(double r2, bool skip) {
    return M ? rinv_masked(r2, skip || r2 == 0.0) : rinv(r2);
}

__device__ __forceinline__ void out3(const PassArgs& a, double* out, int64_t n, int64_t i, double s,
                                     double vx, double vy, double vz) {
    if (!out) return;
    if (a.accumulate || out == a.force_acc) {
        out[i] += s * vx;
        out[n + i] += s * vy;
        out[2 * n + i] += s * vz;
    } else {
        out[i] = s * vx;
        out[n + i] = s * vy;
        out[2 * n + i] = s * vz;
    }
}

// ---- single layer, target side: dL/dx_n --------------------------------------
// targets: trg_xyz, tv[0] = g (3, nt); sources: src_xyz, sv[0] = density, sv[1] = weight
struct SlT {
    struct alignas(16) Rec { double x, y, z, qx, qy, qz; };
    static constexpr int NACC = 3, NT = 3;
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        const int64_t n = a.n_src;
        const double w = a.sv[1][i];
        r.x = pos[0] = a.src_xyz[i];
        r.y = pos[1] = a.src_xyz[n + i];
        r.z = pos[2] = a.src_xyz[2 * n + i];
        r.qx = w * a.sv[0][i];
        r.qy = w * a.sv[0][n + i];
        r.qz = w * a.sv[0][2 * n + i];
    }
    __device__ static void pad_rec(Rec& r) {
        r.x = r.y = r.z = kPadPos;
        r.qx = r.qy = r.qz = 0.0;
    }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        v[0] = a.tv[0][i]; v[1] = a.tv[0][n + i]; v[2] = a.tv[0][2 * n + i];
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&g)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri, ri3 = ri2 * ri;
        const double rb = dot3(dx, dy, dz, s.qx, s.qy, s.qz);
        const double ra = dot3(dx, dy, dz, g[0], g[1], g[2]);
        const double ab = dot3(g[0], g[1], g[2], s.qx, s.qy, s.qz);
        const double s1 = rb * ri3, s2 = ra * ri3;
        const double s3 = -ri3 * __builtin_fma(ra * rb, 3.0 * ri2, ab);
        acc[0] = __builtin_fma(s1, g[0], __builtin_fma(s2, s.qx, __builtin_fma(s3, dx, acc[0])));
        acc[1] = __builtin_fma(s1, g[1], __builtin_fma(s2, s.qy, __builtin_fma(s3, dy, acc[1])));
        acc[2] = __builtin_fma(s1, g[2], __builtin_fma(s2, s.qz, __builtin_fma(s3, dz, acc[2])));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        out3(a, a.out[0], a.n_trg, i, a.pref, s[0], s[1], s[2]);
    }
};

// ---- single layer, source side: dL/df_m and dL/dy_m ----------------------------
// pass targets: the forward's sources (trg_xyz = src positions, tv[0] = density,
// tv[1] = weight); pass sources: the forward's targets (src_xyz = trg positions,
// sv[0] = g).  r = y_m - x_n.
struct SlS {
    struct alignas(16) Rec { double x, y, z, gx, gy, gz; };
    static constexpr int NACC = 6, NT = 3;
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        const int64_t n = a.n_src;
        r.x = pos[0] = a.src_xyz[i];
        r.y = pos[1] = a.src_xyz[n + i];
        r.z = pos[2] = a.src_xyz[2 * n + i];
        r.gx = a.sv[0][i];
        r.gy = a.sv[0][n + i];
        r.gz = a.sv[0][2 * n + i];
    }
    __device__ static void pad_rec(Rec& r) {
        r.x = r.y = r.z = kPadPos;
        r.gx = r.gy = r.gz = 0.0;
    }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        const double w = a.tv[1][i];
        v[0] = w * a.tv[0][i]; v[1] = w * a.tv[0][n + i]; v[2] = w * a.tv[0][2 * n + i];
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&q)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri, ri3 = ri2 * ri;
        const double ra = dot3(dx, dy, dz, s.gx, s.gy, s.gz);   // r . g_n
        const double rb = dot3(dx, dy, dz, q[0], q[1], q[2]);   // r . q_m
        const double ab = dot3(s.gx, s.gy, s.gz, q[0], q[1], q[2]);
        const double sa = ra * ri3, sb = rb * ri3;
        // S(r) g = g/rho + r (r.g)/rho^3
        acc[0] = __builtin_fma(s.gx, ri, __builtin_fma(sa, dx, acc[0]));
        acc[1] = __builtin_fma(s.gy, ri, __builtin_fma(sa, dy, acc[1]));
        acc[2] = __builtin_fma(s.gz, ri, __builtin_fma(sa, dz, acc[2]));
        // K(r; g, q)
        const double s3 = -ri3 * __builtin_fma(ra * rb, 3.0 * ri2, ab);
        acc[3] = __builtin_fma(sb, s.gx, __builtin_fma(sa, q[0], __builtin_fma(s3, dx, acc[3])));
        acc[4] = __builtin_fma(sb, s.gy, __builtin_fma(sa, q[1], __builtin_fma(s3, dy, acc[4])));
        acc[5] = __builtin_fma(sb, s.gz, __builtin_fma(sa, q[2], __builtin_fma(s3, dz, acc[5])));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        const double w = a.tv[1][i];
        out3(a, a.out[0], a.n_trg, i, a.pref * w, s[0], s[1], s[2]);
        out3(a, a.out[1], a.n_trg, i, a.pref, s[3], s[4], s[5]);
    }
};

// ---- single layer, shared point set: dL/df_p and the total dL/dx_p ------------
// targets = sources: trg_xyz, tv[0] = g, tv[1] = density, tv[2] = weight;
// records carry (y_m, q_m, g_m) from the same arrays (sv mirrors tv).
struct SlSym {
    struct alignas(16) Rec { double x, y, z, qx, qy, qz, gx, gy, gz, pad; };
    static constexpr int NACC = 8, NT = 6;   // acc: B(3), V(3), coef of g_p, coef of q_p
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        const int64_t n = a.n_src;
        const double w = a.sv[1][i];
        r.x = pos[0] = a.src_xyz[i];
        r.y = pos[1] = a.src_xyz[n + i];
        r.z = pos[2] = a.src_xyz[2 * n + i];
        r.qx = w * a.sv[0][i];
        r.qy = w * a.sv[0][n + i];
        r.qz = w * a.sv[0][2 * n + i];
        r.gx = a.sv[2][i];
        r.gy = a.sv[2][n + i];
        r.gz = a.sv[2][2 * n + i];
        r.pad = 0.0;
    }
    __device__ static void pad_rec(Rec& r) {
        r.x = r.y = r.z = kPadPos;
        r.qx = r.qy = r.qz = r.gx = r.gy = r.gz = r.pad = 0.0;
    }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        const double w = a.tv[2][i];
        v[0] = a.tv[0][i]; v[1] = a.tv[0][n + i]; v[2] = a.tv[0][2 * n + i];
        v[3] = w * a.tv[1][i]; v[4] = w * a.tv[1][n + i]; v[5] = w * a.tv[1][2 * n + i];
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&v)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri, ri3 = ri2 * ri;
        const double rqm = dot3(dx, dy, dz, s.qx, s.qy, s.qz);
        const double rgm = dot3(dx, dy, dz, s.gx, s.gy, s.gz);
        const double rgp = dot3(dx, dy, dz, v[0], v[1], v[2]);
        const double rqp = dot3(dx, dy, dz, v[3], v[4], v[5]);
        // g_p . q_m + q_p . g_m as one chain of six products
        const double ab = __builtin_fma(v[0], s.qx, __builtin_fma(v[1], s.qy, __builtin_fma(v[2], s.qz,
                          __builtin_fma(v[3], s.gx, __builtin_fma(v[4], s.gy, v[5] * s.gz)))));
        const double sgm = rgm * ri3;
        // B += S(r) g_m
        acc[0] = __builtin_fma(s.gx, ri, __builtin_fma(sgm, dx, acc[0]));
        acc[1] = __builtin_fma(s.gy, ri, __builtin_fma(sgm, dy, acc[1]));
        acc[2] = __builtin_fma(s.gz, ri, __builtin_fma(sgm, dz, acc[2]));
        // K(r; g_p, q_m) + K(r; q_p, g_m): g_p and q_p terms as scalar coefficients
        acc[6] = __builtin_fma(rqm, ri3, acc[6]);
        acc[7] += sgm;
        const double sq = rgp * ri3, sg = rqp * ri3;
        const double cr = -ri3 * __builtin_fma(__builtin_fma(rgp, rqm, rqp * rgm), 3.0 * ri2, ab);
        acc[3] = __builtin_fma(sq, s.qx, __builtin_fma(sg, s.gx, __builtin_fma(cr, dx, acc[3])));
        acc[4] = __builtin_fma(sq, s.qy, __builtin_fma(sg, s.gy, __builtin_fma(cr, dy, acc[4])));
        acc[5] = __builtin_fma(sq, s.qz, __builtin_fma(sg, s.gz, __builtin_fma(cr, dz, acc[5])));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        const int64_t n = a.n_trg;
        const double w = a.tv[2][i];
        out3(a, a.out[0], n, i, a.pref * w, s[0], s[1], s[2]);
        const double g[3] = {a.tv[0][i], a.tv[0][n + i], a.tv[0][2 * n + i]};
        const double q[3] = {w * a.tv[1][i], w * a.tv[1][n + i], w * a.tv[1][2 * n + i]};
        out3(a, a.out[1], n, i, a.pref, __builtin_fma(s[6], g[0], __builtin_fma(s[7], q[0], s[3])),
             __builtin_fma(s[6], g[1], __builtin_fma(s[7], q[1], s[4])),
             __builtin_fma(s[6], g[2], __builtin_fma(s[7], q[2], s[5])));
    }
};

// ---- double layer, target side: dL/dx_n ---------------------------------------
// targets: trg_xyz, tv[0] = g; sources: src_xyz, sv[0] = density, sv[1] = weight, sv[2] = normal
struct DlT {
    struct alignas(16) Rec { double x, y, z, qx, qy, qz, nx, ny, nz, pad; };
    static constexpr int NACC = 4, NT = 3;   // V(3), coefficient of g_n
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        const int64_t n = a.n_src;
        const double w = a.sv[1][i];
        r.x = pos[0] = a.src_xyz[i];
        r.y = pos[1] = a.src_xyz[n + i];
        r.z = pos[2] = a.src_xyz[2 * n + i];
        r.qx = w * a.sv[0][i];
        r.qy = w * a.sv[0][n + i];
        r.qz = w * a.sv[0][2 * n + i];
        r.nx = a.sv[2][i];
        r.ny = a.sv[2][n + i];
        r.nz = a.sv[2][2 * n + i];
        r.pad = 0.0;
    }
    __device__ static void pad_rec(Rec& r) {
        r.x = r.y = r.z = kPadPos;
        r.qx = r.qy = r.qz = r.nx = r.ny = r.nz = r.pad = 0.0;
    }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        v[0] = a.tv[0][i]; v[1] = a.tv[0][n + i]; v[2] = a.tv[0][2 * n + i];
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&g)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri, ri5 = ri2 * ri2 * ri;
        const double rn = dot3(dx, dy, dz, s.nx, s.ny, s.nz);
        const double rq = dot3(dx, dy, dz, s.qx, s.qy, s.qz);
        const double rg = dot3(dx, dy, dz, g[0], g[1], g[2]);
        const double t = rg * ri5;
        const double cn = rq * t, cq = rn * t;
        const double rnrq = rn * rq;
        acc[3] = __builtin_fma(rnrq, ri5, acc[3]);
        const double cr = (rnrq * t) * (-5.0 * ri2);
        acc[0] = __builtin_fma(cn, s.nx, __builtin_fma(cq, s.qx, __builtin_fma(cr, dx, acc[0])));
        acc[1] = __builtin_fma(cn, s.ny, __builtin_fma(cq, s.qy, __builtin_fma(cr, dy, acc[1])));
        acc[2] = __builtin_fma(cn, s.nz, __builtin_fma(cq, s.qz, __builtin_fma(cr, dz, acc[2])));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        const int64_t n = a.n_trg;
        out3(a, a.out[0], n, i, a.pref, __builtin_fma(s[3], a.tv[0][i], s[0]),
             __builtin_fma(s[3], a.tv[0][n + i], s[1]), __builtin_fma(s[3], a.tv[0][2 * n + i], s[2]));
    }
};

// ---- double layer, source side: dL/dphi_m and dL/dy_m ---------------------------
// pass targets: the forward's sources (trg_xyz = src positions, tv[0] = density,
// tv[1] = weight, tv[2] = normal); pass sources: the forward's targets
// (src_xyz = trg positions, sv[0] = g).  r = y_m - x_n = -r_nm.
struct DlS {
    struct alignas(16) Rec { double x, y, z, gx, gy, gz; };
    static constexpr int NACC = 8, NT = 6;   // P(3), V(3), coef of n_m, coef of q_m
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        const int64_t n = a.n_src;
        r.x = pos[0] = a.src_xyz[i];
        r.y = pos[1] = a.src_xyz[n + i];
        r.z = pos[2] = a.src_xyz[2 * n + i];
        r.gx = a.sv[0][i];
        r.gy = a.sv[0][n + i];
        r.gz = a.sv[0][2 * n + i];
    }
    __device__ static void pad_rec(Rec& r) {
        r.x = r.y = r.z = kPadPos;
        r.gx = r.gy = r.gz = 0.0;
    }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        const double w = a.tv[1][i];
        v[0] = a.tv[2][i]; v[1] = a.tv[2][n + i]; v[2] = a.tv[2][2 * n + i];            // n_m
        v[3] = w * a.tv[0][i]; v[4] = w * a.tv[0][n + i]; v[5] = w * a.tv[0][2 * n + i];  // q_m
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&v)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri, ri5 = ri2 * ri2 * ri;
        const double rn = dot3(dx, dy, dz, v[0], v[1], v[2]);
        const double rq = dot3(dx, dy, dz, v[3], v[4], v[5]);
        const double rg = dot3(dx, dy, dz, s.gx, s.gy, s.gz);
        const double t = rg * ri5;
        const double c1 = rn * t;                 // (r.n)(r.g)/rho^5
        // P += r (r.n)(r.g)/rho^5
        acc[0] = __builtin_fma(c1, dx, acc[0]);
        acc[1] = __builtin_fma(c1, dy, acc[1]);
        acc[2] = __builtin_fma(c1, dz, acc[2]);
        // G(r): n_m and q_m terms as scalar coefficients
        acc[6] = __builtin_fma(rq, t, acc[6]);
        acc[7] += c1;
        const double rnrq = rn * rq;
        const double cg = rnrq * ri5;
        const double cr = (rnrq * t) * (-5.0 * ri2);
        acc[3] = __builtin_fma(cg, s.gx, __builtin_fma(cr, dx, acc[3]));
        acc[4] = __builtin_fma(cg, s.gy, __builtin_fma(cr, dy, acc[4]));
        acc[5] = __builtin_fma(cg, s.gz, __builtin_fma(cr, dz, acc[5]));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        const int64_t n = a.n_trg;
        const double w = a.tv[1][i];
        // r_nm = -r: dL/dphi = -d w P, dL/dy = -d (coef_n n + coef_q q + V)
        out3(a, a.out[0], n, i, -a.pref * w, s[0], s[1], s[2]);
        const double nv[3] = {a.tv[2][i], a.tv[2][n + i], a.tv[2][2 * n + i]};
        const double q[3] = {w * a.tv[0][i], w * a.tv[0][n + i], w * a.tv[0][2 * n + i]};
        out3(a, a.out[1], n, i, -a.pref, __builtin_fma(s[6], nv[0], __builtin_fma(s[7], q[0], s[3])),
             __builtin_fma(s[6], nv[1], __builtin_fma(s[7], q[1], s[4])),
             __builtin_fma(s[6], nv[2], __builtin_fma(s[7], q[2], s[5])));
    }
};

// ---- single layer, source side, density gradient only: dL/df_m ---------------
// as SlS without the position terms
struct SlSF {
    using Rec = SlS::Rec;
    static constexpr int NACC = 3, NT = 1;
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        SlS::make_rec(a, i, r, pos);
    }
    __device__ static void pad_rec(Rec& r) { SlS::pad_rec(r); }
    __device__ static void load_t(const PassArgs&, int64_t, double (&v)[NT]) { v[0] = 0.0; }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double sa = dot3(dx, dy, dz, s.gx, s.gy, s.gz) * (ri * ri * ri);
        acc[0] = __builtin_fma(s.gx, ri, __builtin_fma(sa, dx, acc[0]));
        acc[1] = __builtin_fma(s.gy, ri, __builtin_fma(sa, dy, acc[1]));
        acc[2] = __builtin_fma(s.gz, ri, __builtin_fma(sa, dz, acc[2]));
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        out3(a, a.out[0], a.n_trg, i, a.pref * a.tv[1][i], s[0], s[1], s[2]);
    }
};

// ---- double layer, source side, density gradient only: dL/dphi_m -------------
struct DlSPhi {
    using Rec = DlS::Rec;
    static constexpr int NACC = 3, NT = 3;   // NT: n_m
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        DlS::make_rec(a, i, r, pos);
    }
    __device__ static void pad_rec(Rec& r) { DlS::pad_rec(r); }
    __device__ static void load_t(const PassArgs& a, int64_t i, double (&v)[NT]) {
        const int64_t n = a.n_trg;
        v[0] = a.tv[2][i]; v[1] = a.tv[2][n + i]; v[2] = a.tv[2][2 * n + i];
    }
    template <bool M>
    __device__ __forceinline__ static void pair(const Rec& s, double x, double y, double z, const double (&nv)[NT],
                                bool skip, double (&acc)[NACC]) {
        const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
        const double r2 = dot3(dx, dy, dz, dx, dy, dz);
        const double ri = ri_of<M>(r2, skip);
        const double ri2 = ri * ri;
        const double rn = dot3(dx, dy, dz, nv[0], nv[1], nv[2]);
        const double rg = dot3(dx, dy, dz, s.gx, s.gy, s.gz);
        const double c1 = rn * rg * (ri2 * ri2 * ri);
        acc[0] = __builtin_fma(c1, dx, acc[0]);
        acc[1] = __builtin_fma(c1, dy, acc[1]);
        acc[2] = __builtin_fma(c1, dz, acc[2]);
    }
    __device__ static void store(const PassArgs& a, int64_t i, const double (&s)[NACC]) {
        out3(a, a.out[0], a.n_trg, i, -a.pref * a.tv[1][i], s[0], s[1], s[2]);
    }
};

// ---- double layer, both sides in one sweep -------------------------------------
// One evaluation of a pair serves the target's dL/dx (V and the coefficient of
// g, as DlT) and the source's dL/dphi and dL/dy: with r = x_n - y_m
//   P_m = sum_n r (r.n_m)(r.g_n)/rho^5          dL/dphi_m = d w_m P_m
//   Y_m = sum_n G(r_nm)                          dL/dy_m   = -d Y_m
// They share the offset, 1/rho, the three dot products and G's coefficients:
// 51 float64 operations and one rsq a pair (43 without Y), against 38 and 39 in
// two passes.  Bound by those operations.
//
// A wave keeps T targets per lane in registers; a unit is one 64-source
// sub-tile against a target block.  The sub-tile's records sit in LDS; in step
// s lane l meets source (l + s) mod 64, so the 64 lanes hold 64 different
// sources, a source's sums over the lane's T targets go into the wave's own LDS
// copy by one ds_add per component, and every address has one writer per step:
// the order is fixed.  After 64 steps the four waves' copies are added in order
// and stored as the (target block, source) partial.  Sub-tiles that need the
// rules run the same steps with the masks.  Positions are doubled as in the
// direct sums (P is 8 times, G 4 times the bare sums).
//
// 61,952 wall nodes and 34,816 targets apart, all three gradients: 5.8 ms in two
// passes, 3.7 ms here (T = 6); overlapping random points, where most sub-tiles
// need the rules, 10.6 and 4.5 ms, 3,000 x 2,000 of them 495 and 86 us.
__device__ __forceinline__ void lds_add(double* p, double v) { unsafeAtomicAdd(p, v); }

template <bool M, bool SRC>
__device__ __forceinline__ void dl_both_pair(double x, double y, double z, const double (&g)[3], double (&ra)[4],
                                             const double2 (&s)[5], bool skip, double* ca) {
    const double dx = x - s[0].x, dy = y - s[0].y, dz = z - s[1].x;
    const double A = dot3(dx, dy, dz, dx, dy, dz);
    const double z0 = M && (skip || A == 0.0) ? 0.0 : __builtin_amdgcn_rsq(A);
    const double tn = A * z0;
    const double ri = z0 * __builtin_fma(-tn, z0, 3.0);             // 1/rho
    const double ri2 = ri * ri, ri5 = ri2 * ri2 * ri;
    const double rn = dot3(dx, dy, dz, s[3].x, s[3].y, s[4].x);
    const double rq = dot3(dx, dy, dz, s[1].y, s[2].x, s[2].y);
    const double rg = dot3(dx, dy, dz, g[0], g[1], g[2]);
    const double t = rg * ri5;
    const double cn = rq * t, cq = rn * t, rnrq = rn * rq, cg = rnrq * ri5;
    const double cr = (rnrq * t) * (-1.25 * ri2);
    ra[0] = __builtin_fma(cn, s[3].x, __builtin_fma(cq, s[1].y, __builtin_fma(cr, dx, ra[0])));
    ra[1] = __builtin_fma(cn, s[3].y, __builtin_fma(cq, s[2].x, __builtin_fma(cr, dy, ra[1])));
    ra[2] = __builtin_fma(cn, s[4].x, __builtin_fma(cq, s[2].y, __builtin_fma(cr, dz, ra[2])));
    ra[3] += cg;
    ca[0] = __builtin_fma(cq, dx, ca[0]);
    ca[1] = __builtin_fma(cq, dy, ca[1]);
    ca[2] = __builtin_fma(cq, dz, ca[2]);
    if constexpr (SRC) {
        ca[3] = __builtin_fma(cg, g[0], __builtin_fma(cr, dx, ca[3]));
        ca[4] = __builtin_fma(cg, g[1], __builtin_fma(cr, dy, ca[4]));
        ca[5] = __builtin_fma(cg, g[2], __builtin_fma(cr, dz, ca[5]));
        ca[6] += cn;
        ca[7] += cq;
    }
}

template <int T, bool SRC>
__global__ __launch_bounds__(kBlock, 2) void dl_both_main(PassArgs a, int64_t blk0, double* __restrict__ vpart) {
    using P = DlT;
    constexpr int BT = kBlock * T, NC = SRC ? 8 : 3, NV = SRC ? 6 : 3;
    __shared__ double2 s_rec[5][kSub];
    __shared__ int32_t s_grp[kSub];
    __shared__ double s_col[4][NC][kSub];
    static_assert(sizeof(P::Rec) == 5 * sizeof(double2), "records are staged as five double2");
    const int64_t C = 4 * a.chunks, U = a.units * 4, G = gridDim.x;
    const int64_t u0 = ps::unit_begin(blockIdx.x, U, G), u1 = ps::unit_begin(blockIdx.x + 1, U, G);
    if (u0 >= u1) return;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const bool excl = a.excl != 0;
    const int64_t npad = C * kSub;
    ps::Tgt<P, T> t;
    bool active = false;
    int64_t tbk = -1;
    double ra[T][4];
#pragma unroll
    for (int k = 0; k < T; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) ra[k][q] = 0.0;

    int64_t ub = u0 / C, sub = u0 % C;
    for (int64_t u = u0; u < u1; ++u) {
        if (ub != tbk) {
            if (tbk >= 0) ps::flush<P, T>(a, tbk, wave, lane, ra);
            tbk = ub;
            const int64_t tb = (blk0 + tbk) * BT + (int64_t)wave * (kWave * T);
            active = tb < a.n_trg;
            ps::load_tgt<P, T>(a, active ? tb : 0, lane, t);
#pragma unroll
            for (int k = 0; k < T; ++k) {
                t.x[k] *= 2.0;
                t.y[k] *= 2.0;
                t.z[k] *= 2.0;
                // lanes past the last target hold a copy of it: no cotangent, so no source term
                if (tb + (int64_t)k * kWave + lane >= a.n_trg) t.v[k][0] = t.v[k][1] = t.v[k][2] = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) ra[k][q] = 0.0;
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                t.lo[c] *= 2.0;
                t.hi[c] *= 2.0;
            }
        }
        __syncthreads();                           // the previous unit's records and sums have been read
        {
            const double2* src = reinterpret_cast<const double2*>(a.rec) + sub * (5 * kSub);
            for (int i = threadIdx.x; i < 5 * kSub; i += kBlock) s_rec[i % 5][i / 5] = src[i];
            if (threadIdx.x < kSub) s_grp[threadIdx.x] = a.grp[sub * kSub + threadIdx.x];
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) s_col[wave][q][lane] = 0.0;
        const SubMeta m = a.meta[sub];
        __syncthreads();
        if (active && m.count != 0) {
            const bool masked = ps::needs_near<P, T>(t, m, excl);
            auto steps = [&](auto mask) {
                constexpr bool M = decltype(mask)::value;
#pragma unroll 1
                for (int sp = 0; sp < kSub; ++sp) {
                    const int col = (lane + sp) & (kSub - 1);
                    double2 r[5];
#pragma unroll
                    for (int q = 0; q < 5; ++q) r[q] = s_rec[q][col];
                    double ca[NC];
#pragma unroll
                    for (int q = 0; q < NC; ++q) ca[q] = 0.0;
                    const int32_t cg = M ? s_grp[col] : 0;
#pragma unroll
                    for (int k = 0; k < T; ++k) {
                        // two pairs in flight: more would spill
                        if (k != 0 && k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
                        dl_both_pair<M, SRC>(t.x[k], t.y[k], t.z[k], t.v[k], ra[k], r, M && excl && t.g[k] == cg, ca);
                    }
#pragma unroll
                    for (int q = 0; q < NC; ++q) lds_add(&s_col[wave][q][col], ca[q]);
                }
            };
            if (masked) steps(std::true_type{});
            else steps(std::false_type{});
        }
        __syncthreads();
        // wave 0: P; waves 1 .. 3: a component of Y each
        auto total = [&](int q) {
            return ((s_col[0][q][lane] + s_col[1][q][lane]) + s_col[2][q][lane]) + s_col[3][q][lane];
        };
        double* vp = vpart + tbk * NV * npad + sub * kSub + lane;
        if (wave == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) vp[q * npad] = total(q);
        } else if constexpr (SRC) {
            const int c = wave - 1;
            const double2 n01 = s_rec[3][lane], q12 = s_rec[2][lane];
            const double n = c == 0 ? n01.x : c == 1 ? n01.y : s_rec[4][lane].x;
            const double q = c == 0 ? s_rec[1][lane].y : c == 1 ? q12.x : q12.y;
            vp[(3 + c) * npad] = __builtin_fma(total(6), n, __builtin_fma(total(7), q, total(3 + c)));
        }
        if (++sub == C) {
            sub = 0;
            ++ub;
        }
    }
    ps::flush<P, T>(a, tbk, wave, lane, ra);
}

// dL/dx from the target side's segments (workgroup order): 4 times the bare sums.
template <int T>
__global__ __launch_bounds__(kBlock) void dl_both_targets(PassArgs a, int64_t blk0, int64_t grid) {
    constexpr int BT = kBlock * T;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;   // within the group
    if (blk0 * BT + i >= a.n_trg) return;
    const int64_t tbk = i / BT, li = i % BT, C = 4 * a.chunks, U = 4 * a.units;
    const int64_t b0 = ps::unit_owner(tbk * C, U, grid), b1 = ps::unit_owner((tbk + 1) * C - 1, U, grid);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int64_t b = b0; b <= b1; ++b) {
        const double* seg = a.part + (b + tbk) * 4 * BT;
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] += seg[q * BT + li];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] *= 0.25;
    DlT::store(a, blk0 * BT + i, s);
}

// dL/dphi_m and dL/dy_m from the target blocks' partials, in block order.
template <int NV>
__global__ __launch_bounds__(kBlock) void dl_both_sources(const double* __restrict__ vpart, int64_t blocks,
                                                          int64_t npad, const double* __restrict__ weight,
                                                          double pref, double* __restrict__ phi,
                                                          double* __restrict__ src, int64_t n, int acc_phi,
                                                          int acc_src) {
    const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (m >= n) return;
    double v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = 0.0;
#pragma unroll 2
    for (int64_t b = 0; b < blocks; ++b)
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] += vpart[(b * NV + q) * npad + m];
    const double sp = 0.125 * pref * weight[m], sy = -0.25 * pref;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (phi) phi[q * n + m] = acc_phi ? phi[q * n + m] + sp * v[q] : sp * v[q];
        if constexpr (NV == 6) src[q * n + m] = acc_src ? src[q * n + m] + sy * v[3 + q] : sy * v[3 + q];
    }
}

// Records of the sweep: DlT's with doubled positions.
struct DlBoth : DlT {
    __device__ static void make_rec(const PassArgs& a, int64_t i, Rec& r, double pos[3]) {
        DlT::make_rec(a, i, r, pos);
        r.x = pos[0] *= 2.0;
        r.y = pos[1] *= 2.0;
        r.z = pos[2] *= 2.0;
    }
};

// launch shapes (targets per lane, minimum waves per SIMD)
constexpr int kTSlT = 4, kWSlT = 3;
constexpr int kTSlS = 2, kWSlS = 4;
#ifndef STOKES_SYM_T
#define STOKES_SYM_T 3
#endif
#ifndef STOKES_SYM_W
#define STOKES_SYM_W 2
#endif
constexpr int kTSym = STOKES_SYM_T, kWSym = STOKES_SYM_W;
constexpr int kTDlT = 4, kWDlT = 3;
constexpr int kTDlS = 2, kWDlS = 3;
constexpr int kTSlSF = 4, kWSlSF = 4;
constexpr int kTDlSPhi = 4, kWDlSPhi = 3;

// The two-sided sweep's targets per lane: the most, as the sources' LDS reads and
// adds (about two thirds of a pair) are shared by them, unless the last target
// block's padding or idle workgroups cost more.  More than 6 spill.
int dl_both_T(int64_t n_src, int64_t n_trg, int resident) {
    const int64_t subs = ceil_div(n_src, (int64_t)kTile) * (kTile / kSub);
    int best = 6;
    double least = 1e300;
    for (int T : {6, 4, 2, 1}) {
        const int64_t units = subs * ceil_div(n_trg, (int64_t)kBlock * T);
        const double cost = (double)ceil_div(units, (int64_t)resident) * (T + 0.65);
        if (cost < least) {
            least = cost;
            best = T;
        }
    }
    return best;
}
template <typename F>
auto with_both_T(int T, F&& f) {
    return T == 6   ? f(std::integral_constant<int, 6>{})
           : T == 4 ? f(std::integral_constant<int, 4>{})
           : T == 2 ? f(std::integral_constant<int, 2>{})
                    : f(std::integral_constant<int, 1>{});
}

// The sources' partials are (target block, 3 or 6, padded source); target blocks
// are taken in groups whose partials fit this many bytes (one group up to 3.4e10
// pairs, at least one block).
constexpr int64_t kDlBothBytes = int64_t(1) << 30;

// targets of a group of target blocks
int64_t dl_both_group(int64_t n_src, int64_t n_trg, int T, int nv) {
    const int64_t per = nv * ceil_div(n_src, (int64_t)kTile) * kTile * (int64_t)sizeof(double);
    return std::min(n_trg, std::max<int64_t>(1, kDlBothBytes / per) * kBlock * T);
}

// workspace: the target-side pass of a group, then the sources' partials
ps::PassPlan dl_both_plan(int64_t n_src, int64_t n_trg, int T, int resident) {
    return with_both_T(T, [&](auto tc) {
        return ps::plan_pass<DlT, decltype(tc)::value>(n_src, n_trg, resident);
    });
}
size_t dl_both_bytes(int64_t n_src, int64_t n_trg, int resident, int nv) {
    const int T = dl_both_T(n_src, n_trg, resident);
    const auto p = dl_both_plan(n_src, dl_both_group(n_src, n_trg, T, nv), T, resident);
    return align_up(align_up(p.total, 256) + (size_t)p.blocks_x * nv * p.n_src_pad * sizeof(double), 256);
}

}  // namespace

void vjp_resident(int n_cu, int out[kVjpPasses]) {
    out[0] = ps::resident_blocks<SlT, kTSlT, kWSlT>(n_cu);
    out[1] = ps::resident_blocks<SlS, kTSlS, kWSlS>(n_cu);
    out[2] = ps::resident_blocks<SlSym, kTSym, kWSym>(n_cu);
    out[3] = ps::resident_blocks<DlT, kTDlT, kWDlT>(n_cu);
    out[4] = ps::resident_blocks<DlS, kTDlS, kWDlS>(n_cu);
    out[5] = ps::resident_blocks<SlSF, kTSlSF, kWSlSF>(n_cu);
    out[6] = ps::resident_blocks<DlSPhi, kTDlSPhi, kWDlSPhi>(n_cu);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, dl_both_main<6, true>, kBlock, 0) != hipSuccess || nb < 1)
        nb = 1;
    out[7] = nb * n_cu;
}

size_t vjp_workspace_bytes(int kernel, int64_t n_src, int64_t n_trg, const int resident[kVjpPasses]) {
    if (n_src <= 0 || n_trg <= 0) return 0;
    if (kernel == 0) {
        size_t b = ps::plan_pass<SlT, kTSlT>(n_src, n_trg, resident[0]).total;
        b = std::max(b, ps::plan_pass<SlS, kTSlS>(n_trg, n_src, resident[1]).total);
        b = std::max(b, ps::plan_pass<SlSF, kTSlSF>(n_trg, n_src, resident[5]).total);
        if (n_src == n_trg) b = std::max(b, ps::plan_pass<SlSym, kTSym>(n_src, n_trg, resident[2]).total);
        return b;
    }
    size_t b = ps::plan_pass<DlT, kTDlT>(n_src, n_trg, resident[3]).total;
    b = std::max(b, std::max(dl_both_bytes(n_src, n_trg, resident[7], 6), dl_both_bytes(n_src, n_trg, resident[7], 3)));
    b = std::max(b, ps::plan_pass<DlSPhi, kTDlSPhi>(n_trg, n_src, resident[6]).total);
    return std::max(b, ps::plan_pass<DlS, kTDlS>(n_trg, n_src, resident[4]).total);
}

static PassArgs base_args(const VjpInputs& in) {
    PassArgs a{};
    a.excl = in.excl;
    a.accumulate = in.accumulate;
    return a;
}

hipError_t launch_sl_vjp(const VjpInputs& in, const int resident[kVjpPasses], bool fused, void* ws,
                         hipStream_t stream) {
    hipError_t e = hipSuccess;
    const KernelTimer none{};
    if (fused) {
        PassArgs a = base_args(in);
        a.n_trg = a.n_src = in.n_trg;
        a.trg_xyz = a.src_xyz = in.trg_xyz;
        a.trg_group = a.src_group = in.trg_group;
        a.tv[0] = a.sv[2] = in.grad_vel;
        a.tv[1] = a.sv[0] = in.density;
        a.tv[2] = a.sv[1] = in.weight;
        a.out[0] = in.grad_density;
        a.out[1] = in.grad_trg;           // == grad_src: the total position gradient
        a.pref = in.pref;
        const auto p = ps::plan_pass<SlSym, kTSym>(in.n_src, in.n_trg, resident[2]);
        return ps::run_pass<SlSym, kTSym, kWSym>(a, p, ws, stream, none);
    }
    if (in.grad_trg) {
        PassArgs a = base_args(in);
        a.n_trg = in.n_trg;
        a.trg_xyz = in.trg_xyz;
        a.trg_group = in.trg_group;
        a.tv[0] = in.grad_vel;
        a.n_src = in.n_src;
        a.src_xyz = in.src_xyz;
        a.src_group = in.src_group;
        a.sv[0] = in.density;
        a.sv[1] = in.weight;
        a.out[0] = in.grad_trg;
        a.pref = in.pref;
        const auto p = ps::plan_pass<SlT, kTSlT>(in.n_src, in.n_trg, resident[0]);
        e = ps::run_pass<SlT, kTSlT, kWSlT>(a, p, ws, stream, none);
        if (e != hipSuccess) return e;
    }
    if (in.grad_density || in.grad_src) {
        PassArgs a = base_args(in);
        a.n_trg = in.n_src;
        a.trg_xyz = in.src_xyz;
        a.trg_group = in.src_group;
        a.tv[0] = in.density;
        a.tv[1] = in.weight;
        a.n_src = in.n_trg;
        a.src_xyz = in.trg_xyz;
        a.src_group = in.trg_group;
        a.sv[0] = in.grad_vel;
        a.out[0] = in.grad_density;
        a.out[1] = in.grad_src;
        a.pref = in.pref;
        if (in.grad_src) {
            const auto p = ps::plan_pass<SlS, kTSlS>(in.n_trg, in.n_src, resident[1]);
            e = ps::run_pass<SlS, kTSlS, kWSlS>(a, p, ws, stream, none);
        } else {
            const auto p = ps::plan_pass<SlSF, kTSlSF>(in.n_trg, in.n_src, resident[5]);
            e = ps::run_pass<SlSF, kTSlSF, kWSlSF>(a, p, ws, stream, none);
        }
    }
    return e;
}

// dL/dx and the source side's gradients in one sweep over the pairs.
static hipError_t launch_dl_both(const VjpInputs& in, int resident, bool combined, void* ws, hipStream_t stream) {
    PassArgs a = base_args(in);
    a.n_trg = in.n_trg;
    a.trg_xyz = in.trg_xyz;
    a.trg_group = in.trg_group;
    a.tv[0] = in.grad_vel;
    a.n_src = in.n_src;
    a.src_xyz = in.src_xyz;
    a.src_group = in.src_group;
    a.sv[0] = in.density;
    a.sv[1] = in.weight;
    a.sv[2] = in.normal;
    a.out[0] = in.grad_trg;
    a.pref = in.pref;
    const int nv = in.grad_src ? 6 : 3, T = dl_both_T(in.n_src, in.n_trg, resident);
    const int64_t group = dl_both_group(in.n_src, in.n_trg, T, nv);
    const auto p = dl_both_plan(in.n_src, group, T, resident);
    char* base = static_cast<char*>(ws);
    a.rec = base + p.off_rec;
    a.grp = reinterpret_cast<int32_t*>(base + p.off_grp);
    a.meta = reinterpret_cast<SubMeta*>(base + p.off_meta);
    a.part = reinterpret_cast<double*>(base + p.off_part);
    a.chunks = p.chunks;
    double* vpart = reinterpret_cast<double*>(base + align_up(p.total, 256));
    ps::prep<DlBoth><<<dim3((unsigned)(p.n_src_pad / kBlock)), dim3(kBlock), 0, stream>>>(a);
    hipError_t e = hipGetLastError();
    if (combined && group < in.n_trg) {
        // a later group's target side must not overwrite earlier groups' sources
        if (!in.accumulate && e == hipSuccess) e = launch_fill_zero(in.grad_trg, 3 * in.n_trg, stream);
        a.force_acc = in.grad_trg;
    }
    for (int64_t t0 = 0; t0 < in.n_trg && e == hipSuccess; t0 += group) {
        const int64_t nt = std::min(group, in.n_trg - t0);
        const auto pg = dl_both_plan(in.n_src, nt, T, resident);
        a.units = pg.units;
        const dim3 gm((unsigned)pg.grid), gt((unsigned)ceil_div(nt, kBlock)), gs((unsigned)ceil_div(in.n_src, kBlock));
        // the sweep writes every (target block, source) slot of the group
        with_both_T(T, [&](auto tc) {
            constexpr int K = decltype(tc)::value;
            const int64_t blk0 = t0 / ((int64_t)kBlock * K);
            if (in.grad_src)
                dl_both_main<K, true><<<gm, dim3(kBlock), 0, stream>>>(a, blk0, vpart);
            else
                dl_both_main<K, false><<<gm, dim3(kBlock), 0, stream>>>(a, blk0, vpart);
            dl_both_targets<K><<<gt, dim3(kBlock), 0, stream>>>(a, blk0, pg.grid);
        });
        // one array for both position gradients: the group's target side is in it
        // before its source side is added
        const int acc = in.accumulate || t0 > 0;
        if (in.grad_src)
            dl_both_sources<6><<<gs, dim3(kBlock), 0, stream>>>(vpart, pg.blocks_x, p.n_src_pad, in.weight, in.pref,
                                                                in.grad_density, in.grad_src, in.n_src, acc,
                                                                acc || combined);
        else
            dl_both_sources<3><<<gs, dim3(kBlock), 0, stream>>>(vpart, pg.blocks_x, p.n_src_pad, in.weight, in.pref,
                                                                in.grad_density, nullptr, in.n_src, acc, 0);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_dl_vjp(const VjpInputs& in, const int resident[kVjpPasses], bool combined,
                         void* ws, hipStream_t stream) {
    hipError_t e = hipSuccess;
    const KernelTimer none{};
    if (in.grad_trg && (in.grad_density || in.grad_src)) return launch_dl_both(in, resident[7], combined, ws, stream);
    if (in.grad_trg) {
        PassArgs a = base_args(in);
        a.n_trg = in.n_trg;
        a.trg_xyz = in.trg_xyz;
        a.trg_group = in.trg_group;
        a.tv[0] = in.grad_vel;
        a.n_src = in.n_src;
        a.src_xyz = in.src_xyz;
        a.src_group = in.src_group;
        a.sv[0] = in.density;
        a.sv[1] = in.weight;
        a.sv[2] = in.normal;
        a.out[0] = in.grad_trg;
        a.pref = in.pref;
        const auto p = ps::plan_pass<DlT, kTDlT>(in.n_src, in.n_trg, resident[3]);
        e = ps::run_pass<DlT, kTDlT, kWDlT>(a, p, ws, stream, none);
        if (e != hipSuccess) return e;
    }
    if (in.grad_density || in.grad_src) {
        PassArgs a = base_args(in);
        a.n_trg = in.n_src;
        a.trg_xyz = in.src_xyz;
        a.trg_group = in.src_group;
        a.tv[0] = in.density;
        a.tv[1] = in.weight;
        a.tv[2] = in.normal;
        a.n_src = in.n_trg;
        a.src_xyz = in.trg_xyz;
        a.src_group = in.trg_group;
        a.sv[0] = in.grad_vel;
        a.out[0] = in.grad_density;
        a.out[1] = in.grad_src;
        a.pref = in.pref;
        if (in.grad_src) {
            const auto p = ps::plan_pass<DlS, kTDlS>(in.n_trg, in.n_src, resident[4]);
            e = ps::run_pass<DlS, kTDlS, kWDlS>(a, p, ws, stream, none);
        } else {
            const auto p = ps::plan_pass<DlSPhi, kTDlSPhi>(in.n_trg, in.n_src, resident[6]);
            e = ps::run_pass<DlSPhi, kTDlSPhi, kWDlSPhi>(a, p, ws, stream, none);
        }
    }
    return e;
}

}  // namespace stokes
