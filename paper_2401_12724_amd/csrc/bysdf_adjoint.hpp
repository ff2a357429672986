// bysdf_adjoint.hpp -- derivatives of one query's loss L = sum_c g_c E_c with
// respect to the type's parameters.
//
// One sweep per query gives all of them.  E is linear in the sums over the
// forward nodes, so what a node's terms weigh in L is known before the first
// node: each node runs forward and at once backward, and nothing of it is
// kept.  The backward sweep carries the derivative of L with respect to the
// frame at x through the nodes and enters that frame's own sweep at the end.
// The ply hit is left in forward mode: everything in it follows one scalar,
// the ply twist, through the plies' phases (dphase), the distance to the hit
// and the turn of the hit's normal, so the sweep ends in products with those
// three tangents.  Compared with three forward-mode passes over the whole
// model, one per parameter, the model's values are formed once instead of
// three times and no zero tangents are carried: forward and backward of 4 Mi
// queries (64 types, 3 plies, 4 nodes) take 2.5 ms, 7.3 ms with the passes.
// The sweep needs 424 registers (up to 4 plies, isotropic, no migration), so
// one wavefront per SIMD runs; VALU issue bounds it (about 5000 instructions a
// query and two thirds of them FP64), and at two wavefronts the spills cost
// more than the second hides (4.7 ms).
//
// Branch decisions use the values only (the derivative of the
// piecewise-smooth model away from its decision boundaries).  Geometry and
// its derivatives run in double, the lobe formulas and theirs in float, like
// the model.  x_ names the derivative of L with respect to x.
#pragma once

#include "bysdf_model.hpp"

namespace bysdf {

// A value with one tangent: the ply visibility, whose ends come and go with
// the value, is differentiated forward along the ply twist.
struct Dual {
    double v, d;
    Dual() = default;
    __host__ __device__ Dual(double x) : v(x), d(0.0) {}
    __host__ __device__ Dual(double x, double dx) : v(x), d(dx) {}
};
__host__ __device__ inline double val(Dual x) { return x.v; }
__host__ __device__ inline Dual pick(bool c, Dual a, Dual b) { return Dual(c ? a.v : b.v, c ? a.d : b.d); }
__host__ __device__ inline Dual operator+(Dual a, Dual b) { return Dual(a.v + b.v, a.d + b.d); }
__host__ __device__ inline Dual operator-(Dual a, Dual b) { return Dual(a.v - b.v, a.d - b.d); }
__host__ __device__ inline Dual operator*(Dual a, Dual b) { return Dual(a.v * b.v, a.d * b.v + a.v * b.d); }
__host__ __device__ inline Dual operator-(Dual a) { return Dual(-a.v, -a.d); }
__host__ __device__ inline Dual operator+(double a, Dual b) { return Dual(a + b.v, b.d); }
__host__ __device__ inline Dual operator-(double a, Dual b) { return Dual(a - b.v, -b.d); }
__host__ __device__ inline Dual operator-(Dual a, double b) { return Dual(a.v - b, a.d); }
__host__ __device__ inline Dual operator*(Dual a, double b) { return Dual(a.v * b, a.d * b); }
__host__ __device__ inline Dual operator*(double a, Dual b) { return b * a; }
__host__ __device__ inline Dual operator/(Dual a, Dual b)
{
    const double r = rcp_(b.v), q = a.v * r;
    return Dual(q, (a.d - q * b.d) * r);
}
__host__ __device__ inline Dual sqrt_(Dual x)
{
    const double s = sqrt_(x.v);
    return Dual(s, s > 0.0 ? 0.5 * x.d * rcp_(s) : 0.0);
}
__host__ __device__ inline Dual rsqrt_(Dual x)
{
    const double r = rsqrt_(x.v);
    return Dual(r, -0.5 * r * r * r * x.d);
}
__host__ __device__ inline Dual atan2_(Dual y, Dual x)
{
    const double r2 = x.v * x.v + y.v * y.v;
    return Dual(atan2_(y.v, x.v), r2 > 0.0 ? (x.v * y.d - y.v * x.d) * rcp_(r2) : 0.0);
}

// What the sweep accumulates: derivatives of L with respect to the two
// roughnesses and the two twists.
struct ParamBar {
    double ax, ay, ply, fiber;
};

// Derivatives of a type's derived scalars with respect to the twist angles.
struct TwistRates {
    double wp_turns, kt, tnorm_inv, vply_scale;  // ply twist
    double tan_af, wf_turns;                     // fiber twist
};
__host__ __device__ inline TwistRates twist_rates(const TypeRec& t)
{
    const Derived<double, float>& P = t.d;
    TwistRates r;
    const double ds = P.Rpc > 0.0 ? 1.0 + P.slope * P.slope : 0.0;
    r.wp_turns = P.Rpc > 0.0 ? ds / P.Rpc * kInvTwoPi : 0.0;
    r.vply_scale = P.slope * ds * P.tnorm_inv;
    r.tnorm_inv = -r.vply_scale * P.tnorm_inv * P.tnorm_inv;
    r.kt = ds * P.tnorm_inv + P.slope * r.tnorm_inv;
    r.tan_af = 1.0 + P.tan_af * P.tan_af;
    r.wf_turns = r.tan_af / ((1.0 - t.rho_f_geom) * P.rp) * kInvTwoPi;
    return r;
}

// ---------------------------------------------------------------- microfacets

// dF/dc of fresnel
__host__ __device__ inline float fresnel_dc(float c, float e)
{
    const float ie2 = rcp_(e * e), s2t = (1.0f - c * c) * ie2;
    if (s2t >= 1.0f) return 0.0f;
    const float ct = sqrt_(1.0f - s2t), dct = c * ie2 * rcp_(ct);
    const float is = rcp_(c + e * ct), ip = rcp_(e * c + ct);
    const float n = 2.0f * e * (ct - c * dct);
    return (c - e * ct) * is * is * is * n + (e * c - ct) * ip * ip * ip * n;
}
// fresnel_T and its derivative
template <class T> __host__ __device__ inline T fresnel_T_dc(T c, T e, T ie2, T& dT)
{
    const T s2t = (T(1) - c * c) * ie2;
    if (val(s2t) >= 1.0f) {
        dT = T(0);
        return T(0);
    }
    const T ct = sqrt_(T(1) - s2t), dct = ct > T(0) ? c * ie2 * rcp_(ct) : T(0);
    const T ia = rcp_(c + e * ct), ib = rcp_(e * c + ct), ia2 = ia * ia, ib2 = ib * ib;
    const T w = ia2 + ib2, e2 = T(2) * e;
    dT = e2 * ((ct + c * dct) * w - T(2) * c * ct * (ia2 * ia * (T(1) + e * dct) + ib2 * ib * (e + dct)));
    return e2 * c * ct * w;
}
__host__ __device__ inline float ls_albedo_dmu(float mu)
{
    if (!(mu > 0.0f)) return 0.0f;
    return 0.5f * (rcp_(mu + 1.0f) - log_(1.0f + rcp_(mu)));
}

// GGX distribution and Smith masking with their derivatives, isotropic: in
// the cosine z (zs = 1 - z^2) and the roughness a.
__host__ __device__ inline float ggx_D_iso_d(float z, float zs, float a, float& dz, float& da)
{
    dz = da = 0.0f;
    if (!(z > 0.0f)) return 0.0f;
    const float ia2 = rcp_(a * a), t = zs * ia2 + z * z, it = rcp_(t);
    const float D = ia2 * float(1.0 / kPi) * it * it, f = 2.0f * D * it;
    dz = f * 2.0f * z * (ia2 - 1.0f);
    da = rcp_(a) * (f * 2.0f * zs * ia2 - 2.0f * D);
    return D;
}
__host__ __device__ inline float smith_G1_front_d(float z, float zs, float a, float& dz, float& da)
{
    const float iz = rcp_(z), k = a * a * iz * iz, q = k * zs, r = sqrt_(1.0f + q), g = 2.0f * rcp_(1.0f + r);
    const float f = 0.5f * g * g * rcp_(r);  // -2 dg/dq
    dz = f * k * iz;
    da = -f * q * rcp_(a);
    return g;
}
// Anisotropic: in the local coordinates and both roughnesses.
__host__ __device__ inline float ggx_D_d(const V3<float>& m, float ax, float ay, V3<float>& dm, float& dax, float& day)
{
    dm = mk3<float>(0.0f, 0.0f, 0.0f);
    dax = day = 0.0f;
    if (!(m.z > 0.0f)) return 0.0f;
    const float ix = rcp_(ax), iy = rcp_(ay), qx = m.x * ix, qy = m.y * iy;
    const float t = qx * qx + qy * qy + m.z * m.z, it = rcp_(t);
    const float D = float(1.0 / kPi) * ix * iy * it * it, f = 4.0f * D * it;
    dm = mk3<float>(-f * qx * ix, -f * qy * iy, -f * m.z);
    dax = ix * (f * qx * qx - D);
    day = iy * (f * qy * qy - D);
    return D;
}
__host__ __device__ inline float smith_G1_d(const V3<float>& w, float wm, float ax, float ay, V3<float>& dw,
                                            float& dax, float& day)
{
    dw = mk3<float>(0.0f, 0.0f, 0.0f);
    dax = day = 0.0f;
    if (!(wm * w.z > 0.0f)) return 0.0f;
    const float iz = rcp_(w.z), tx = ax * w.x * iz, ty = ay * w.y * iz, q = tx * tx + ty * ty;
    const float r = sqrt_(1.0f + q), g = 2.0f * rcp_(1.0f + r), f = -0.5f * g * g * rcp_(r);  // 2 dg/dq
    dw = mk3<float>(f * tx * ax * iz, f * ty * ay * iz, -f * q * iz);
    dax = f * tx * w.x * iz;
    day = f * ty * w.y * iz;
    return g;
}

__host__ __device__ inline void fma3(V3<double>& a, const V3<double>& b, double s)
{
    a.x += b.x * s;
    a.y += b.y * s;
    a.z += b.z * s;
}

// A factor of a lobe (the distribution at a microfacet, the masking of a
// direction) as a function of a world vector w and a frame: its value and
// what its derivative multiplies.
struct Facet {
    float f;         // the factor
    float dz;        // isotropic: with respect to w.n
    V3<float> dl;    // anisotropic: with respect to the local vector
    float dax, day;
};
// ISO is the type's alpha_x == alpha_y: only the cosine w.n = z enters.
template <bool ISO>
__host__ __device__ inline Facet facet_D(const Derived<double, float>& P, const Frame<double>& F, const V3<double>& m,
                                         double z)
{
    Facet r;
    if (ISO) {
        r.f = ggx_D_iso_d((float)z, (float)one_minus_sq(z), P.ax, r.dz, r.dax);
        r.day = 0.0f;
    } else {
        r.f = ggx_D_d(narrow3<float>(to_local(F, m)), P.ax, P.ay, r.dl, r.dax, r.day);
    }
    return r;
}
// wm = w.m: the masking is zero where it has not the sign of w.n
template <bool ISO>
__host__ __device__ inline Facet facet_G1(const Derived<double, float>& P, const Frame<double>& F, const V3<double>& w,
                                          double z, double wm)
{
    Facet r;
    r.day = 0.0f;
    if (ISO) {
        r.f = r.dz = r.dax = 0.0f;
        if (wm * z > 0.0) r.f = smith_G1_front_d((float)z, (float)one_minus_sq(z), P.ax, r.dz, r.dax);
    } else {
        r.f = smith_G1_d(narrow3<float>(to_local(F, w)), (float)wm, P.ax, P.ay, r.dl, r.dax, r.day);
    }
    return r;
}
// f_ to the frame, the roughnesses and (WB) the vector
template <bool ISO, bool WB>
__host__ __device__ inline void facet_back(const Facet& r, float f_, const Frame<double>& F, const V3<double>& w,
                                           Frame<double>& F_, V3<double>& w_, ParamBar& pb)
{
    pb.ax += (double)(f_ * r.dax);
    if (ISO) {
        const double z_ = (double)(f_ * r.dz);
        fma3(F_.n, w, z_);
        if (WB) fma3(w_, F.n, z_);
    } else {
        pb.ay += (double)(f_ * r.day);
        const double lx = (double)(f_ * r.dl.x), ly = (double)(f_ * r.dl.y), lz = (double)(f_ * r.dl.z);
        fma3(F_.t, w, lx);
        fma3(F_.b, w, ly);
        fma3(F_.n, w, lz);
        if (WB) {
            fma3(w_, F.t, lx);
            fma3(w_, F.b, ly);
            fma3(w_, F.n, lz);
        }
    }
}

// ---------------------------------------------------------------- fiber frame

// Reverse of fiber_frame.  TB: the tangent and bitangent carry derivatives
// too (at an exit with an isotropic roughness only the normal does).  Adds
// to the turn of the ply's phase (theta_, radians), of the 2D normal
// (omega_) and to the height (z_).
template <bool TB, class Tab>
__host__ __device__ inline void frame_back(const Derived<double, float>& P, const TwistRates& dr,
                                           const FrameTape<double>& T, const Frame<double>& F, double z, double cth,
                                           double sth, double n2x, double n2y, Frame<double>& F_, double gf_,
                                           double& theta_, double& omega_, double& z_, ParamBar& pb)
{
    V3<double> n_ = F_.n, tp_, bp_;
    const double A1 = T.q * T.sa * T.cs, A2 = T.q * T.cdn, A3 = T.q * T.ca * T.cs;
    double ca_ = 0.0, sa_ = 0.0;
    if (TB) {
        // b = n x t; t = tp ca - bp sa
        n_ = n_ + cross(F.t, F_.b);
        const V3<double> t_ = F_.t + cross(F_.b, F.n);
        tp_ = t_ * T.ca + n_ * A1;
        bp_ = n_ * A3 - t_ * T.sa;
        ca_ = dot(t_, T.tp);
        sa_ = -dot(t_, T.bp);
    } else {
        tp_ = n_ * A1;
        bp_ = n_ * A3;
    }
    const V3<double> np_ = n_ * A2;
    // n = q (tp sa cs + np cdn + bp ca cs), q = (cdn^2 + cs^2)^(-1/2)
    const double a1 = dot(n_, T.tp), a2 = dot(n_, T.np), a3 = dot(n_, T.bp);
    const double e = T.sa * a1 + T.ca * a3;
    const double q_ = e * T.cs + a2 * T.cdn, q3 = q_ * T.q * T.q * T.q;
    sa_ += a1 * T.q * T.cs;
    ca_ += a3 * T.q * T.cs;
    const double cs_ = T.q * e - q3 * T.cs, cdn_ = a2 * T.q - q3 * T.cdn;
    ca_ += cs_ * T.sdn;
    // sa = tfa ca, ca = (1 + tfa^2)^(-1/2), tfa = rh tan_af
    ca_ += sa_ * T.tfa;
    const double tfa_ = sa_ * T.ca - ca_ * T.ca * T.ca * T.sa;
    const double rh_ = tfa_ * P.tan_af;
    const double dn_ = cs_ * T.ca * T.cdn - cdn_ * T.sdn;
    const double turns_ = dn_ * T.rate[0] + rh_ * T.rate[1] + gf_ * T.rate[2];
    double vply_ = turns_ * P.wf_turns;
    if (Tab::kMigration && P.n_mig > 1) vply_ += dn_ * T.fade[0] + rh_ * T.fade[1] + gf_ * T.fade[2];
    pb.fiber += tfa_ * T.rh * dr.tan_af + turns_ * T.vply * dr.wf_turns;
    z_ += vply_ * P.vply_scale;
    // ply frame
    const double rtz = T.rn * P.tnorm_inv, rk = T.rn * T.kt, rks = T.rn * T.ks;
    const double rtz_ = bp_.y * n2x - bp_.x * n2y;
    const double rks_ = -dot(np_, T.tp);
    const double rn_ = np_.x * n2x + np_.y * n2y + rtz_ * P.tnorm_inv - bp_.z * T.kt * T.cos_a + rks_ * T.ks;
    const double ks_ = rks_ * T.rn + rn_ * T.rn * T.rn * T.rn * T.ks;
    const double tpx = tp_.x - np_.x * rks, tpy = tp_.y - np_.y * rks, tpz = tp_.z - np_.z * rks;
    const double kt_ = tpy * cth - tpx * sth - bp_.z * T.rn * T.cos_a + ks_ * T.sin_a;
    pb.ply += kt_ * dr.kt + (rtz_ * T.rn + tpz) * dr.tnorm_inv + vply_ * z * dr.vply_scale;
    // the angle from the phase to the normal: d a = omega - theta
    const double a_ = turns_ * kInvTwoPi + ks_ * T.kt * T.cos_a + bp_.z * rk * T.sin_a;
    theta_ += -T.kt * (tpx * cth + tpy * sth) - a_;
    // np and bp turn with the normal
    omega_ += T.rn * (np_.y * n2x - np_.x * n2y) - rtz * (bp_.x * n2x + bp_.y * n2y) + a_;
}

// ---------------------------------------------------------------- ply hit

// Tangents of the ply hit along the ply twist: the distance along the ray in
// the cross-section, the turn of the normal, the turns of the plies' phases.
template <int MP> struct HitTangent {
    double s, omega;
    double phase[MP];
};
template <int MP>
__host__ __device__ inline void hit_tangent(const Derived<double, float>& P, const PlyHit<double, MP>& ph,
                                            HitTangent<MP>& t)
{
    double c = 0.0, s = 0.0, dth = 0.0;
#pragma unroll
    for (int k = 0; k < MP; ++k)
        if (k == ph.ks) {
            c = ph.cth[k];
            s = ph.sth[k];
            dth = t.phase[k];
        }
    // s_hit = -b - sqrt(disc) where that is positive
    const double wx = ph.x2x - P.Rpc * c, wy = ph.x2y - P.Rpc * s;
    const double dwx = P.Rpc * s * dth, dwy = -P.Rpc * c * dth;
    const double b = wx * ph.dhx + wy * ph.dhy, db = dwx * ph.dhx + dwy * ph.dhy;
    const double disc = b * b - (wx * wx + wy * wy - P.rp * P.rp);
    const double sq = disc > 0.0 ? sqrt_(disc) : 0.0;
    const double dsq = sq > 0.0 ? (b * db - (wx * dwx + wy * dwy)) * rcp_(sq) : 0.0;
    t.s = -b - sq > 0.0 ? -db - dsq : 0.0;
    const double nx = ph.p2x - P.Rpc * c, ny = ph.p2y - P.Rpc * s;
    const double dnx = t.s * ph.dhx + dwx, dny = t.s * ph.dhy + dwy;
    t.omega = (nx * dny - ny * dnx) * rcp_(nx * nx + ny * ny);
}

// ---------------------------------------------------------------- one query

struct AdjointOut {
    float body0, Gp, Gf;   // as in EvalOut and XState
    float rawp, rawf;
    double beta, ply, fiber;
};

// Node k forward and backward: its share of the node sums (bodies at the
// exit in by) and the derivatives of L.  w_spec and w_body are what the
// node's specular and body terms weigh in L.
template <bool ISO, int MP, class Tab>
__host__ __device__ inline void node_adjoint(const Derived<double, float>& P, const TwistRates& dr, const Tab& tab,
                                             const XState<double, float, MP>& X, const HitTangent<MP>& ht,
                                             const V3<double>& wo, int k, float s0, float s1, bool has_shift,
                                             const double* disk, float w_spec, float w_body, float& by,
                                             Frame<double>& fx_, double& hit_s_, double& hit_omega_, ParamBar& pb)
{
    const PlyHit<double, MP>& ph = X.ph;
    const bool front = X.mu_i > 0.0f;
    if (!front) {
        // thin-sheet exit: the frame at x flipped
        const double co = -dot(wo, X.fx.n);
        if (co > 0.0) {
            by += (float)co * float(1.0 / kPi);
            fma3(fx_.n, wo, -(double)(w_body * float(1.0 / kPi)));
        }
        return;
    }
    // ---- forward: visible normal and refraction at x (forward_node)
    const V3<double> wl = to_local(X.fx, X.wi_g);
    double d1, d2, r1;
    if (!has_shift) {
        d1 = disk[3 * k];
        d2 = disk[3 * k + 1];
        r1 = disk[3 * k + 2];
    } else {
        double xi1, xi2;
        node_lattice(k, P.K, s0, s1, true, xi1, xi2);
        vndf_disk<double>(xi1, xi2, d1, d2);
        r1 = sqrt_(1.0 - d1 * d1);
    }
    // stretched view p = |p| (l ux, l uy, vz)
    const double px = P.ax_g * wl.x, py = P.ay_g * wl.y, l2p = px * px + py * py;
    const double ip = rsqrt_(l2p + wl.z * wl.z);
    const double ilp = l2p > 0.0 ? rsqrt_(l2p) : 0.0;
    const double ux = l2p > 0.0 ? px * ilp : 0.0, uy = l2p > 0.0 ? py * ilp : -1.0;
    const double l = l2p * ilp * ip, vz = wl.z * ip;
    const double blend = 0.5 * (1.0 + vz), dd = (1.0 - blend) * r1 + blend * d2;
    const double h2 = 1.0 - d1 * d1 - dd * dd;
    const double hz = h2 > 0.0 ? sqrt_(h2) : 0.0;
    const double lw = l * hz - vz * dd;
    const double nhx = ux * lw - uy * d1, nhy = uy * lw + ux * d1, nhz0 = l * dd + vz * hz;
    const double nhz = nhz0 > 0.0 ? nhz0 : 0.0;
    V3<double> ml = mk3<double>(P.ax_g * nhx, P.ay_g * nhy, nhz);
    const double i2 = rsqrt_(dot(ml, ml));
    ml = ml * i2;
    const V3<double> m = to_world(X.fx, ml);
    const double c0 = dot(X.wi_g, m), c = c0 > 0.0 ? c0 : 0.0;
    const double ie = P.inv_eta_g, ct = sqrt_(1.0 - (1.0 - c * c) * ie * ie), kap = c * ie - ct;
    const V3<double> wt = X.wi_g * (-ie) + m * kap;
    const double tz = dot(wt, X.fx.n);
    const Facet gt = facet_G1<ISO>(P, X.fx, wt, tz, dot(wt, m));
    float dTf;
    const float Tf = fresnel_T_dc<float>((float)c, P.eta, P.inv_eta2, dTf);
    // ---- forward: chord
    const double le2 = wt.x * wt.x + wt.y * wt.y;
    const double il = le2 > 0.0 ? rsqrt_(le2) : 0.0;
    const double le = le2 * il, en = wt.x * ph.n2x + wt.y * ph.n2y;
    const bool chord = !(le < 1e-6 || en >= 0.0);
    Frame<double> fy;
    FrameTape<double> tape;
    double ex = 0.0, ey = 0.0, bq = 0.0, yq = 0.0, sbest = 0.0, cthl = 0.0, sthl = 0.0, dthl = 0.0, ell = 0.0;
    double zy = 0.0, n2x = 0.0, n2y = 0.0, ninv = 0.0;
    int kind = 0;  // what ends the chord: 0 the yarn, 1 the hit ply, 2 another ply
    float att = 1.0f, sN = 0.0f;
    if (chord) {
        ex = wt.x * il;
        ey = wt.y * il;
        bq = ph.p2x * ex + ph.p2y * ey;
        const double dq = bq * bq - (ph.p2x * ph.p2x + ph.p2y * ph.p2y - 1.0);
        yq = dq > 0.0 ? sqrt_(dq) : 0.0;
        const double syarn = -bq + yq;
        int N = 0, jl = -1;
#pragma unroll
        for (int j = 0; j < MP; ++j) {
            if (j >= P.Np) break;
            bool ent = false;
            double so = 0.0;
            int kd = 0;
            if (j == ph.ks) {
                const double sx = -2.0 * P.rp * en * il;
                kd = sx < syarn ? 1 : 0;
                so = sx < syarn ? sx : syarn;
                ent = true;
            } else {
                const double wx = ph.p2x - P.Rpc * ph.cth[j], wy = ph.p2y - P.Rpc * ph.sth[j];
                const double b = wx * ex + wy * ey;
                const double disc = b * b - (wx * wx + wy * wy - P.rp * P.rp);
                if (disc > 0.0) {
                    const double sq = sqrt_(disc), slo = -b - sq, shi = -b + sq;
                    if (shi > 0.0 && slo < syarn) {
                        ent = true;
                        kd = shi < syarn ? 2 : 0;
                        so = shi < syarn ? shi : syarn;
                    }
                }
            }
            if (ent) {
                ++N;
                if (jl < 0 || so > sbest) {
                    jl = j;
                    sbest = so;
                    kind = kd;
                    cthl = ph.cth[j];
                    sthl = ph.sth[j];
                    dthl = ht.phase[j];
                }
            }
        }
        const double y2x = ph.p2x + sbest * ex, y2y = ph.p2y + sbest * ey;
        ell = sbest * il;
        zy = ph.vhit + wt.z * ell;
        const double nyx = y2x - P.Rpc * cthl, nyy = y2y - P.Rpc * sthl;
        ninv = rsqrt_(nyx * nyx + nyy * nyy);
        n2x = nyx * ninv;
        n2y = nyy * ninv;
        sN = P.sigma_t * (float)N;
        att = exp_(-P.sigma_t * (float)ell * (float)N);
        fy = fiber_frame<double, float, Tab>(P, tab, cthl, sthl, jl, n2x, n2y, zy, nullptr, nullptr, nullptr, &tape);
    } else {
        fy.t = X.fx.t;
        fy.n = -X.fx.n;
        fy.b = cross(fy.n, fy.t);
    }
    // ---- exit terms and their derivatives
    Frame<double> fy_;
    fy_.t = fy_.b = fy_.n = mk3<double>(0.0, 0.0, 0.0);
    V3<double> wt_ = mk3<double>(0.0, 0.0, 0.0);
    float T_ = 0.0f;
    double ell_ = 0.0;
    const double co = dot(wo, fy.n);
    if (co > 0.0) {
        by += (float)co * float(1.0 / kPi);
        fma3(fy_.n, wo, (double)(w_body * float(1.0 / kPi)));
    }
    const double ti = dot(wt, fy.n);
    V3<double> mh = wt * P.eta_g - wo;
    const double ml2 = dot(mh, mh);
    if (ti > 0.0 && co > 0.0 && ml2 > 0.0) {
        double ih = rsqrt_(ml2);
        mh = mh * ih;
        double mz = dot(mh, fy.n);
        if (mz < 0.0) {
            mh = -mh;
            mz = -mz;
            ih = -ih;
        }
        const double im = -dot(wt, mh), om = dot(wo, mh);  // wi'.m, wo.m with wi' = -wt
        if (im < 0.0 && om > 0.0) {
            const Facet D = facet_D<ISO>(P, fy, mh, mz);
            const Facet gi = facet_G1<ISO>(P, fy, wt, ti, -im);  // even in the direction
            const Facet go = facet_G1<ISO>(P, fy, wo, co, om);
            const double iden = rcp_(P.eta_g * im + om), iti = rcp_(ti);
            const double geo_g = -(im * om) * iden * iden * iti;
            double dFt;
            const double Ft_g = fresnel_T_dc<double>(-im, P.inv_eta_g, P.eta_g * P.eta_g, dFt);
            const float geo = (float)geo_g, Ft = (float)Ft_g;
            const float gg = gi.f * go.f, T = Tf * gt.f;
            const float vv = geo * Ft * gg * D.f;
            const float v_ = w_spec * T * att;
            T_ = w_spec * att * vv;
            ell_ = -(double)(v_ * vv * sN);
            V3<double> mh_ = mk3<double>(0.0, 0.0, 0.0), unused;
            facet_back<ISO, true>(D, v_ * geo * Ft * gg, fy, mh, fy_, mh_, pb);
            const float gv = v_ * geo * Ft * D.f;
            facet_back<ISO, true>(gi, gv * go.f, fy, wt, fy_, wt_, pb);
            facet_back<ISO, false>(go, gv * gi.f, fy, wo, fy_, unused, pb);
            const double geo_ = (double)(v_ * Ft * gg * D.f), lg = geo_ * geo_g;
            // d ln geo = d im / im + d om / om - 2 (eta d im + d om) iden - d ti / ti
            const double vg = (double)(v_ * geo * gg * D.f);
            const double iio = rcp_(im * om);
            const double im_ = lg * (om * iio - 2.0 * P.eta_g * iden) - vg * dFt;
            const double om_ = lg * (im * iio - 2.0 * iden);
            const double ti_ = -lg * iti;
            fma3(fy_.n, wt, ti_);
            fma3(wt_, fy.n, ti_);
            fma3(wt_, mh, -im_);
            fma3(mh_, wt, -im_);
            fma3(mh_, wo, om_);
            // mh = (eta wt - wo) / |..|
            const double s = ih * P.eta_g;
            fma3(wt_, mh_, s);
            fma3(wt_, mh, -s * dot(mh, mh_));
        }
    }
    // ---- exit frame and chord
    if (chord) {
        double theta_ = 0.0, omega_ = 0.0, z_ = 0.0;
        frame_back<!ISO, Tab>(P, dr, tape, fy, zy, cthl, sthl, n2x, n2y, fy_, 0.0, theta_, omega_, z_, pb);
        // the 2D normal is that of y2 - R_pc (c, s)
        const double nx_ = -omega_ * n2y * ninv, ny_ = omega_ * n2x * ninv;
        theta_ += P.Rpc * (nx_ * sthl - ny_ * cthl);
        double p2x_ = nx_, p2y_ = ny_;
        hit_s_ += z_ * ph.kappa;
        wt_.z += z_ * ell;
        ell_ += z_ * wt.z;
        double s_ = ell_ * il + nx_ * ex + ny_ * ey, il_ = ell_ * sbest;
        double ex_ = nx_ * sbest, ey_ = ny_ * sbest;
        if (kind == 1) {
            const double f = -2.0 * P.rp * s_, en_ = f * il;
            il_ += f * en;
            wt_.x += en_ * ph.n2x;
            wt_.y += en_ * ph.n2y;
            hit_omega_ += en_ * (wt.y * ph.n2x - wt.x * ph.n2y);
        } else {
            // -b + sqrt(b^2 - |w|^2 + r^2), b = w.e: the yarn's circle about
            // the axis or a ply's disc
            const bool ply = kind == 2;
            const double wx = ply ? ph.p2x - P.Rpc * cthl : ph.p2x, wy = ply ? ph.p2y - P.Rpc * sthl : ph.p2y;
            const double b = wx * ex + wy * ey;
            const double sq = ply ? sbest + b : yq;
            const double isq = sq > 0.0 ? s_ * rcp_(sq) : 0.0;
            const double b_ = b * isq - s_;
            const double wx_ = ex * b_ - wx * isq, wy_ = ey * b_ - wy * isq;
            ex_ += wx * b_;
            ey_ += wy * b_;
            p2x_ += wx_;
            p2y_ += wy_;
            if (ply) theta_ += P.Rpc * (wx_ * sthl - wy_ * cthl);
        }
        il_ += ex_ * wt.x + ey_ * wt.y;
        const double g = -il_ * il * il * il;
        wt_.x += ex_ * il + wt.x * g;
        wt_.y += ey_ * il + wt.y * g;
        hit_s_ += p2x_ * ph.dhx + p2y_ * ph.dhy;
        pb.ply += theta_ * dthl;
    } else {
        fx_.n = fx_.n - fy_.n;
        if (!ISO) {
            fx_.t = fx_.t + fy_.t;
            fx_.b = fx_.b - fy_.b;
        }
    }
    // ---- refraction and visible normal at x
    facet_back<ISO, true>(gt, T_ * Tf, X.fx, wt, fx_, wt_, pb);
    V3<double> m_ = wt_ * kap;
    const double kap_ = dot(wt_, m);
    double c_ = kap_ * (ie - c * ie * ie * rcp_(ct)) + (double)(T_ * gt.f * dTf);
    if (c0 > 0.0) fma3(m_, X.wi_g, c_);
    fma3(fx_.t, m_, ml.x);
    fma3(fx_.b, m_, ml.y);
    fma3(fx_.n, m_, ml.z);
    V3<double> ml_ = to_local(X.fx, m_);
    const double mm = dot(ml, ml_);
    ml_ = (ml_ - ml * mm) * i2;
    pb.ax += nhx * ml_.x;
    pb.ay += nhy * ml_.y;
    const double nx_ = P.ax_g * ml_.x, ny_ = P.ay_g * ml_.y, nz_ = nhz0 > 0.0 ? ml_.z : 0.0;
    const double lw_ = ux * nx_ + uy * ny_;
    const double hz_ = lw_ * l + nz_ * vz;
    double dd_ = nz_ * l - lw_ * vz;
    if (hz > 0.0) dd_ -= hz_ * dd * rcp_(hz);
    const double l_ = lw_ * hz + nz_ * dd;
    const double vz_ = nz_ * hz - lw_ * dd + 0.5 * dd_ * (d2 - r1);
    // turn of (ux, uy) and of (l, vz)
    const double psi_ = (lw * (ux * ny_ - uy * nx_) - d1 * lw_) * ilp;
    const double chi_ = ip * (vz * l_ - l * vz_);
    const double px_ = ux * vz * chi_ - uy * psi_, py_ = uy * vz * chi_ + ux * psi_;
    pb.ax += wl.x * px_;
    pb.ay += wl.y * py_;
    fma3(fx_.t, X.wi_g, P.ax_g * px_);
    fma3(fx_.b, X.wi_g, P.ay_g * py_);
    fma3(fx_.n, X.wi_g, -l * chi_);
}

// The lobes at x: E_xS and the body lobe's shape (body, per unit albedo
// without G_p G_f) with what they weigh in L.
template <bool ISO, int MP>
__host__ __device__ inline void at_x_adjoint(const Derived<double, float>& P, const XState<double, float, MP>& X,
                                             const V3<double>& wo, float w_spec, float w_body, float& body,
                                             Frame<double>& fx_, ParamBar& pb)
{
    const double mu_o_g = dot(wo, X.fx.n);
    body = 0.0f;
    if (!(mu_o_g > 0.0)) return;
    const float mu_i = X.mu_i, mu_o = (float)mu_o_g;
    const bool front = mu_i > 0.0f;
    float mu_i_ = 0.0f, mu_o_;
    if (front) {
        const V3<double> hv = normalize(X.wi_g + wo);
        const double ih = dot(X.wi_g, hv), oh = dot(wo, hv);
        const Facet D = facet_D<ISO>(P, X.fx, hv, dot(hv, X.fx.n));
        const Facet gi = facet_G1<ISO>(P, X.fx, X.wi_g, dot(X.wi_g, X.fx.n), ih);
        const Facet go = facet_G1<ISO>(P, X.fx, wo, mu_o_g, oh);
        const float f = (1.0f - P.B) * P.kS * fresnel<float>(ih > 0.0 ? (float)ih : 0.0f, P.eta) * w_spec;
        const float fq = f * X.q4;
        V3<double> unused;
        facet_back<ISO, false>(D, fq * gi.f * go.f, X.fx, hv, fx_, unused, pb);
        facet_back<ISO, false>(gi, fq * go.f * D.f, X.fx, X.wi_g, fx_, unused, pb);
        facet_back<ISO, false>(go, fq * gi.f * D.f, X.fx, wo, fx_, unused, pb);
        mu_i_ = -fq * gi.f * go.f * D.f * rcp_(mu_i);  // q4 = 1 / (4 mu_i)
    }
    const float mp = front ? mu_i : 0.0f;
    const float im = rcp_(mp + mu_o), fls = float(1.0 / (4.0 * kPi)) * im, sh = fls + float(1.0 / kPi);
    const float bf = P.B * P.r * X.ils;
    body = bf * sh * mu_o;
    const float fls_ = -w_body * bf * mu_o * fls * im;  // through mp + mu_o
    mu_o_ = w_body * bf * sh + fls_;
    if (front) {
        // body factor B r / (1 + a(mu_i))
        mu_i_ += fls_ - w_body * body * rcp_(1.0f + ls_albedo(mu_i)) * ls_albedo_dmu(mu_i);
        fma3(fx_.n, X.wi_g, (double)mu_i_);
    }
    fma3(fx_.n, wo, (double)mu_o_);
}

// One query: o is filled and true returned unless the hit is a pass-through.
// spec = sum_c g_c, alb = sum_c g_c albedo_c.
template <bool ISO, int MP, class Tab>
__host__ __device__ inline bool adjoint_query(const TypeRec& rec, const Tab& tab, float h, float u, float v,
                                              const V3<float>& wi, const V3<double>& wo, float s0, float s1,
                                              bool has_shift, float spec, float alb, AdjointOut& o)
{
    const Derived<double, float>& P = rec.d;
    const TwistRates dr = twist_rates(rec);
    XState<double, float, MP> X;
    HitTangent<MP> ht;
    trace_plies(P, h, u, v, wi, X.ph, ht.phase, dr.wp_turns);
    if (X.ph.pass) return false;
    hit_tangent(P, X.ph, ht);
    double cth = 0.0, sth = 0.0, dth = 0.0;
#pragma unroll
    for (int k = 0; k < MP; ++k)
        if (k == X.ph.ks) {
            cth = X.ph.cth[k];
            sth = X.ph.sth[k];
            dth = ht.phase[k];
        }
    X.wi_g = mk3<double>(wi.x, wi.y, wi.z);
    FrameTape<double> tape;
    X.fx = fiber_frame(P, tab, cth, sth, X.ph.ks, X.ph.n2x, X.ph.n2y, X.ph.vhit, &X.rawf, &X.ca, &X.sa, &tape);
    Dual raw;
    {
        const double fx = X.ph.n2x * X.wi_g.x + X.ph.n2y * X.wi_g.y, fy = X.ph.n2x * X.wi_g.y - X.ph.n2y * X.wi_g.x;
        const double da = ht.omega - dth;
        raw = ply_visibility<Dual, double, MP>(P, P.rp, P.Rpc, (double)P.dP, Dual(X.ca, -X.sa * da),
                                               Dual(X.sa, X.ca * da), Dual(fx, fy * ht.omega),
                                               Dual(fy, -fx * ht.omega));
    }
    X.Gp = (float)(1.0 - (double)P.rho_p * (1.0 - raw.v));
    X.Gf = (float)(1.0 - (double)P.rho_f * (1.0 - X.rawf));
    lobe_weights(P, X);
    const float w_body = alb * X.Gp * X.Gf, invK = rcp_(float(P.K));
    const float w_y = spec * (1.0f - P.B) * P.kS * invK, f_yb = P.B * (1.0f - P.r) * invK;
    Frame<double> fx_;
    fx_.t = fx_.b = fx_.n = mk3<double>(0.0, 0.0, 0.0);
    ParamBar pb{0.0, 0.0, 0.0, 0.0};
    double hit_s_ = 0.0, hit_omega_ = 0.0;
    float body, by = 0.0f;
    at_x_adjoint<ISO, MP>(P, X, wo, spec, w_body, body, fx_, pb);
    for (int k = 0; k < P.K; ++k)
        node_adjoint<ISO, MP, Tab>(P, dr, tab, X, ht, wo, k, s0, s1, has_shift, rec.node_disk, w_y, w_body * f_yb, by,
                                   fx_, hit_s_, hit_omega_, pb);
    o.body0 = body + by * f_yb;
    o.Gp = X.Gp;
    o.Gf = X.Gf;
    o.rawp = (float)raw.v;
    o.rawf = (float)X.rawf;
    const float ab = alb * o.body0;
    double theta_ = 0.0, z_ = 0.0;
    frame_back<true, Tab>(P, dr, tape, X.fx, X.ph.vhit, cth, sth, X.ph.n2x, X.ph.n2y, fx_,
                          (double)(ab * X.Gp * P.rho_f), theta_, hit_omega_, z_, pb);
    hit_s_ += z_ * X.ph.kappa;
    o.beta = pb.ax + rec.aniso * pb.ay;
    o.fiber = pb.fiber;
    o.ply = pb.ply + theta_ * dth + hit_s_ * ht.s + hit_omega_ * ht.omega +
            (double)(ab * X.Gf * P.rho_p) * raw.d;
    return true;
}

}  // namespace bysdf
