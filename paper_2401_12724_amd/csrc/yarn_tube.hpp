// yarn_tube.hpp -- device side of ray / yarn-tube intersection.
//
// A yarn is a uniform cubic B-spline centreline (the explicit yarn curves
// of Sec. 3.3) with radius R; its tube is the union of the balls of radius
// R centred on the curve.  Entering through the ball at C(s) happens at
// ray parameter T(s) = z(s) - sqrt(R^2 - r^2(s)), with z the distance of
// C(s) along the ray and r its distance from the ray, so the entry into a
// span is the minimum of T over s (an interior minimum is where the ray
// meets the tube surface, the closest-point condition).  Per span: T is
// sampled at a few points, the best sample is bracketed and polished by
// safeguarded Newton on dT/ds in double precision.
//
// The BVH is built binary (binned SAH) and collapsed to four children per
// node, so a ray fetches half as many nodes one after another as in the
// binary tree; each ray is traced by the four lanes of a quad, one child or
// span per lane.  Hit children are visited near first, and the per-ray stack
// lives in LDS.  The closest-hit traversal runs nodes and span scans in
// separate loops, with postponed leaves, so the span scans of a wavefront
// run together; the point query for tubes holding the origin stops each
// span's distance test as soon as a sample decides it.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "../../include/bysdf.h"
#include "bysdf_math.hpp"

namespace yarn {

constexpr int kStack = 64;        // binary BVH depth bound enforced by the builder
constexpr int kWideDepthMax = 40; // depth bound of the 4-wide tree (LDS stack: 123 entries)
// Entries of a ray's traversal stack for a 4-wide BVH whose deepest node
// sits at the given depth (root 0): a visit pushes at most three siblings,
// and a path holds depth + 1 nodes, so 3 (depth + 1) entries never
// overflow.  The traversal kernels size their LDS stacks with this at launch.
inline int stack_entries(int depth) { return 3 * (depth + 1); }
constexpr int kWaveRays = 16;     // rays a wavefront traces side by side
// LDS bytes of the stacks of a traversal workgroup of `block` lanes
inline size_t stack_bytes(int entries, int block) { return sizeof(int) * entries * kWaveRays * (block / 64); }
constexpr int kMaxExcluded = 4;   // yarns holding the ray origin
constexpr double kExcludeFrac = 1e-3;

// hit flags
constexpr uint32_t HIT_MISS = 1u << 0;
constexpr uint32_t HIT_CAP = 1u << 1;
constexpr uint32_t HIT_EXCLUDED = 1u << 2;
constexpr uint32_t HIT_BAD_INPUT = 1u << 9;

// binary node of the build: child boxes lo0 hi0 lo1 hi1 packed, child codes
// (>= 0 node, < 0 leaf: -(first*4 + count-1) - 1)
struct BNode {
    float4 a, b, c;
    int4 d;
};
// node of the traversed 4-wide tree: one 32-byte record per child, read by
// one lane each (two 16-byte loads; a quad reads the node's 128-byte line).
// lo_code.w holds the child's code as above (node codes index the wide
// nodes), hi_yarn.w the yarn of a leaf whose spans are all of one yarn (-1
// otherwise: consecutive spans of a yarn share a leaf, and a ray that leaves
// a yarn passes its leaves by without scanning them); an unused slot has an
// empty box (lo and hi +inf)
struct WChild {
    float4 lo_code, hi_yarn;
};
struct WNode {
    WChild child[4];
};

// span record (leaf order): first control point, yarn, index in the
// yarn, samples | first-span bit 16 | last-span bit 17
struct SpanRec {
    int cp0, yarn, seg, info;
};

struct SceneView {
    const float4* cp;       // x y z R per control point
    const SpanRec* span;    // leaf order
    const float4* frame;    // per span (leaf order): RMF normal at s = 0, arc length at s = 0
    const WNode* node;
    // per node, then per span: where it or its leaf hangs, 4 node + slot (a
    // node's index is above its parent's)
    const int* up;
    const float* yarn_phase;
    const int* yarn_type;
    int n_nodes;
    int stack;  // entries of a ray's traversal stack
};

struct D3 {
    double x, y, z;
};
__host__ __device__ inline D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__host__ __device__ inline D3 operator+(D3 a, D3 b) { return d3(a.x + b.x, a.y + b.y, a.z + b.z); }
__host__ __device__ inline D3 operator-(D3 a, D3 b) { return d3(a.x - b.x, a.y - b.y, a.z - b.z); }
__host__ __device__ inline D3 operator*(D3 a, double s) { return d3(a.x * s, a.y * s, a.z * s); }
__host__ __device__ inline double dot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__host__ __device__ inline D3 cross(D3 a, D3 b)
{
    return d3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__host__ __device__ inline D3 unit(D3 a) { return a * bysdf::rsqrt_(dot(a, a)); }

// uniform cubic B-spline basis and its first two derivatives
__host__ __device__ inline void basis(double s, double* b)
{
    double u = 1.0 - s, s2 = s * s, s3 = s2 * s;
    b[0] = u * u * u * (1.0 / 6.0);
    b[1] = (3.0 * s3 - 6.0 * s2 + 4.0) * (1.0 / 6.0);
    b[2] = (-3.0 * s3 + 3.0 * s2 + 3.0 * s + 1.0) * (1.0 / 6.0);
    b[3] = s3 * (1.0 / 6.0);
}
__host__ __device__ inline void basis1(double s, double* b)
{
    double u = 1.0 - s;
    b[0] = -0.5 * u * u;
    b[1] = 1.5 * s * s - 2.0 * s;
    b[2] = -1.5 * s * s + s + 0.5;
    b[3] = 0.5 * s * s;
}
__host__ __device__ inline void basis2(double s, double* b)
{
    b[0] = 1.0 - s;
    b[1] = 3.0 * s - 2.0;
    b[2] = -3.0 * s + 1.0;
    b[3] = s;
}
__host__ __device__ inline D3 comb(const D3* c, const double* b)
{
    return d3(b[0] * c[0].x + b[1] * c[1].x + b[2] * c[2].x + b[3] * c[3].x,
              b[0] * c[0].y + b[1] * c[1].y + b[2] * c[2].y + b[3] * c[3].y,
              b[0] * c[0].z + b[1] * c[1].z + b[2] * c[2].z + b[3] * c[3].z);
}

// Ray-space view of one span: control points relative to the origin.
struct SpanGeo {
    D3 c[4];
    double R;
};

// Power-form coefficients a0 + a1 s + a2 s^2 + a3 s^3 of a uniform cubic
// B-spline coordinate with control values c0..c3 (the basis above, expanded).
__host__ __device__ inline void spline_power(const double* c, double* a)
{
    a[0] = (c[0] + 4.0 * c[1] + c[2]) * (1.0 / 6.0);
    a[1] = (c[2] - c[0]) * 0.5;
    a[2] = (c[0] - 2.0 * c[1] + c[2]) * 0.5;
    a[3] = (c[3] - c[0] + 3.0 * (c[1] - c[2])) * (1.0 / 6.0);
}

// A span seen from the ray: the centreline's offset (u, w) from the ray
// and its position z along it, each a cubic in s in power form.
struct RayCubic {
    double u[4], w[4], z[4];
};

__host__ __device__ inline double horner3(const double* a, double s)
{
    return fma(fma(fma(a[3], s, a[2]), s, a[1]), s, a[0]);
}

// entry T(s) = z - sqrt(R^2 - u^2 - w^2) if above t_min, else +inf
__host__ __device__ inline double entry_at(const RayCubic& rc, double R, double s, double t_min)
{
    const double u = horner3(rc.u, s), w = horner3(rc.w, s);
    const double q2 = R * R - (u * u + w * w);
    if (!(q2 > 0.0)) return INFINITY;
    const double t = horner3(rc.z, s) - bysdf::sqrt_(q2);
    return t > t_min ? t : INFINITY;
}

// dT/ds and d2T/ds2 at s; returns false where the ball misses the ray
__host__ __device__ inline bool entry_slope(const RayCubic& rc, double R, double s, double* g1, double* g2)
{
    double u = horner3(rc.u, s), w = horner3(rc.w, s);
    double q2 = R * R - (u * u + w * w);
    if (!(q2 > 0.0)) return false;
    // first and second derivatives of the three cubics
    auto d1 = [s](const double* a) { return fma(fma(3.0 * a[3], s, 2.0 * a[2]), s, a[1]); };
    auto d2 = [s](const double* a) { return fma(6.0 * a[3], s, 2.0 * a[2]); };
    const double u1 = d1(rc.u), w1 = d1(rc.w), z1 = d1(rc.z);
    const double u2 = d2(rc.u), w2 = d2(rc.w), z2 = d2(rc.z);
    const double q = bysdf::sqrt_(q2), iq = bysdf::rcp_(q);
    const double h = u * u1 + w * w1;  // (r^2)' / 2
    *g1 = z1 + h * iq;
    const double hp = u1 * u1 + w1 * w1 + u * u2 + w * w2;
    *g2 = z2 + (hp + h * h / q2) * iq;
    return true;
}

// Two unit vectors across a ray of direction d.
__host__ __device__ inline void across_ray(D3 d, D3* e1, D3* e2)
{
    const D3 a = fabs(d.x) < 0.9 ? d3(1, 0, 0) : d3(0, 1, 0);
    *e1 = unit(cross(d, a));
    *e2 = cross(d, *e1);
}

// A span to sample: its view from the ray, R^2 and 1 / samples.
struct SpanView {
    RayCubic rc;
    double R2, inv;
};

// Whether a span may be entered at t_min < t <= t_lim: false when the hull of
// its control points misses the ray's R-slab in that range.  Fills its view.
__host__ __device__ inline bool span_view(const SpanGeo& g, D3 d, D3 e1, D3 e2, double t_min, double t_lim,
                                          int nsamp, SpanView* v)
{
    const double R = g.R;
    bool all_pu = true, all_nu = true, all_pw = true, all_nw = true, all_b = true, all_f = true;
    double pu[4], pw[4], pz[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double u = dot(g.c[k], e1), w = dot(g.c[k], e2), z = dot(g.c[k], d);
        pu[k] = u;
        pw[k] = w;
        pz[k] = z;
        all_pu &= u > R;
        all_nu &= u < -R;
        all_pw &= w > R;
        all_nw &= w < -R;
        all_b &= z + R < t_min;
        all_f &= z - R > t_lim;
    }
    if (all_pu || all_nu || all_pw || all_nw || all_b || all_f) return false;
    // the curve lies in the hull of its control points: in the plane across
    // the ray, a hull entirely more than R to one side of the line through
    // the outer two points' direction (the span's chord) misses the ray; the
    // outer points are equally far from that line
    {
        const double cx = pu[3] - pu[0], cy = pw[3] - pw[0];
        const double rl = R * bysdf::sqrt_(cx * cx + cy * cy);
        bool all_p = true, all_n = true;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double sd = cx * pw[k] - cy * pu[k];
            all_p &= sd > rl;
            all_n &= sd < -rl;
        }
        if (rl > 1e-12 * R * R && (all_p || all_n)) return false;
    }
    // in the ray's frame (e1, e2, d) the centreline's offset (u, w) from the
    // ray and its position z along it are cubics in s, in power form from the
    // projected control points, so a sample costs three Horner steps per
    // coordinate and r^2 = u^2 + w^2 has no cancellation
    spline_power(pu, v->rc.u);
    spline_power(pw, v->rc.w);
    spline_power(pz, v->rc.z);
    v->R2 = R * R;
    v->inv = 1.0 / nsamp;
    return true;
}

// The smallest entry T(s_i) > t_min over the samples i = i0, i0 + di, ... <=
// nsamp and its index (+inf, -1: none).
__host__ __device__ inline void span_sample(const SpanView& v, double t_min, int i0, int di, int nsamp,
                                            double* t_out, int* i_out)
{
    double bt = INFINITY;
    int bi = -1;
    for (int i = i0; i <= nsamp; i += di) {
        const double s = i * v.inv, u = horner3(v.rc.u, s), w = horner3(v.rc.w, s);
        const double q2 = fma(-u, u, fma(-w, w, v.R2));
        // a ball that misses the ray (q2 <= 0) makes the root a NaN, which no
        // comparison takes
        const double t = horner3(v.rc.z, s) - bysdf::sqrt_positive(q2);
        const bool in = t > t_min && t < bt;
        bt = in ? t : bt;
        bi = in ? i : bi;
    }
    *t_out = bt;
    *i_out = bi;
}

// The entry at sample bi of a span whose ball there meets the ray.  Where two
// spans join, both hold the same entry up to rounding, and the last bits of
// this value and of the refined one say which of them is reported; every
// product is fused as written, so that all kernels report the same span.  The
// order of the z projection's products differs between even and odd control
// points for no reason of geometry: it is the order in which the compiler
// fused them when the traversal had one lane per ray, kept so that the span
// reported at a joint stays the same.
// The scan decided that the ball meets the ray from products fused in another
// order; a ray that touches the ball may have a half chord squared below zero
// here, by rounding, and it is zero then.
__host__ __device__ inline double sample_entry(const SpanGeo& g, D3 d, D3 e1, D3 e2, int nsamp, int bi)
{
#pragma clang fp contract(off)
    auto across = [](D3 a, D3 b) { return fma(a.z, b.z, fma(a.x, b.x, a.y * b.y)); };
    auto power = [](const double* c, double s) {
        const double a0 = (fma(4.0, c[1], c[0]) + c[2]) * (1.0 / 6.0), a1 = (c[2] - c[0]) * 0.5;
        const double a2 = (fma(-2.0, c[1], c[0]) + c[2]) * 0.5;
        const double a3 = fma(3.0, c[1] - c[2], c[3] - c[0]) * (1.0 / 6.0);
        return fma(fma(fma(a3, s, a2), s, a1), s, a0);
    };
    double pu[4], pw[4], pz[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        pu[k] = across(g.c[k], e1);
        pw[k] = across(g.c[k], e2);
        pz[k] = k & 1 ? across(g.c[k], d) : fma(g.c[k].z, d.z, fma(g.c[k].y, d.y, g.c[k].x * d.x));
    }
    const double s = bi * (1.0 / nsamp), u = power(pu, s), w = power(pw, s);
    const double q2 = g.R * g.R - fma(u, u, w * w);
    return power(pz, s) - bysdf::sqrt_(fmax(q2, 0.0));
}

// Minimum of T in the bracket of sample bi (best sampled value bt):
// safeguarded Newton on dT/ds in double precision.
__host__ __device__ inline void span_refine(const SpanGeo& g, D3 d, D3 e1, D3 e2, double t_min, int nsamp, int bi,
                                            double bt, double* t_out, double* s_out)
{
    RayCubic rc;
    {
        // Newton's last steps move s by far more than an ulp when a product
        // rounds differently, so the order of these sums is fixed here and
        // not left to how the compiler fuses them in each place
        auto proj = [](D3 a, D3 b) { return fma(a.z, b.z, fma(a.y, b.y, a.x * b.x)); };
        double pu[4], pw[4], pz[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pu[k] = proj(g.c[k], e1);
            pw[k] = proj(g.c[k], e2);
            pz[k] = proj(g.c[k], d);
        }
        spline_power(pu, rc.u);
        spline_power(pw, rc.w);
        spline_power(pz, rc.z);
    }
    const double R = g.R;
    const double inv = 1.0 / nsamp;
    double lo = bi > 0 ? (bi - 1) * inv : 0.0, hi = bi < nsamp ? (bi + 1) * inv : 1.0;
    double s = bi * inv, g1, g2;
    // slope at the bracket ends (a ball that misses the ray reads as a
    // steep wall: -inf on the left, +inf on the right)
    double glo = entry_slope(rc, R, lo, &g1, &g2) ? g1 : -INFINITY;
    double ghi = entry_slope(rc, R, hi, &g1, &g2) ? g1 : INFINITY;
    double sb = s;
    if (glo >= 0.0) {
        sb = lo;
    } else if (ghi <= 0.0) {
        sb = hi;
    } else {
        for (int it = 0; it < 24; ++it) {
            double sn;
            if (entry_slope(rc, R, s, &g1, &g2)) {
                if (g1 < 0.0)
                    lo = s;
                else
                    hi = s;
                sn = s - g1 * bysdf::rcp_(g2);
                if (!(g2 > 0.0) || !(sn > lo && sn < hi)) sn = 0.5 * (lo + hi);
            } else {
                sn = 0.5 * (lo + hi);
            }
            bool done = fabs(sn - s) < 1e-15 || hi - lo < 1e-15;
            s = sn;
            if (done) break;
        }
        sb = s;
    }
    double t = entry_at(rc, R, sb, t_min);
    // where T is flat the refined value ties the best sample to rounding:
    // keep the refined parameter
    if (t <= bt + 1e-12 * fmax(1.0, fabs(bt))) {
        *t_out = fmin(t, bt);
        *s_out = sb;
    } else {
        *t_out = bt;
        *s_out = bi * inv;
    }
}

__host__ __device__ inline void load_span(const SceneView& S, const SpanRec& r, D3 o, SpanGeo* g)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float4 p = S.cp[r.cp0 + k];
        g->c[k] = d3((double)p.x - o.x, (double)p.y - o.y, (double)p.z - o.z);
        if (k == 0) g->R = (double)p.w;
    }
}

// Whether the curve comes closer than lim to the origin of the span view,
// as the squared distance from the samples refined by safeguarded Newton on
// the derivative of |C(s)|^2 decides it.  Two exits skip the refinement
// without changing the answer: a sample already closer than lim (the
// refinement only lowers the minimum), and samples all farther than
// lim + L / (2 nsamp), with L = max_k |c_{k+1} - c_k| bounding the speed
// |C'(s)| (the derivative of a uniform cubic B-spline segment is a convex
// combination of its control-point differences), so that no point of the
// curve, being within 1 / (2 nsamp) of a sample, can come closer than lim.
__host__ __device__ inline bool span_within(const SpanGeo& g, int nsamp, double lim)
{
    // the centreline relative to the point, a cubic per coordinate
    double cx[4], cy[4], cz[4], ax[4], ay[4], az[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        cx[k] = g.c[k].x;
        cy[k] = g.c[k].y;
        cz[k] = g.c[k].z;
    }
    spline_power(cx, ax);
    spline_power(cy, ay);
    spline_power(cz, az);
    auto at = [&](double s) { return d3(horner3(ax, s), horner3(ay, s), horner3(az, s)); };
    double inv = 1.0 / nsamp, bv = INFINITY;
    int bi = 0;
    for (int i = 0; i <= nsamp; ++i) {
        D3 p = at(i * inv);
        double v = dot(p, p);
        if (v < bv) {
            bv = v;
            bi = i;
        }
    }
    const double lim2 = lim * lim;
    if (bv < lim2) return true;
    double L2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const D3 dc = g.c[k + 1] - g.c[k];
        L2 = fmax(L2, dot(dc, dc));
    }
    // the relative margin covers the rounding of the samples and of L
    const double m = lim + 0.5 * bysdf::sqrt_(L2) * inv;
    if (bv > m * m * (1.0 + 1e-9)) return false;
    double lo = bi > 0 ? (bi - 1) * inv : 0.0, hi = bi < nsamp ? (bi + 1) * inv : 1.0, s = bi * inv;
    for (int it = 0; it < 20; ++it) {
        D3 p = at(s);
        auto d1 = [s](const double* a) { return fma(fma(3.0 * a[3], s, 2.0 * a[2]), s, a[1]); };
        auto d2 = [s](const double* a) { return fma(6.0 * a[3], s, 2.0 * a[2]); };
        D3 p1 = d3(d1(ax), d1(ay), d1(az)), p2 = d3(d2(ax), d2(ay), d2(az));
        double f1 = dot(p, p1), f2 = dot(p1, p1) + dot(p, p2);
        double v = dot(p, p);
        if (v < bv) bv = v;
        if (f1 < 0.0)
            lo = s;
        else
            hi = s;
        double sn = s - f1 * bysdf::rcp_(f2);
        if (!(f2 > 0.0) || !(sn > lo && sn < hi)) sn = 0.5 * (lo + hi);
        if (fabs(sn - s) < 1e-15) break;
        s = sn;
    }
    D3 p = at(s);
    double v = dot(p, p);
    return (v < bv ? v : bv) < lim2;
}
// True when the span is certainly farther than lim from the origin of the
// span view: the curve lies in the hull of its control points, which lies
// within the slab of the chord direction they span and within the
// cylinder around the chord line that holds them.
__host__ __device__ inline bool span_far(const SpanGeo& g, double lim)
{
    D3 ch = g.c[3] - g.c[0];
    double cl2 = dot(ch, ch);
    if (!(cl2 > 0.0)) return false;
    D3 t = ch * bysdf::rsqrt_(cl2);
    bool all_p = true, all_n = true;
    double rho2 = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double a = dot(g.c[k], t);
        all_p &= a > lim;
        all_n &= a < -lim;
        D3 q = g.c[k] - g.c[0];
        D3 pq = q - t * dot(q, t);
        rho2 = fmax(rho2, dot(pq, pq));
    }
    if (all_p || all_n) return true;
    D3 p0 = g.c[0] - t * dot(g.c[0], t);  // origin to the chord line
    double dl = bysdf::sqrt_(dot(p0, p0)) - bysdf::sqrt_(rho2);
    return dl > lim;
}

__host__ __device__ inline void decode_leaf(int code, int* first, int* count)
{
    int c = -code - 1;
    *first = c >> 2;
    *count = (c & 3) + 1;
}
__host__ __device__ inline int leaf_code(int first, int count) { return -((first << 2) | (count - 1)) - 1; }
// end of a traversal: below every leaf code of a scene of fewer than 2^29 spans
constexpr int kTraceDone = INT32_MIN;

// ---------------------------------------------------------------- four lanes per ray
// The traversal kernels give each ray the four lanes of a quad (16 rays per
// wavefront).  A lane tests one child of a 4-wide node and scans one span of
// a leaf (leaves hold up to four), so a node or leaf step of a ray takes a
// quarter of the instructions in a row that one lane would need, and a
// wavefront waits for the longest of 16 rays instead of 64.  Every lane of a
// quad holds the ray's state and takes the same branches; the exchanges
// below are register moves within the quad (DPP), and the ray's stack sits in
// LDS, one entry per ray and level.
constexpr int kQuad = 4;

__device__ inline int quad_lane() { return __lane_id() & (kQuad - 1); }
template <int CTRL> __device__ inline int quad_perm(int x)
{
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
// the value of the lane whose index in the quad differs by the given bits
__device__ inline int quad_xor1(int x) { return quad_perm<0xb1>(x); }
__device__ inline int quad_xor2(int x) { return quad_perm<0x4e>(x); }
__device__ inline float quad_xor1(float x) { return __int_as_float(quad_xor1(__float_as_int(x))); }
__device__ inline float quad_xor2(float x) { return __int_as_float(quad_xor2(__float_as_int(x))); }
__device__ inline double quad_xor1(double x)
{
    return __hiloint2double(quad_xor1(__double2hiint(x)), quad_xor1(__double2loint(x)));
}
__device__ inline double quad_xor2(double x)
{
    return __hiloint2double(quad_xor2(__double2hiint(x)), quad_xor2(__double2loint(x)));
}
__device__ inline int quad_or(int x)
{
    x |= quad_xor1(x);
    return x | quad_xor2(x);
}
__device__ inline double quad_min(double x)
{
    x = fmin(x, quad_xor1(x));
    return fmin(x, quad_xor2(x));
}
// the predicate of the quad's four lanes as bits 0..3
__device__ inline int quad_bits(bool p)
{
    return (int)((__ballot(p) >> (__lane_id() & ~(kQuad - 1))) & 0xf);
}
// Orders the LDS accesses of a wavefront's lanes to each other's slots: LDS
// serves a wavefront's operations in issue order, so this emits nothing and
// only keeps the compiler from moving accesses across it.
__device__ inline void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// child of the calling lane in a wide node
struct ChildBox {
    float3 lo, hi;
    int code, yarn;
};
__device__ inline ChildBox load_child(const WNode* node, int code)
{
    const WChild w = node[code].child[quad_lane()];
    ChildBox b;
    b.lo = make_float3(w.lo_code.x, w.lo_code.y, w.lo_code.z);
    b.code = __float_as_int(w.lo_code.w);
    b.hi = make_float3(w.hi_yarn.x, w.hi_yarn.y, w.hi_yarn.z);
    b.yarn = __float_as_int(w.hi_yarn.w);
    return b;
}

__device__ inline bool box_ray(float3 lo, float3 hi, float3 o, float3 inv, float t0, float t1, float* tn)
{
    float ax = (lo.x - o.x) * inv.x, bx = (hi.x - o.x) * inv.x;
    float ay = (lo.y - o.y) * inv.y, by = (hi.y - o.y) * inv.y;
    float az = (lo.z - o.z) * inv.z, bz = (hi.z - o.z) * inv.z;
    float tmin = fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), fmaxf(fminf(az, bz), t0));
    float tmax = fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), fminf(fmaxf(az, bz), t1));
    // conservative against the rounding of the slab distances
    tmax *= 1.0000004f;
    *tn = tmin;
    return tmin <= tmax;
}

__device__ inline bool box_point(float3 lo, float3 hi, float3 p)
{
    return p.x >= lo.x && p.x <= hi.x && p.y >= lo.y && p.y <= hi.y && p.z >= lo.z && p.z <= hi.z;
}

// Yarns a ray skips: those whose tube holds its origin (at most
// kMaxExcluded) and the yarn it leaves.  Unused entries are -1.
struct Excluded {
    int yarn[kMaxExcluded + 1];
    int n;
    __device__ bool has(int y) const
    {
        bool h = false;
#pragma unroll
        for (int k = 0; k <= kMaxExcluded; ++k) h |= yarn[k] == y;
        return h;
    }
    __device__ void add(int y)
    {
#pragma unroll
        for (int k = 0; k <= kMaxExcluded; ++k) yarn[k] = k == n ? y : yarn[k];
        ++n;
    }
};

// Yarns whose tube holds the origin (distance to the centreline below
// R (1 - 1e-3)).  Point query through the BVH, a quad per origin; the ray's
// stack at stk[k * stride].  Yarn `skip` (-1: none) is left out of the query
// and comes first: a ray leaving a yarn skips that yarn whatever its origin.
__device__ inline Excluded excluded_yarns(const SceneView& S, D3 o, int* stk, int stride, int skip)
{
    const float3 of = make_float3((float)o.x, (float)o.y, (float)o.z);
    // the float origin may sit a rounding step outside a box that holds the
    // double origin: grow the test box by a relative ulp
    const float3 e = make_float3(fabsf(of.x) * 2.4e-7f + 1e-30f, fabsf(of.y) * 2.4e-7f + 1e-30f,
                                 fabsf(of.z) * 2.4e-7f + 1e-30f);
    const int me = quad_lane();
    Excluded ex;
#pragma unroll
    for (int k = 0; k <= kMaxExcluded; ++k) ex.yarn[k] = -1;
    ex.n = 0;
    if (skip >= 0) ex.add(skip);
    const int full = kMaxExcluded + (skip >= 0 ? 1 : 0);
    int sp = 0, code = 0;
    while (true) {
        if (code >= 0) {
            const ChildBox b = load_child(S.node, code);
            const float3 lo = make_float3(b.lo.x - e.x, b.lo.y - e.y, b.lo.z - e.z);
            const float3 hi = make_float3(b.hi.x + e.x, b.hi.y + e.y, b.hi.z + e.z);
            const int m = quad_bits(box_point(lo, hi, of) && !(skip >= 0 && b.yarn == skip));
            if (m) {
                // the last hit child is visited next, the others pushed
                const bool mine = (m >> me) & 1, last = mine && (m >> (me + 1)) == 0;
                if (mine && !last) stk[(sp + __popc(m & ((1 << me) - 1))) * stride] = b.code;
                wave_lds_order();
                sp += __popc(m) - 1;
                code = quad_or(last ? b.code : 0);
                continue;
            }
        } else {
            int first, count;
            decode_leaf(code, &first, &count);
            bool in = false;
            int y = -1;
            if (me < count) {
                const SpanRec r = S.span[first + me];
                y = r.yarn;
                if (!ex.has(y) && ex.n < full) {
                    SpanGeo g;
                    load_span(S, r, o, &g);
                    const double lim = g.R * (1.0 - kExcludeFrac);
                    in = !span_far(g, lim) && span_within(g, r.info & 0xffff, lim);
                }
            }
            const int m = quad_bits(in);
            if (m) {
                // the leaf's spans in order, each yarn once
                const int ys[kQuad] = {quad_perm<0x00>(y), quad_perm<0x55>(y), quad_perm<0xaa>(y), quad_perm<0xff>(y)};
#pragma unroll
                for (int k = 0; k < kQuad; ++k)
                    if (((m >> k) & 1) && !ex.has(ys[k]) && ex.n < full) ex.add(ys[k]);
            }
        }
        if (sp == 0) break;
        code = stk[--sp * stride];
    }
    return ex;
}

// ---------------------------------------------------------------- rays of a wavefront
// A wavefront traces the rays its lanes hold (one per lane, up to 32).  The
// search works on 16 at a time, a quad each, with the ray in LDS; the spans
// it finds go to a list, are refined one per lane whatever rays they belong
// to, and each ray's closest entry returns to its lane, which forms the hit
// with the other lanes.  So the refinement and everything after it run on
// full wavefronts, once per ray instead of once per lane of its quad, and
// the traversal keeps its registers for the span scans.
//
// Candidates for refinement are the spans whose best sample lies within
// kCandMargin R of the ray's best sample.  A minimum between samples
// undershoots its bracket's best sample by far less than that unless the
// ray only grazes the tube (samples are at most 0.05 R apart along the
// curve), so the true first entry is among them.
constexpr double kCandMargin = 0.1;

struct Candidate {
    double t;  // best sampled entry
    int span;
    unsigned tag;  // index of the sample (16 bits), lane of the ray
};
// a double's bits in an order-preserving unsigned form, and back
__device__ inline unsigned long long ordered_bits(double x)
{
    const long long b = __double_as_longlong(x);
    return (unsigned long long)b ^ ((unsigned long long)(b >> 63) | 0x8000000000000000ull);
}
__device__ inline double from_ordered(unsigned long long k)
{
    const unsigned long long b = (k >> 63) ? k ^ 0x8000000000000000ull : ~k;
    return __longlong_as_double((long long)b);
}

constexpr int kStragglers = 2 * kQuad;  // lanes still at nodes when leaves are scanned
constexpr int kRays = 32;     // rays of a wavefront at most
// spans whose samples a wavefront shares at a time: 8, 12 and 32 take 1.32,
// 1.28 and 1.27 ms on the primary rays, 16 takes 1.23 (more rounds below,
// more LDS and fewer wavefronts above)
constexpr int kShared = 16;
struct WaveRays {
    double dx[kRays], dy[kRays], dz[kRays], e1x[kRays], e1y[kRays], e1z[kRays], e2x[kRays], e2y[kRays], e2z[kRays], t_max[kRays];
    unsigned long long tb[kRays];             // smallest sampled entry so far, or t_max, as ordered bits
    unsigned long long key[kRays], key2[kRays];  // the closest entry and its sample, likewise
    double s[kRays];
    float ox[kRays], oy[kRays], oz[kRays];
    int pick[kRays];                             // its span
    int skip[kRays], list[kRays];
    int excl[kMaxExcluded + 1][kRays], n_excl[kRays];  // the ray's Excluded
    int give[kWaveRays];
    Candidate cand[128];
    // spans whose samples are shared among lanes: views, samples, results
    SpanView view[kShared];
    unsigned long long best[kShared];
    int samples[kShared], best_at[kShared];
    __device__ D3 origin(int l) const { return d3(ox[l], oy[l], oz[l]); }
    __device__ D3 dir(int l) const { return d3(dx[l], dy[l], dz[l]); }
    // two unit vectors across the ray
    __device__ D3 e1(int l) const { return d3(e1x[l], e1y[l], e1z[l]); }
    __device__ D3 e2(int l) const { return d3(e2x[l], e2y[l], e2z[l]); }
    // lane l's ray; the origin's components are single-precision values
    __device__ void set(int l, D3 o, D3 d, double tmax, int skip_yarn)
    {
        move(l, o, tmax, skip_yarn);
        dx[l] = d.x;
        dy[l] = d.y;
        dz[l] = d.z;
        D3 e1, e2;
        across_ray(d, &e1, &e2);
        e1x[l] = e1.x;
        e1y[l] = e1.y;
        e1z[l] = e1.z;
        e2x[l] = e2.x;
        e2y[l] = e2.y;
        e2z[l] = e2.z;
    }
    // what the box tests of lane l's ray take: its origin, the reciprocal
    // direction, and the slack of the slab interval, a relative ulp of the
    // origin along the ray
    __device__ void box_test(int l, float3& of, float3& inv, float& slack) const
    {
        const D3 d = dir(l);
        of = make_float3(ox[l], oy[l], oz[l]);
        inv = make_float3(1.0f / (fabs(d.x) > 1e-30 ? (float)d.x : 1e-30f),
                          1.0f / (fabs(d.y) > 1e-30 ? (float)d.y : 1e-30f),
                          1.0f / (fabs(d.z) > 1e-30 ? (float)d.z : 1e-30f));
        slack = 2.4e-7f * (fabsf(of.x) + fabsf(of.y) + fabsf(of.z)) + 1e-30f;
    }
    // the same ray from another point
    __device__ void move(int l, D3 o, double tmax, int skip_yarn)
    {
        ox[l] = (float)o.x;
        oy[l] = (float)o.y;
        oz[l] = (float)o.z;
        t_max[l] = tmax;
        tb[l] = ordered_bits(tmax);
        skip[l] = skip_yarn;
    }
};

// Whether a ray that searches its tree alone, near children first, meets span
// a before span b.  Where two spans join, or two yarns coincide, both may hold
// the same entry to the last bit; this order then says which is reported,
// whoever scanned them and when.  Only such ties come here, so the function is
// called: inlined, its registers cost the search 1 % (primary rays of the weave
// 1244 us, 1229 called).
__device__ __noinline__ inline bool met_before(const WNode* node, const int* up, int n_nodes, const WaveRays& W,
                                               int ray, int a, int b, double t_min)
{
    int ua = up[n_nodes + a], ub = up[n_nodes + b];
    if (ua == ub) return a < b;
    // up to the node where their ways part
    while (ua >> 2 != ub >> 2) {
        if (ua > ub)
            ua = up[ua >> 2];
        else
            ub = up[ub >> 2];
    }
    // the children there in the order of a five-step sorting network on their
    // entry distances: equal distances (boxes that hold the origin) keep the
    // order that such a search visits them in
    float3 of, inv;
    float slack, tn[4];
    int slot[4] = {0, 1, 2, 3};
    W.box_test(ray, of, inv, slack);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const WChild c = node[ua >> 2].child[k];
        if (!box_ray(make_float3(c.lo_code.x, c.lo_code.y, c.lo_code.z),
                     make_float3(c.hi_yarn.x, c.hi_yarn.y, c.hi_yarn.z), of, inv, (float)t_min - slack,
                     (float)W.t_max[ray] + slack, &tn[k]))
            tn[k] = INFINITY;
    }
    auto order = [&](int x, int y) {
        const bool sw = tn[y] < tn[x];
        const float t = sw ? tn[y] : tn[x];
        const int c = sw ? slot[y] : slot[x];
        tn[y] = sw ? tn[x] : tn[y];
        slot[y] = sw ? slot[x] : slot[y];
        tn[x] = t;
        slot[x] = c;
    };
    order(0, 1);
    order(2, 3);
    order(0, 2);
    order(1, 3);
    order(1, 2);
    for (int k = 0; k < 4; ++k) {
        if (slot[k] == (ua & 3)) return true;
        if (slot[k] == (ub & 3)) return false;
    }
    return false;
}

// Refines the listed candidates [first, first + n), n <= 64, one per lane, and
// folds them into their rays' closest entries (equal entries: the smaller
// sample, then met_before).  A candidate beyond its ray's margin by now is
// dropped.  Called by the whole wavefront.
__device__ inline void refine_listed(const SceneView& S, WaveRays& W, int first, int n, double t_min)
{
    const int lane = __lane_id();
    bool ok = lane < n;
    int ray = 0;
    double s = 0.0;
    unsigned long long key = ~0ull, key2 = ~0ull;
    int pick = -1;
    if (ok) {
        const Candidate c = W.cand[first + lane];
        ray = c.tag >> 16;
        pick = c.span;
        const SpanRec r = S.span[c.span];
        const int nsamp = r.info & 0xffff, at = c.tag & 0xffff;
        double bt = 0.0;
        {
            SpanGeo g;
            load_span(S, r, W.origin(ray), &g);
            ok = c.t <= from_ordered(W.tb[ray]) + kCandMargin * g.R;
            if (ok) bt = sample_entry(g, W.dir(ray), W.e1(ray), W.e2(ray), nsamp, at);
        }
        // the span and the ray are read again rather than kept in registers
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (ok) {
            SpanGeo g;
            load_span(S, r, W.origin(ray), &g);
            double t;
            span_refine(g, W.dir(ray), W.e1(ray), W.e2(ray), t_min, nsamp, at, bt, &t, &s);
            ok = t <= W.t_max[ray];
            key = ordered_bits(t);
            key2 = ordered_bits(bt);
        }
    }
    const unsigned long long before = ok ? W.key[ray] : 0ull;
    wave_lds_order();
    if (ok) atomicMin(&W.key[ray], key);
    wave_lds_order();
    bool win = ok && W.key[ray] == key;
    if (win && key < before) {
        W.key2[ray] = ~0ull;
        W.pick[ray] = -1;
    }
    wave_lds_order();
    const unsigned long long before2 = win ? W.key2[ray] : 0ull;
    wave_lds_order();
    if (win) atomicMin(&W.key2[ray], key2);
    wave_lds_order();
    win = win && W.key2[ray] == key2;
    if (win && key2 < before2) W.pick[ray] = -1;
    wave_lds_order();
    if (win && W.pick[ray] < 0) W.pick[ray] = pick;
    wave_lds_order();
    // ties: every round puts an earlier span in the place of each ray that has
    // one, of at most 64
    bool tie = win && W.pick[ray] != pick;
    for (int round = 0; round < 64 && __any((int)tie); ++round) {
        tie = tie && met_before(S.node, S.up, S.n_nodes, W, ray, pick, W.pick[ray], t_min);
        wave_lds_order();
        if (tie) W.pick[ray] = pick;
        wave_lds_order();
        tie = tie && W.pick[ray] != pick;
    }
    if (win && W.pick[ray] == pick) W.s[ray] = s;
    wave_lds_order();
}

struct RayHit {
    double t, s;
    int span;  // leaf-order span index, -1 for a miss
};

// Closest entering hits with t_min < t <= t_max of the wavefront's rays: lane
// l's ray if live, left in slot l of W by the caller.  n_ex returns how many
// yarns hold the ray's origin.  Called by the whole wavefront; stk: its
// quads' stacks, entry k of quad q at stk[16 k + q].
//
// The quads take 16 rays; a quad that is done takes the farthest pending
// subtree of a quad that still works, so that one long ray (a path that skims
// the cloth visits thousands of nodes) has up to 64 lanes, and when all are
// done they take the next 16 (a quad that took its next ray by itself would
// make the point queries of new rays run a few at a time: 1.32 against 1.20 ms
// on the weave's primary rays).  Spans are ranked by their
// sampled entries (an upper bound of the true entry, so it is safe for
// culling), and a ray's bound is shared by every quad working on it.
//
// The traversal is bound by VALU issue where the chip is full and by the
// dependent loads of the longest ray where it is not.  Against one lane per
// ray (a fan of 64 rays waits for its longest; 17 samples of a span in a row
// for any lane that needs them) a 320 x 180 preview at 4 spp and depth 4 went
// from 4.24 to 2.18 ms and a 48 x 48 crop with its gradient at 16 spp from
// 3.35 to 0.98 ms; the weave's 2.07 M primary rays take 1.23 instead of 1.25
// ms (fewer lanes idle, but rays are set up and finished 32 at a time).
__device__ inline RayHit trace_wave(const SceneView& S, WaveRays& W, int* stk, bool live, double t_min, int& n_ex)
{
    const int lane = __lane_id(), quad = lane / kQuad, me = quad_lane();
    const unsigned long long kLeaders = 0x1111111111111111ull;
    const unsigned long long below = (1ull << (lane & ~(kQuad - 1))) - 1ull;  // lanes of lower quads
    int* my = stk + quad;
    const unsigned long long m = __ballot(live);
    const int n = __popcll(m), slot = __popcll(m & ((1ull << lane) - 1ull));
    if (live) {
        W.list[slot] = lane;
        W.key[lane] = W.key2[lane] = ~0ull;
        W.pick[lane] = -1;
    }
    wave_lds_order();
    int listed = 0, next = 0;
    int ray = 0, sp = 0, bottom = 0, code = kTraceDone;
    int leaf = 0;  // the held leaf's code, 0 for none
    float3 of = make_float3(0.f, 0.f, 0.f), inv = of;
    float slack = 0.f;
    int leaving = -1, n_excl = 0;  // the ray's skip and its number of excluded yarns
    while (true) {
        const bool idle = code == kTraceDone && leaf == 0;
        const unsigned long long mi = __ballot(idle) & kLeaders;
        const int n_idle = __popcll(mi);
        bool take = false;
        if (listed >= 64 || (listed > 0 && n_idle == kWaveRays && next >= n)) {
            const int k = min(listed, 64);
            listed -= k;
            refine_listed(S, W, listed, k, t_min);
            continue;
        }
        if (n_idle == kWaveRays) {
            if (next >= n) break;
            const int k = next + quad;
            take = k < n;
            if (take) {
                ray = W.list[k];
                const int skip = W.skip[ray];
                const Excluded ex = excluded_yarns(S, W.origin(ray), my, kWaveRays, skip);
                if (me == 0) {
                    W.n_excl[ray] = ex.n;
#pragma unroll
                    for (int e = 0; e <= kMaxExcluded; ++e) W.excl[e][ray] = ex.yarn[e];
                }
                code = 0;
            }
            next += kWaveRays;
            wave_lds_order();
        } else if (n_idle > 0) {
            const bool gives = !idle && sp > bottom;
            const unsigned long long mg = __ballot(gives) & kLeaders;
            if (mg) {
                const int rank = __popcll((idle ? mi : mg) & below);
                if (gives && me == 0) W.give[rank] = quad;
                wave_lds_order();
                take = idle && rank < __popcll(mg);
                const int from = take ? W.give[rank] : quad;
                const int fray = __shfl(ray, from * kQuad), fbottom = __shfl(bottom, from * kQuad);
                if (take) {
                    ray = fray;
                    code = stk[fbottom * kWaveRays + from];
                }
                if (gives && rank < n_idle) ++bottom;
                wave_lds_order();
            }
        }
        if (take) {
            W.box_test(ray, of, inv, slack);
            leaving = W.skip[ray];
            n_excl = W.n_excl[ray];
            sp = bottom = 0;
            if (code < 0) {
                leaf = code;
                code = kTraceDone;
            }
        }
        // Two inner loops (the while-while form of Aila and Laine, HPG 2009,
        // with their postponed leaves): a ray that reaches a leaf holds it
        // and goes on through nodes until all but two quads hold a leaf or are
        // done (1.200 ms on the primary rays; none 1.225, four 1.212);
        // then the held leaves are scanned, one span per lane.  A quad may
        // visit nodes before scanning a leaf it holds, with the larger bound
        // of that moment, and the spans of a leaf are scanned with the bound
        // from before it: that costs only pruning.  A span that survives the
        // final filter of the candidates (sampled entry within kCandMargin R
        // of the ray's smallest) passes the scan limit whenever it is
        // scanned, and equal entries are settled by met_before, so the hit
        // does not depend on the order.
        double tb = from_ordered(W.tb[ray]);
        const float t0 = (float)t_min - slack, t1 = (float)tb + slack;
        while (code >= 0) {
            const ChildBox b = load_child(S.node, code);
            float tn;
            // an unused slot's box lies at infinity, which t1 may equal
            const bool hit = box_ray(b.lo, b.hi, of, inv, t0, t1, &tn) && tn < INFINITY &&
                             !(leaving >= 0 && b.yarn == leaving);
            if (!hit) tn = INFINITY;
            // the rank of this lane's child, near first; ties in lane order
            const float n1 = quad_xor1(tn), n2 = quad_xor2(tn), n3 = quad_xor2(n1);
            const int rank = (n1 < tn || (n1 == tn && (me & 1))) + (n2 < tn || (n2 == tn && (me & 2))) +
                             (n3 < tn || (n3 == tn && (me & 2)));
            const int nh = __popc(quad_bits(hit));
            if (nh > 0) {
                // push the farther hits, farthest first
                if (hit && rank > 0) my[(sp + nh - 1 - rank) * kWaveRays] = b.code;
                wave_lds_order();
                sp += nh - 1;
                code = quad_or(rank == 0 ? b.code : 0);
            } else {
                code = sp > bottom ? my[--sp * kWaveRays] : kTraceDone;
            }
            if (leaf == 0 && code < 0 && code != kTraceDone) {
                leaf = code;
                code = sp > bottom ? my[--sp * kWaveRays] : kTraceDone;
            }
            if (__popcll(__ballot(leaf == 0 && code != kTraceDone)) <= kStragglers) break;
        }
        double t = INFINITY, lim = 0.0;
        int bi = -1, span = -1, nsamp = 0;
        SpanView v;
        bool sample = false;
        if (leaf != 0) {
            int first, count;
            decode_leaf(leaf, &first, &count);
            if (me < count) {
                span = first + me;
                const SpanRec r = S.span[span];
                bool skip = false;
                for (int e = 0; e < n_excl; ++e) skip |= W.excl[e][ray] == r.yarn;
                if (!skip) {
                    SpanGeo g;
                    load_span(S, r, d3(of.x, of.y, of.z), &g);
                    lim = fmin(W.t_max[ray], tb + kCandMargin * g.R);
                    nsamp = r.info & 0xffff;
                    sample = span_view(g, W.dir(ray), W.e1(ray), W.e2(ray), t_min, lim, nsamp, &v);
                }
            }
            leaf = 0;
            if (code < 0 && code != kTraceDone) {
                // a leaf met meanwhile
                leaf = code;
                code = sp > bottom ? my[--sp * kWaveRays] : kTraceDone;
            }
        }
        // The spans left to sample are few (about a third of the lanes' spans):
        // their views go through LDS and the wavefront's 64 lanes share the
        // samples, 4 to 32 lanes per span, which cuts the longest part of a
        // leaf step from 17 samples in a row to 5 or fewer.
        for (unsigned long long ms; (ms = __ballot(sample)) != 0;) {
            const int n_s = min(__popcll(ms), kShared), at = __popcll(ms & ((1ull << lane) - 1ull));
            const bool mine = sample && at < kShared;
            if (mine) {
                W.view[at] = v;
                W.samples[at] = nsamp;
                W.best[at] = ~0ull;
                W.best_at[at] = INT32_MAX;
            }
            wave_lds_order();
            const int sh = min(5, __clz(n_s - 1) - 26);  // log2 of the lanes per span
            const int k = lane >> sh;
            double st = INFINITY;
            int si = -1;
            if (k < n_s) {
                const SpanView vk = W.view[k];
                span_sample(vk, t_min, lane & ((1 << sh) - 1), 1 << sh, W.samples[k], &st, &si);
                if (si >= 0) atomicMin(&W.best[k], ordered_bits(st));
            }
            wave_lds_order();
            if (si >= 0 && W.best[k] == ordered_bits(st)) atomicMin(&W.best_at[k], si);
            wave_lds_order();
            if (mine) {
                if (W.best_at[at] != INT32_MAX) {
                    bi = W.best_at[at];
                    t = from_ordered(W.best[at]);
                }
                sample = false;
            }
        }
        const bool add = bi >= 0 && t <= lim;
        const unsigned long long ma = __ballot(add);
        if (ma) {
            if (add) {
                const int k = __popcll(ma & ((1ull << lane) - 1ull));
                W.cand[listed + k] = Candidate{t, span, (unsigned)bi | (unsigned)ray << 16};
                atomicMin(&W.tb[ray], ordered_bits(t));
            }
            wave_lds_order();
            listed += __popcll(ma);
        }
    }
    RayHit h{INFINITY, 0.0, -1};
    n_ex = 0;
    if (live) {
        n_ex = W.n_excl[lane] - (W.skip[lane] >= 0 ? 1 : 0);
        if (W.pick[lane] >= 0) {
            h.t = from_ordered(W.key[lane]);
            h.s = W.s[lane];
            h.span = W.pick[lane];
        }
    }
    wave_lds_order();
    return h;
}

// Rays a wavefront takes per visit of its lanes: 32 where that leaves the
// chip full (4,096 wavefronts from 131,072 rays on), 16 for the short queues
// of late bounces and small batches, whose time is the longest ray's and not
// the issue rate.  Random rays onto a weave of 128 x 128 yarns, 16 and 32 a
// wavefront: 16,384 rays 148 and 236 us, 131,072 rays 403 and 470, 524,288
// rays 1343 and 1336, 1,048,576 rays 2567 and 2500.
__host__ __device__ inline int rays_per_wave(int64_t n) { return n >= 2 * 65536 ? kRays : kWaveRays; }

// Frame, h and arc length at a hit.
struct HitFrame {
    D3 T, N, B, c;  // tangent, reference normal, binormal, centreline point
    double v;       // arc length from the yarn start
};

__host__ __device__ inline HitFrame hit_frame(const SceneView& S, int span, double s)
{
    SpanRec r = S.span[span];
    D3 c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float4 p = S.cp[r.cp0 + k];
        c[k] = d3(p.x, p.y, p.z);
    }
    double b[4];
    basis(0.0, b);
    D3 x0 = comb(c, b);
    basis1(0.0, b);
    D3 t0 = unit(comb(c, b));
    basis(s, b);
    D3 x1 = comb(c, b);
    basis1(s, b);
    D3 t1 = unit(comb(c, b));
    float4 f = S.frame[span];
    D3 n0 = d3(f.x, f.y, f.z);
    // one double-reflection step of the rotation-minimising frame
    // (Wang, Juettler, Zheng and Liu 2008) from the span start to s
    // a chord at rounding level has a random direction; its limit for a
    // vanishing step is the tangent
    D3 v1 = x1 - x0;
    double c1 = dot(v1, v1);
    if (!(c1 > 1e-16 * (dot(x0, x0) + dot(x1, x1)))) {
        v1 = t0;
        c1 = 1.0;
    }
    D3 nl = n0 - v1 * (2.0 * dot(v1, n0) / c1);
    D3 tl = t0 - v1 * (2.0 * dot(v1, t0) / c1);
    D3 v2 = t1 - tl;
    double c2 = dot(v2, v2);
    if (c2 > 0.0) nl = nl - v2 * (2.0 * dot(v2, nl) / c2);
    HitFrame h;
    h.T = t1;
    h.N = unit(nl - t1 * dot(nl, t1));
    h.B = cross(h.T, h.N);
    h.c = x1;
    // arc length inside the span: 5-point Gauss-Legendre on [0, s]
    const double gx[5] = {0.0, -0.5384693101056831, 0.5384693101056831, -0.9061798459386640,
                          0.9061798459386640};
    const double gw[5] = {0.5688888888888889, 0.4786286704993665, 0.4786286704993665,
                          0.2369268850561891, 0.2369268850561891};
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        basis1(0.5 * s * (1.0 + gx[k]), b);
        D3 dd = comb(c, b);
        acc += gw[k] * bysdf::sqrt_(dot(dd, dd));
    }
    h.v = (double)f.w + 0.5 * s * acc;
    return h;
}

// Rays [i, i + count) by one wavefront, lane l ray i + l: exclusion point
// query, closest entering hit, hit frame, h, v.
__device__ inline void intersect_rays(const SceneView& S, int64_t i0, int count, const yarn_ray_soa& R, double t_min,
                                      const yarn_hit_soa& H, WaveRays& W, int* stk)
{
    const int lane = __lane_id();
    const int64_t i = i0 + lane;
    const bool in = lane < count;
    uint32_t flags = 0;
    bool ok = false;
    if (in) {
        const D3 o = d3(R.o_x[i], R.o_y[i], R.o_z[i]);
        const D3 dr = d3(R.d_x[i], R.d_y[i], R.d_z[i]);
        const double tm = R.t_max[i];
        const double l2 = dot(dr, dr);
        ok = __builtin_isfinite(o.x) && __builtin_isfinite(o.y) && __builtin_isfinite(o.z) &&
             __builtin_isfinite(l2) && l2 > 0.0 && !__builtin_isnan(tm);
        if (ok) {
            W.set(lane, o, dr * (1.0 / sqrt(l2)), tm, -1);
        } else {
            flags |= HIT_BAD_INPUT;
        }
    }
    int n_ex;
    const RayHit hit = trace_wave(S, W, stk, ok, t_min, n_ex);
    if (n_ex) flags |= HIT_EXCLUDED;
    if (!in) return;
    if (hit.span >= 0) {
        const D3 o = W.origin(lane), d = W.dir(lane);
        SpanRec r = S.span[hit.span];
        HitFrame f = hit_frame(S, hit.span, hit.s);
        D3 p = o + d * hit.t;
        D3 q = p - f.c;
        double qn = dot(q, f.N), qb = dot(q, f.B);
        double wn = -dot(d, f.N), wb = -dot(d, f.B);
        double ql = sqrt(qn * qn + qb * qb), wl = sqrt(wn * wn + wb * wb);
        double h = (ql > 0.0 && wl > 0.0) ? (qb * wn - qn * wb) / (ql * wl) : 0.0;
        h = fmin(1.0, fmax(-1.0, h));
        if (((r.info >> 16) & 1) && hit.s <= 0.0) flags |= HIT_CAP;
        if (((r.info >> 17) & 1) && hit.s >= 1.0) flags |= HIT_CAP;
        H.t[i] = (float)hit.t;
        H.yarn[i] = r.yarn;
        H.seg[i] = r.seg;
        H.s[i] = (float)hit.s;
        H.h[i] = (float)h;
        H.u[i] = S.yarn_phase[r.yarn];
        H.v[i] = (float)f.v;
        H.tan_x[i] = (float)f.T.x;
        H.tan_y[i] = (float)f.T.y;
        H.tan_z[i] = (float)f.T.z;
        H.nrm_x[i] = (float)f.N.x;
        H.nrm_y[i] = (float)f.N.y;
        H.nrm_z[i] = (float)f.N.z;
        H.flags[i] = flags;
        return;
    }
    H.t[i] = INFINITY;
    H.yarn[i] = -1;
    H.seg[i] = -1;
    H.s[i] = 0.f;
    H.h[i] = 0.f;
    H.u[i] = 0.f;
    H.v[i] = 0.f;
    H.tan_x[i] = H.tan_y[i] = H.tan_z[i] = 0.f;
    H.nrm_x[i] = H.nrm_y[i] = H.nrm_z[i] = 0.f;
    H.flags[i] = flags | HIT_MISS;
}

}  // namespace yarn
