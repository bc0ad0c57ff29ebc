// Lossy 128-bit arc codec (the compressive arc representation of Sec.
// 4.2.1, error bound Eq. 5).  An arc x(t) = c + a sin t + b cos t,
// t in [t1, t2] (node-local) keeps: a as (r, theta, phi) on 12 / 15 / 16
// bits with r in [R_min, 4 R_max]; the length of b on 12 bits in
// [0.1 R_min, R_max] (its direction is a x d / |a x d| for a reference
// direction d recomputed from the lattice: the strut's own direction for a
// tangency circle, the normal (g_p - g_q) / |g_p - g_q| of the seam plane
// for an ellipse); c as (r, theta, phi) with r in [0, R_max]; t1 on 15 bits
// over [0, 2 pi) and the span t2 - t1 on 15 bits over [0, 2 pi].  Fields go
// least significant bit first into four 32-bit words in that order.  An arc
// outside these ranges, or whose b does not lie where a x d puts it, is kept
// whole in a fallback list (its code then holds the list slot).
//
// Quantisation decides integers, so the encoder computes in FP64 and this
// file is compiled without floating-point contraction.
#include <math.h>

#include "common.h"

namespace lm {
namespace {

constexpr int kNr = 12, kMth = 15, kMph = 16, kNt = 15;
constexpr double kPi = 3.14159265358979323846;

struct D3 {
    double x, y, z;
};
__device__ inline D3 d3(double x, double y, double z) { return D3{x, y, z}; }
__device__ inline D3 sub(D3 a, D3 b) { return d3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ inline D3 scl(D3 a, double s) { return d3(a.x * s, a.y * s, a.z * s); }
__device__ inline D3 dvd(D3 a, double s) { return d3(a.x / s, a.y / s, a.z / s); }
__device__ inline double nrm(D3 a) { return sqrt(a.x * a.x + a.y * a.y + a.z * a.z); }
__device__ inline D3 crs(D3 a, D3 b)
{
    return d3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}

struct CodecArgs {
    Inputs in;
    Work w;
    const float *arc;       // [11][ld]
    const uint32_t *u32;    // [3][ld]: p | q << 8 | whole << 16, ends, node
    int64_t E, ld;
    double rmin, rmax;
    double step_a, step_b, step_c;  // of the three lengths' codes
    uint32_t *codes;        // [E][4]
    uint32_t *mask;         // [(E + 31) / 32]
    float *fb;              // [fb_cap][11]
    int64_t fb_cap;
    unsigned long long *fb_n;
    float *out;             // decode: [11][ld_out]
    int64_t ld_out;
};

// Strut of label lab (1..v) at node n, centre c, in FP64: its unit direction,
// or g = e / kappa = d / sqrt(|d|^2 - (r - r_far)^2) for d = far - node, with
// one square root either way; whether it runs to a higher node id.
__device__ inline bool strut_dir(const CodecArgs &A, int64_t n, float4 c, int lab, bool unit, D3 &g)
{
    const int2 he = A.w.he[A.w.row[n] + lab - 1];
    const float4 f = A.w.node4[he.x];
    const D3 d = sub(d3(f.x, f.y, f.z), d3(c.x, c.y, c.z));
    const double dr = unit ? 0.0 : (double)c.w - (double)f.w;
    g = dvd(d, sqrt(d.x * d.x + d.y * d.y + d.z * d.z - dr * dr));
    return (int64_t)he.x > n;
}

// The reference direction of arc j: for a circle the strut's direction from
// the lower to the higher node id, for an ellipse the normal of the seam
// plane.
__device__ inline D3 ref_dir(const CodecArgs &A, int64_t j)
{
    const uint32_t u0 = A.u32[j];
    const int p = (int)(u0 & 0xffu), q = (int)((u0 >> 8) & 0xffu);
    const int64_t n = (int64_t)A.u32[2 * A.ld + j];
    const float4 c = A.w.node4[n];
    D3 gq, gp;
    const bool up = strut_dir(A, n, c, q, p == 0, gq);
    if (p == 0) return up ? gq : scl(gq, -1.0);
    strut_dir(A, n, c, p, false, gp);
    const D3 nv = sub(gp, gq);
    return dvd(nv, nrm(nv));
}

__device__ inline uint32_t qlin(double v, double lo, double hi, int bits)
{
    const double levels = (double)((1 << bits) - 1);
    double s = (v - lo) / (hi - lo) * levels;
    s = s < 0.0 ? 0.0 : (s > levels ? levels : s);
    return (uint32_t)rint(s);
}
__host__ __device__ constexpr double lin_step(double lo, double hi, int bits)
{
    return (hi - lo) / (double)((1 << bits) - 1);
}
__device__ inline uint32_t qper(double ang, int bits)
{
    const double n = (double)(1u << bits);
    return (uint32_t)(int64_t)rint(ang / (2.0 * kPi) * n) & ((1u << bits) - 1);
}
__device__ inline double dper(uint32_t q, int bits) { return (double)q * (2.0 * kPi) / (double)(1u << bits); }

__device__ inline void sph(D3 v, double &r, double &th, double &ph)
{
    r = nrm(v);
    double z = r > 0.0 ? v.z / r : 1.0;
    z = z < -1.0 ? -1.0 : (z > 1.0 ? 1.0 : z);
    th = acos(z);
    ph = atan2(v.y, v.x);
    if (ph < 0.0) ph = ph + 2.0 * kPi;
}
// sin and cos of quarter turn k plus x, |x| <= pi / 4, by their series
// (the first terms left out are below 1e-19 and 2.1e-18)
__device__ inline void sincos_at(int k, double x, double &s, double &c)
{
    constexpr double S[8] = {-1.0 / 6,          1.0 / 120,           -1.0 / 5040,           1.0 / 362880,
                             -1.0 / 39916800.0, 1.0 / 6227020800.0, -1.0 / 1307674368000.0, 1.0 / 355687428096000.0};
    constexpr double C[7] = {1.0 / 24,          -1.0 / 720,         1.0 / 40320,           -1.0 / 3628800,
                             1.0 / 479001600.0, -1.0 / 87178291200.0, 1.0 / 20922789888000.0};
    const double z = x * x, h = 0.5 * z, w = 1.0 - h;
    double ps = S[7], pc = C[6];
#pragma unroll
    for (int i = 6; i >= 0; --i) ps = fma(ps, z, S[i]);
#pragma unroll
    for (int i = 5; i >= 0; --i) pc = fma(pc, z, C[i]);
    const double sx = fma(x * z, ps, x), cx = w + fma(z * z, pc, (1.0 - w) - h);
    s = k & 1 ? cx : sx;
    c = k & 1 ? sx : cx;
    s = k & 2 ? -s : s;
    c = (k + 1) & 2 ? -c : c;
}
// Unit vector along the quantised angles.  A code is a whole number
// of steps, so its quarter turn and the rest are found exactly; the general
// sin and cos spent most of the decoder's time on their reduction (with them
// 63 us for 1.65 M arcs of octet 24^3, with these 54 us; then the strut table
// with one square root per strut and a's direction as it comes, 40 us).
__device__ inline D3 unit_at(uint32_t qth, uint32_t qph)
{
    constexpr int T = (1 << kMth) - 1;  // theta = pi q / T
    const int kt = (int)((4 * qth + T) / (2 * T));
    double st, ct, sp, cp;
    sincos_at(kt, (double)(2 * (int)qth - T * kt) * (kPi / (2 * T)), st, ct);
    constexpr int Q = 1 << (kMph - 2);  // phi = (pi / 2) q / Q
    const int kp = (int)((qph + Q / 2) / Q);
    sincos_at(kp, (double)((int)qph - Q * kp) * (kPi / (2 * Q)), sp, cp);
    return d3(st * cp, st * sp, ct);
}

struct Bits {
    unsigned long long lo = 0, hi = 0;
    int pos = 0;
    __device__ void put(uint32_t v, int bits)
    {
        const unsigned long long x = (unsigned long long)v;
        if (pos >= 64) {
            hi |= x << (pos - 64);
        } else {
            lo |= x << pos;
            if (pos + bits > 64) hi |= x >> (64 - pos);
        }
        pos += bits;
    }
    __device__ uint32_t get(int bits)
    {
        unsigned long long x;
        if (pos >= 64) {
            x = hi >> (pos - 64);
        } else {
            x = lo >> pos;
            if (pos + bits > 64) x |= hi << (64 - pos);
        }
        pos += bits;
        return (uint32_t)(x & ((1ull << bits) - 1));
    }
};

__global__ void k_arc_encode(CodecArgs A)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= A.E) return;
    const D3 c = d3(A.arc[j], A.arc[A.ld + j], A.arc[2 * A.ld + j]);
    const D3 a = d3(A.arc[3 * A.ld + j], A.arc[4 * A.ld + j], A.arc[5 * A.ld + j]);
    const D3 b = d3(A.arc[6 * A.ld + j], A.arc[7 * A.ld + j], A.arc[8 * A.ld + j]);
    const double t1 = A.arc[9 * A.ld + j], t2 = A.arc[10 * A.ld + j];
    const D3 d = ref_dir(A, j);
    double ra, tha, pha, rc, thc, phc;
    sph(a, ra, tha, pha);
    sph(c, rc, thc, phc);
    const double rb = nrm(b), span = t2 - t1;
    const D3 ah = dvd(a, ra > 0.0 ? ra : 1.0);
    const D3 x = crs(ah, d);
    const double xn = nrm(x);
    const D3 bh = dvd(x, xn > 0.0 ? xn : 1.0);
    const D3 bd = dvd(b, rb > 0.0 ? rb : 1.0);
    const bool ok = ra >= A.rmin && ra <= 4.0 * A.rmax && rb >= 0.1 * A.rmin && rb <= A.rmax && rc <= A.rmax &&
                    t1 >= 0.0 && t1 < 2.0 * kPi && span >= 0.0 && span <= 2.0 * kPi && xn > 1e-6 &&
                    nrm(sub(bh, bd)) <= 1e-3;
    // two words of the mask per wave
    const unsigned long long whole = __ballot(!ok);
    if ((threadIdx.x & 31) == 0) A.mask[j >> 5] = (uint32_t)(whole >> (threadIdx.x & 32));
    uint32_t *w = A.codes + 4 * j;
    if (ok) {
        Bits B;
        B.put(qlin(ra, A.rmin, 4.0 * A.rmax, kNr), kNr);
        B.put(qlin(tha, 0.0, kPi, kMth), kMth);
        B.put(qper(pha, kMph), kMph);
        B.put(qlin(rb, 0.1 * A.rmin, A.rmax, kNr), kNr);
        B.put(qlin(rc, 0.0, A.rmax, kNr), kNr);
        B.put(qlin(thc, 0.0, kPi, kMth), kMth);
        B.put(qper(phc, kMph), kMph);
        B.put(qper(t1, kNt), kNt);
        B.put(qlin(span, 0.0, 2.0 * kPi, kNt), kNt);
        w[0] = (uint32_t)B.lo;
        w[1] = (uint32_t)(B.lo >> 32);
        w[2] = (uint32_t)B.hi;
        w[3] = (uint32_t)(B.hi >> 32);
    } else {
        const unsigned long long slot = atomicAdd(A.fb_n, 1ull);
        if ((int64_t)slot < A.fb_cap)
            for (int f = 0; f < 11; ++f) A.fb[11 * (int64_t)slot + f] = A.arc[f * A.ld + j];
        w[0] = (uint32_t)slot;
        w[1] = (uint32_t)(slot >> 32);
        w[2] = 0;
        w[3] = 0;
    }
}

__global__ void k_arc_decode(CodecArgs A)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= A.E) return;
    const uint32_t *w = A.codes + 4 * j;
    float *o = A.out;
    const int64_t L = A.ld_out;
    if ((A.mask[j >> 5] >> (j & 31)) & 1u) {
        const int64_t slot = (int64_t)((unsigned long long)w[0] | ((unsigned long long)w[1] << 32));
        for (int f = 0; f < 11; ++f) o[f * L + j] = slot < A.fb_cap ? A.fb[11 * slot + f] : 0.f;
        return;
    }
    Bits B;
    B.lo = (unsigned long long)w[0] | ((unsigned long long)w[1] << 32);
    B.hi = (unsigned long long)w[2] | ((unsigned long long)w[3] << 32);
    const uint32_t qra = B.get(kNr), qtha = B.get(kMth), qpha = B.get(kMph), qrb = B.get(kNr);
    const uint32_t qrc = B.get(kNr), qthc = B.get(kMth), qphc = B.get(kMph), qt1 = B.get(kNt), qsp = B.get(kNt);
    const D3 ah = unit_at(qtha, qpha);
    const D3 a = scl(ah, A.rmin + (double)qra * A.step_a), c = scl(unit_at(qthc, qphc), (double)qrc * A.step_c);
    const D3 d = ref_dir(A, j);
    const D3 x = crs(ah, d);
    const double xn = nrm(x);
    const D3 b = scl(dvd(x, xn > 0.0 ? xn : 1.0), 0.1 * A.rmin + (double)qrb * A.step_b);
    const double t1 = dper(qt1, kNt);
    const double t2 = t1 + (double)qsp * lin_step(0.0, 2.0 * kPi, kNt);
    const double v[11] = {c.x, c.y, c.z, a.x, a.y, a.z, b.x, b.y, b.z, t1, t2};
    for (int f = 0; f < 11; ++f) o[f * L + j] = (float)v[f];
}

}  // namespace

hipError_t launch_arc_codec(const Inputs &in, const Work &w, bool encode, const float *arc, const uint32_t *u32,
                            int64_t E, int64_t ld, double rmin, double rmax, uint32_t *codes, uint32_t *mask,
                            float *fb, int64_t fb_cap, unsigned long long *fb_n, float *out, int64_t ld_out,
                            hipStream_t st)
{
    if (E == 0) return hipSuccess;
    CodecArgs A;
    A.in = in;
    A.w = w;
    A.arc = arc;
    A.u32 = u32;
    A.E = E;
    A.ld = ld;
    A.rmin = rmin;
    A.rmax = rmax;
    A.step_a = lin_step(rmin, 4.0 * rmax, kNr);
    A.step_b = lin_step(0.1 * rmin, rmax, kNr);
    A.step_c = lin_step(0.0, rmax, kNr);
    A.codes = codes;
    A.mask = mask;
    A.fb = fb;
    A.fb_cap = fb_cap;
    A.fb_n = fb_n;
    A.out = out;
    A.ld_out = ld_out;
    const unsigned g = (unsigned)((E + 255) / 256);
    if (encode) k_arc_encode<<<g, 256, 0, st>>>(A);
    else k_arc_decode<<<g, 256, 0, st>>>(A);
    return hipGetLastError();
}

}  // namespace lm
