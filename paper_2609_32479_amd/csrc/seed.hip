// Analytic three-hit seed and per-hit seed residual features on gfx950, in
// fp64 (Sec. Method, "Analytic seed": the seed perigee is computed in double
// precision because the transport to the beam line cancels at high momentum).
//
// A lane pair per track for the seed.  The circle through the track's first three
// hits (transverse plane) comes from the intersection of two perpendicular
// bisectors, written relative to the first hit; this is the same circle the
// paper's conformal map gives.  Its radius gives pT = kappa B R, its turning
// direction the charge, its closest approach to the z axis the perigee
// (d0, phi); the transverse arc lengths of the first and third hit from the
// perigee give cot(theta) and z0.  Then (one lane per hit row, so that the
// hit reads and feature writes are coalesced) every hit of the track gets its
// residual to the seed helix in the curvilinear frame there: the transverse
// component reduces to the signed radial distance from the circle, the other
// to sin(theta) times the z residual; both are asinh-compressed (argument in
// mm), with the helix path length from the perigee as third feature.
//
// What bounds it: vector instructions, then memory.  With the library's atan2,
// sqrt and asinhf a row took about 440 vector instructions (340 of them the two
// asinhf) and the seed of 32 tracks 800 on half the lanes; 1 048 576 tracks (14.7 M
// hits, 0.40 GB in and out) took 226 us, 1.8 TB/s.  Now a row takes about 160
// (arc_length and asinh32 below) and lanes i and i + 32 of a wave share track i's
// seed: each takes the arc of one hit and one of the two angles: 150 us, 2.7 TB/s,
// still bound by the vector unit (one or two waves a workgroup, or five per SIMD
// instead of four, change nothing).  Of the 1 960 vector instructions of a wave (a
// counter's figure, 14 hits a track) the 7 to 7.5 chunks of 64 rows take 1 120 to 1 200,
// a third of these at quarter rate (fp64 reciprocals, roots, conversions, scalings);
// the other 40 % are the seed itself (the library's atan2, three of its square roots,
// six fp64 divisions) and the rows' way to their tracks.
//
// Reads: a wave's rows are one contiguous range.  When it spans at most
// kSeedRows rows (and the wave's offsets are in order), the wave reads it once,
// coalesced, into LDS (a lane writes the three floats of its row 12 bytes on from
// its neighbour's: no bank conflicts), takes each track's first three hits from
// there and computes the features from there.  Otherwise each track lane
// reads its first three hits itself and the row pass reads the range again.
//
// Conventions: the perigee point is d0 (-sin phi, cos phi), phi the direction
// of motion there; k = +1 for counter-clockwise motion seen from +z and the
// charge is -k (field along +z).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "trackfit.h"

namespace {

constexpr double kKappa = 0.299792458;  // pT [GeV] = kappa * B [T] * R [m], unit charge
constexpr int kSeedWaves = 4;           // waves per workgroup
constexpr int kSeedBlock = 64 * kSeedWaves;
constexpr int kSeedTracks = 32;         // tracks per wave (lanes i and i + 32: track i)
constexpr int kSeedChunks = 8;          // 64-row chunks that a wave keeps in LDS
constexpr int kSeedRows = 64 * kSeedChunks;

// sqrt(x) for normal x > 0, to about an ulp: the hardware's 23-bit reciprocal
// square root and two Newton steps (the last on the exact residual).
__device__ __forceinline__ double sqrt64(double x) {
    const double r = __builtin_amdgcn_rsq(x), h = 0.5 * r;
    double y = x * r;
    y = fma(fma(-y, y, x), h, y);
    return fma(fma(-y, y, x), h, y);
}
// a / b for normal b well inside the range, to about an ulp, likewise.
__device__ __forceinline__ double div64(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    r = fma(fma(-b, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// asinh rounded once to fp32.  |x| < 1/2: x + x^3 Q(x^2), Q the interpolant at six
// Chebyshev nodes of x^2 in [0, 1/4] (1.6e-9 relative).  Above: log(y),
// y = |x| + sqrt(x^2 + 1) = 2^k m with k the rounded hardware log2, and
// log m = 2 u + u^3 R(u^2), u = (m - 1) / (m + 1), R the interpolant at four nodes
// (2e-11); root and quotient to 46 bits.  In fp64, whose fused multiply-adds run at
// the fp32 rate here: an fp32 version with the hardware log2 was as fast but
// up to twice as far off (rms 0.56 to 0.79 ulp against 0.29 to 0.41 of the
// library's asinhf on the rounded argument; this one stays at 0.29, the rounding
// of the result).
__device__ __forceinline__ float asinh32(double x) {
    const bool over = fabs(x) >= 3.4028235677973366e38;  // rounds to no fp32 value: infinite
    const double t = over ? 1.0 : fabs(x), z = t * t;
    double p = 0.00993445135043325;
    p = fma(p, z, -0.02052563251636141);
    p = fma(p, z, 0.030155951374083587);
    p = fma(p, z, -0.04463000403740606);
    p = fma(p, z, 0.07499972845438123);
    p = fma(p, z, -0.1666666657260924);
    const double small = fma(t * z, p, t);
    const double s2 = z + 1.0, r = __builtin_amdgcn_rsq(s2), s0 = s2 * r;
    const double y = t + fma(fma(-s0, s0, s2), 0.5 * r, s0);
    // (the hardware log2 takes an fp32 argument: 2^-64 keeps it in range)
    const float k = rintf(__builtin_amdgcn_logf((float)(y * 0x1p-64)) + 64.0f);
    const double m = __builtin_amdgcn_ldexp(y, -(int)k);
    const double d = m + 1.0;
    double q = __builtin_amdgcn_rcp(d);
    q = fma(fma(-d, q, 1.0), q, q);
    const double u = (m - 1.0) * q, v = u * u;
    double w = 0.11666380903870686;
    w = fma(w, v, 0.14275368202679092);
    w = fma(w, v, 0.20000061292292048);
    w = fma(w, v, 0.3333333327679277);
    const double large = fma((double)k, 0.6931471805599453, 2.0 * fma(u * v, w, u));
    const float a = over ? __builtin_inff() : (float)(t < 0.5 ? small : large);
    return copysignf(a, (float)x);
}

// A track's circle: centre, distance of the centre from the axis, sense k, k
// times the radius, z0, cot(theta), sin(theta) and its inverse.
enum { CX, CY, CD, CK, CKR, CZ0, CCOT, CST, CIST, CN };

// Transverse arc from the perigee (direction -C from the centre C, |C| = D) to the
// point at w from the centre, positive along the motion, and rho = |w|.  With
// cr and dt the cross product and minus the dot product of C and w, the turning
// angle a = atan2(cr, dt) is 2 atan(t), t = cr / (D rho + dt).  For |a| <= pi / 4 (any
// outgoing track of a few GeV) |t| <= tan(pi / 8), and atan(t) = t + t^3 P(t^2) with
// P the interpolant at 11 Chebyshev nodes (7e-18 relative); a lane beyond
// that, or with operands too small or large for the bare Newton steps, takes the
// library's functions.  A lane's result does not depend on the others.
__device__ __forceinline__ double arc_length(double wx, double wy, double cx, double cy, double D, double kR,
                                             double &rho) {
    const double w2 = fma(wx, wx, wy * wy);
    const double cr = fma(cy, wx, -(cx * wy)), dt = -fma(cx, wx, cy * wy);
    rho = sqrt64(w2);
    const double den = fma(D, rho, dt);
    const double t = div64(cr, den), z = t * t;
    double p = -0.019169381698603605;
    p = fma(p, z, 0.03922552313874487);
    p = fma(p, z, -0.05085237122079787);
    p = fma(p, z, 0.05858108230387606);
    p = fma(p, z, -0.066645067575513);
    p = fma(p, z, 0.07692182857348952);
    p = fma(p, z, -0.09090904563742808);
    p = fma(p, z, 0.11111111014901609);
    p = fma(p, z, -0.14285714284662115);
    p = fma(p, z, 0.199999999999955);
    p = fma(p, z, -0.3333333333333333);
    double s = 2.0 * kR * fma(t * z, p, t);
    const bool ok = fabs(cr) <= 0.4142 * den && w2 > 1e-200 && w2 < 1e200 && den > 1e-200 && den < 1e200;
    if (__any(!ok)) {
        const double rho_l = sqrt(w2), s_l = kR * atan2(cr, dt);
        rho = ok ? rho : rho_l;
        s = ok ? s : s_l;
    }
    return s;
}

// Seed of the track of lanes i and i + 32 (half: which of the two) from its first
// three hits h = (x1, y1, z1, x2, y2, z2, x3, y3, z3): the circle for the features
// (both lanes) and the perigee parameters to sd[0..4].  False when the three hits
// are collinear in the transverse plane.  Both lanes are active or neither.
__device__ __forceinline__ bool seed_from_hits(const double *h, int half, double b_tesla, double *sd, double (&c)[CN]) {
    const double x1 = h[0], y1 = h[1], z1 = h[2];
    const double bx = h[3] - x1, by = h[4] - y1;
    const double qx = h[6] - x1, qy = h[7] - y1, z3 = h[8];
    // centre relative to hit 1: equidistant from hits 1, 2 and 3
    const double det = 2.0 * (bx * qy - by * qx);
    if (det == 0.0) return false;
    const double b2 = bx * bx + by * by, q2 = qx * qx + qy * qy;
    const double ux = (qy * b2 - by * q2) / det, uy = (bx * q2 - qx * b2) / det;
    const double cx = x1 + ux, cy = y1 + uy;
    const double R = sqrt(ux * ux + uy * uy);
    const double k = det > 0.0 ? 1.0 : -1.0;
    const double D = sqrt(cx * cx + cy * cy);
    // the arcs of the first and third hit, one per lane
    double rho;
    const double own = arc_length((half ? x1 + qx : x1) - cx, (half ? y1 + qy : y1) - cy, cx, cy, D, k * R, rho);
    const double other = __shfl_xor(own, 32);
    const double ds = half ? own - other : other - own, dz = z3 - z1;
    const double s1 = half ? other : own;
    // theta in one lane, phi in the other
    const double ang = atan2(half ? -k * cx : ds, half ? k * cy : dz);
    const double hyp = sqrt(ds * ds + dz * dz);
    c[CX] = cx;
    c[CY] = cy;
    c[CD] = D;
    c[CK] = k;
    c[CKR] = k * R;
    c[CCOT] = dz / ds;
    c[CZ0] = z1 - s1 * c[CCOT];
    c[CST] = hyp > 0.0 ? ds / hyp : 0.0;
    c[CIST] = hyp / ds;
    if (half) {
        sd[2] = ang;
    } else {
        sd[0] = k * (D - R);
        sd[1] = c[CZ0];
        sd[3] = ang;
        sd[4] = -k * c[CST] / (kKappa * b_tesla * R * 1e-3);
    }
    return true;
}

// Residual features of one hit against a track's circle and the line
// z = z0 + s cot(theta) along its transverse arc s from the perigee.  The
// residuals need fp64 (they are differences of values a thousand times
// larger); the features are stored as float32.  cp: the circle's first entry, cs: entries to the next.
__device__ __forceinline__ void hit_features(float px, float py, float pz, const double *cp, int cs, float *f) {
    const double cx = cp[CX * cs], cy = cp[CY * cs];
    double rho;
    const double s = arc_length((double)px - cx, (double)py - cy, cx, cy, cp[CD * cs], cp[CKR * cs], rho);
    const double du = fma(-cp[CK * cs], rho, cp[CKR * cs]);
    const double dv = cp[CST * cs] * ((double)pz - fma(s, cp[CCOT * cs], cp[CZ0 * cs]));
    f[0] = asinh32(du);
    f[1] = asinh32(dv);
    f[2] = (float)(s * cp[CIST * cs]);  // the path length s / sin(theta)
}

// One wave per kSeedTracks consecutive tracks: lanes i and i + 32 seed track
// t0 + i, then the wave walks the hit rows of its tracks one row per lane
// (coalesced).  (32 tracks, about 450 rows at 14 hits a track, take 8.6 KB of LDS:
// four waves per SIMD.)
__global__ __launch_bounds__(kSeedBlock, 4) void tf_seed_kernel(const float *__restrict__ hits, long long n_hits,
                                                                 const int *__restrict__ offsets, int n_tracks,
                                                                 double b_tesla, double *__restrict__ seeds,
                                                                 float *__restrict__ features, int fstride,
                                                                 int *__restrict__ flags) {
    __shared__ float rows[kSeedWaves][kSeedRows * 3];       // the wave's hit rows
    __shared__ double circ[kSeedWaves][CN][kSeedTracks];    // circle entries per track
    __shared__ int wbits[kSeedWaves][kSeedTracks];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int half = lane >> 5, tl = lane & 31;
    const int t0 = (blockIdx.x * kSeedWaves + wv) * kSeedTracks;
    if (t0 >= n_tracks) return;  // the whole wave
    const int i = t0 + tl;
    const bool active = i < n_tracks;
    const double nan = __builtin_nan("");
    const int o0 = offsets[0], oN = offsets[n_tracks];
    const int o = active ? offsets[i] : oN, e = active ? offsets[i + 1] : oN;
    int bits = 0;
    // rows must lie in [0, n_hits) for the hits and in [offsets[0],
    // offsets[n_tracks]) for the features
    if (o < 0 || e < o || (long long)e > n_hits || o < o0 || e > oN)
        bits = TF_SEED_BAD_OFFSETS;
    else if (active && e - o < 3)
        bits = TF_SEED_TOO_SHORT;
    // the wave's rows: [lo, hi) when its offsets are in order
    const bool wave_bad = __ballot(bits == TF_SEED_BAD_OFFSETS) != 0;
    const int lo = __builtin_amdgcn_readlane(o, 0), hi = __builtin_amdgcn_readlane(e, kSeedTracks - 1);
    const int nch = wave_bad ? 0 : (hi - lo + 63) >> 6;
    const bool staged = features && !wave_bad && nch <= kSeedChunks;
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    double h[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (staged) {
        // one coalesced read of the rows, all of it in flight (lanes past the last
        // row read the last row again); then the first three hits of this lane's track
        float r[kSeedChunks][3];
#pragma unroll
        for (int c = 0; c < kSeedChunks; ++c)
            if (c < nch) {
                const float *p = hits + (size_t)min(lo + 64 * c + lane, hi - 1) * 3;
#pragma unroll
                for (int u = 0; u < 3; ++u) r[c][u] = p[u];
            }
#pragma unroll
        for (int c = 0; c < kSeedChunks; ++c)
            if (c < nch) {
#pragma unroll
                for (int u = 0; u < 3; ++u) rows[wv][(64 * c + lane) * 3 + u] = r[c][u];
            }
        wave_sync();
        if (active && !bits) {
            const float *p = rows[wv] + (o - lo) * 3;
#pragma unroll
            for (int u = 0; u < 9; ++u) h[u] = p[u];
        }
    } else if (active && !bits) {
        const float *p = hits + (size_t)o * 3;
#pragma unroll
        for (int u = 0; u < 9; ++u) h[u] = p[u];
    }
    double sc[CN];
#pragma unroll
    for (int u = 0; u < CN; ++u) sc[u] = 0.0;
    if (active && !bits) {
        if (!seed_from_hits(h, half, b_tesla, seeds + (size_t)i * 5, sc)) bits = TF_SEED_NO_CIRCLE;
    }
    if (active && bits && half == 0) {
        double *sd = seeds + (size_t)i * 5;
        for (int j = 0; j < 5; ++j) sd[j] = nan;
        if (flags) atomicOr(flags, bits);
    }
    if (!features) return;
    if (half == 0) {
#pragma unroll
        for (int u = 0; u < CN; ++u) circ[wv][u][tl] = sc[u];
        wbits[wv][tl] = bits;
    }
    wave_sync();
    if (wave_bad) {
        // offsets out of order somewhere in this wave: every good track walks
        // its own rows
        if (half || bits == TF_SEED_BAD_OFFSETS) return;
        for (int hr = o; hr < e; ++hr) {
            float *f = features + (size_t)(hr - o0) * fstride;
            if (bits) {
                f[0] = f[1] = f[2] = (float)nan;
            } else {
                const float *p = hits + (size_t)hr * 3;
                hit_features(p[0], p[1], p[2], &circ[wv][0][tl], kSeedTracks, f);
            }
        }
        return;
    }
    // Rows [lo, hi), 64 at a time.  The track of each lane's row: the tracks that
    // start in the chunk, in order (their starts read from the track lanes), each
    // taking the rows from its start on; a track without hits takes none, as the
    // next one starts at the same row.
    int a = 0, tn = 0;  // the track of the row before the chunk; the next track to start
#pragma unroll 1
    for (int c = 0; c < nch; ++c) {
        const int r = 64 * c + lane;           // row less lo
        a = __builtin_amdgcn_readlane(a, 63);  // the track of the row before the chunk
        for (; tn < kSeedTracks; ++tn) {
            const int st = __builtin_amdgcn_readlane(o, tn) - lo;
            if (st >= 64 * c + 64) break;
            a = r >= st ? tn : a;
        }
        if (r < hi - lo) {
            float *f = features + (size_t)(lo - o0 + r) * fstride;
            if (wbits[wv][a]) {
                f[0] = f[1] = f[2] = (float)nan;
            } else {
                float px, py, pz;
                if (staged) {
                    const float *p = rows[wv] + r * 3;
                    px = p[0], py = p[1], pz = p[2];
                } else {
                    const float *p = hits + (size_t)(lo + r) * 3;
                    px = p[0], py = p[1], pz = p[2];
                }
                float g[3];
                hit_features(px, py, pz, &circ[wv][0][a], kSeedTracks, g);
                f[0] = g[0], f[1] = g[1], f[2] = g[2];
            }
        }
    }
}

}  // namespace

extern "C" tf_status tf_seed_tracks(const float *hits, int64_t n_hits, const int32_t *offsets, int32_t n_tracks,
                                    double b_tesla, double *seeds, float *features, int32_t feature_stride,
                                    int32_t *flags, hipStream_t stream) {
    if (n_tracks < 0 || n_hits < 0 || !(b_tesla > 0.0)) return TF_EINVAL;
    if (feature_stride == 0) feature_stride = 3;
    if (feature_stride < 3) return TF_EINVAL;
    if (n_tracks == 0) return TF_OK;
    if (!offsets || !seeds || (!hits && n_hits > 0)) return TF_EINVAL;
    const int per_block = kSeedWaves * kSeedTracks;
    const int blocks = (n_tracks + per_block - 1) / per_block;  // one wave per kSeedTracks tracks
    hipLaunchKernelGGL(tf_seed_kernel, dim3(blocks), dim3(kSeedBlock), 0, stream, hits, (long long)n_hits, offsets,
                       (int)n_tracks, b_tesla, seeds, features, (int)feature_stride, flags);
    return hipGetLastError() == hipSuccess ? TF_OK : TF_EHIP;
}
