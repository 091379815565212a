// Hybrid rDDMC walk on 1D grids (slab cells along z, or spherical shells): DDMC steps in
// thick states (Sec. 2.3, eqs. 15-16; the Doppler re-binning of Sec. 2.5) and continuous
// Monte Carlo in thin ones (the hybrid section: interface leaks, conversions both ways, the
// eq. 39 acceptance; the MC step with the Voigt opacity of eq. 12 and the redistribution of
// eq. 41, optionally with core-skipping).
//
// One lane carries one packet.  MC packets have a full 3D position and direction; the grid
// enters through its boundaries (planes z = z_f, or spheres r = r_f), their outward normals
// (+-z, or +-r^) and the bulk velocity (u along +z in a slab cell; u r^ in a shell, so its
// direction changes with position).  Per step:
//   DDMC state: the 16-byte hot record {ln2/K, D_hi, S_hi, flags} as on 3D grids; a spatial
//     leak picks face 0 or 1 from the state's 31-bit split; the flags say whether bin j-1 / j+1
//     is thin and whether a face leads into a thin state or vacuum.  Conversions: into a thin
//     bin, a uniform point of the cell (uniform in volume), isotropic, x uniform in the bin;
//     through an interface face, a uniform point of the face, mu uniform in (0, 1] about its
//     outward normal, x uniform in the bin moved to the neighbour's frame,
//     x' = (x + n.u) sqrt(T/T') - n.u' (both velocities at that point), or escape with the lab
//     frequency x + n.u through vacuum; a re-binning into a thin state, MC in the new cell at
//     a uniform point, isotropic, with the shifted x.
//   MC state: distance to the cell boundary along n (planes, or the quadratic for spheres,
//     in FP64) against an exponential optical depth at opacity k0 H(a, x); the comoving x is
//     that of the packet's current point (in a shell it changes by n.(u(p0) - u(p1)) over a
//     flight, the lab frequency being constant), and a flight's opacity is that of its
//     starting x.  Scattering and wall crossings as on 3D grids, with the neighbour's width
//     across the interface in eq. 39.
// Dust (Sec. 2.4): the tables already hold the total scattering coefficient; a DDMC step's
// event draw may land in the absorption band of its thresholds, and an MC flight meets Lya,
// dust scattering (isotropic, coherent in the comoving frame) and dust absorption in
// proportion to their opacities; absorbed packets are counted after their residence.
// Time-dependent estimators (eq. 17): every stretch of a packet's clock spent in a state adds
// its overlap with each census interval to that state's residence time (2^-24 units) and
// counts the packet in that state at every census time it spans.  Packets start at t = 0 or
// uniformly inside their source's emission window.
// Frequency groups (Sec. 5.3): in a cloud built with them, thin states carry a bin instead of
// a continuous frequency; flights meet the bin-averaged opacity and scatterings draw the
// outgoing bin from the eq. 42 alias table of the packet's bin.
// Escapes add face row (slab: face; sphere: one row), lab bin and time to the int64 tallies.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mc_dev.h"
#include "philox.h"
#include "rddmc_internal.h"
#include "wave_dev.h"

namespace rddmc {

namespace {

using namespace mc;

constexpr uint32_t kDom1DH = 0x60000000u;       // counter domain of the 1D hybrid walk's streams

struct Pk1 {
    int cl;
    int cell;
    int j;
    bool mc, active;
    bool left_inner;   // the current flight started on the cell's inner sphere, moving outward
    float3 pos, n;
    float x;
    double t;
    double lw;         // -ln(weight): optical depth of dust absorption so far (continuous weights)
    uint32_t cn;       // next way of the packet's census path cache to evict (round robin)
    int ci;            // first census time at or after the packet's clock (its clock only grows)
    double tn;         // that census time (-inf until the first full update)
    uint64_t steps;
    uint32_t mcs, tomc, toddmc, refl;
    Rng r;
};

__device__ __forceinline__ float dot3f(float3 a, float3 b) { return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z)); }

// unit vector along p (+z at the origin)
__device__ __forceinline__ float3 radial(float3 p)
{
    const float r2 = dot3f(p, p);
    if (!(r2 > 0.0f)) return make_float3(0.f, 0.f, 1.f);
    const float ir = rsqrtf(r2);
    return make_float3(p.x * ir, p.y * ir, p.z * ir);
}

// outward normal of a cell at face f (0 lower / inner, 1 upper / outer) at point p
template <bool SPH>
__device__ __forceinline__ float3 face_normal(int f, float3 p)
{
    const float s = f ? 1.0f : -1.0f;
    if (!SPH) return make_float3(0.f, 0.f, s);
    const float3 e = radial(p);
    return make_float3(s * e.x, s * e.y, s * e.z);
}

// n . u of a cell whose bulk speed (in its thermal units) is u, at point p
template <bool SPH>
__device__ __forceinline__ float n_dot_u(float u, float3 p, float3 n)
{
    if (!SPH) return n.z * u;
    return u * dot3f(n, radial(p));
}

// direction with cosine mu ~ U(0, 1] about the unit vector N, uniform azimuth
__device__ __forceinline__ float3 hemi_about(Rng &r, const McArgs &a, float3 N)
{
    const float mu = uf(draw(r, a));
    const float ph = kTwoPi * uf(draw(r, a));
    const float s = sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
    float sn, cs;
    sincosf(ph, &sn, &cs);
    float3 t1 = fabsf(N.z) < 0.9f ? make_float3(-N.y, N.x, 0.f) : make_float3(0.f, -N.z, N.y);
    const float il = rsqrtf(dot3f(t1, t1));
    t1 = make_float3(t1.x * il, t1.y * il, t1.z * il);
    const float3 t2 = make_float3(N.y * t1.z - N.z * t1.y, N.z * t1.x - N.x * t1.z, N.x * t1.y - N.y * t1.x);
    const float c1 = s * cs, c2 = s * sn;
    return make_float3(fmaf(mu, N.x, fmaf(c1, t1.x, c2 * t2.x)), fmaf(mu, N.y, fmaf(c1, t1.y, c2 * t2.y)),
                       fmaf(mu, N.z, fmaf(c1, t1.z, c2 * t2.z)));
}

// uniform point of face f of cell `cell`
template <bool SPH>
__device__ __forceinline__ float3 face_point(const double *fz, int cell, int f, Rng &r, const McArgs &a)
{
    const float rf = (float)fz[cell + f];
    if (!SPH) return make_float3(0.f, 0.f, rf);
    const float3 w = iso_dir(r, a);
    return make_float3(rf * w.x, rf * w.y, rf * w.z);
}

// uniform point of cell `cell` (uniform in volume)
template <bool SPH>
__device__ __forceinline__ float3 cell_point(const double *fz, int cell, Rng &r, const McArgs &a)
{
    const double lo = fz[cell], hi = fz[cell + 1];
    const double u = (double)uf(draw(r, a));
    if (!SPH) return make_float3(0.f, 0.f, (float)(lo + (hi - lo) * u));
    const float rr = (float)cbrt(lo * lo * lo + u * (hi * hi * hi - lo * lo * lo));
    const float3 w = iso_dir(r, a);
    return make_float3(rr * w.x, rr * w.y, rr * w.z);
}

// distance along n from p to the boundary of a cell with faces lo and hi, and the face it reaches.  A flight
// that starts on the inner sphere moving outward cannot meet that sphere again (a line leaves a
// ball once); `left_inner` says so, where the sign of p . n cannot for a grazing flight.
template <bool SPH>
__device__ __forceinline__ float wall_distance(double lo, double hi, float3 p, float3 n, bool left_inner, int &face)
{
    if (!SPH) {   // one division for either direction
        face = n.z < 0.0f ? 0 : 1;
        const float d = fmaxf(0.0f, (float)(((face ? hi : lo) - (double)p.z) / (double)n.z));
        return n.z == 0.0f ? INFINITY : d;
    }
    const double px = p.x, py = p.y, pz = p.z;
    const double b = px * n.x + py * n.y + pz * n.z;
    // the packet is inside its shell: a point put on a face in float can sit an ulp outside,
    // which would turn the far root into a zero-length crossing back and forth
    const double r = fmin(fmax(sqrt(px * px + py * py + pz * pz), lo), hi);
    double s = -b + sqrt(fmax(0.0, b * b + (hi - r) * (hi + r)));
    face = 1;
    if (lo > 0.0 && b < 0.0 && !left_inner) {
        const double disc = b * b + (lo - r) * (lo + r);
        if (disc > 0.0) {
            const double s_in = fmax(0.0, -b - sqrt(disc));
            if (s_in < s) {
                s = s_in;
                face = 0;
            }
        }
    }
    return (float)fmax(0.0, s);
}

__device__ __forceinline__ int time_bin1(double t)
{
    if (!(t >= 1e-3)) return 0;
    const double u = (log10(t) + 3.0) * (RDDMC_TIME_BINS / 9.0);
    if (u >= (double)RDDMC_TIME_BINS) return RDDMC_TIME_BINS + 1;
    return 1 + (int)u;
}

__device__ __forceinline__ int step_bin1(uint64_t n) { return n <= 1 ? 0 : 63 - __clzll((long long)n); }

// Integral over [a, b) of the weight exp(-(lw0 + ka (t - t0))) of a packet that had log-weight
// lw0 at t0 (c = 1): w(a) (1 - exp(-ka (b - a))) / ka, the residence times the path correction.
__device__ __forceinline__ double weight_integral(double a, double b, double t0, double lw0, double ka)
{
    const double wa = exp(-(lw0 + ka * (a - t0)));
    return ka > 0.0 ? wa * (-expm1(-ka * (b - a)) / ka) : wa * (b - a);
}

constexpr uint64_t kNoKey = ~0ull;
constexpr int kWays = 8;         // ways of a lane's census path cache
constexpr int kBlockMax = 256;   // lanes per block of the walk

// The 'path' estimator's sums go through an eight-way cache per lane, held in LDS (way-major,
// so a wave's accesses to one way are 64 consecutive words): a walk returns to the states it
// has just left (a frequency move and back), so most of its per-step residences add to a held
// sum instead of a device atomic.  Integer sums make the tallies identical to adding every
// residence at once, whatever the evictions.  Each lane touches only its own slots.
__shared__ uint64_t s_path_key[kWays * kBlockMax];
__shared__ uint64_t s_path_sum[kWays * kBlockMax];

__device__ __forceinline__ void path_init()
{
#pragma unroll
    for (int q = 0; q < kWays; ++q) {
        s_path_key[q * kBlockMax + threadIdx.x] = kNoKey;
        s_path_sum[q * kBlockMax + threadIdx.x] = 0ull;
    }
}

__device__ __forceinline__ void path_add(Pk1 &p, unsigned long long *__restrict__ wpath, uint64_t key, uint64_t v)
{
    const int l = threadIdx.x;
#pragma unroll
    for (int q = 0; q < kWays; ++q)
        if (s_path_key[q * kBlockMax + l] == key) {
            s_path_sum[q * kBlockMax + l] += v;
            return;
        }
    const int e = (int)p.cn * kBlockMax + l;
    const uint64_t k0 = s_path_key[e], v0 = s_path_sum[e];
    if (k0 != kNoKey && v0) atomicAdd(&wpath[k0], (unsigned long long)v0);
    s_path_key[e] = key;
    s_path_sum[e] = v;
    p.cn = (p.cn + 1) & (kWays - 1);
}

__device__ __forceinline__ void path_flush(Pk1 &p, unsigned long long *__restrict__ wpath)
{
    const int l = threadIdx.x;
#pragma unroll
    for (int q = 0; q < kWays; ++q) {
        const uint64_t k0 = s_path_key[q * kBlockMax + l], v0 = s_path_sum[q * kBlockMax + l];
        if (k0 != kNoKey && v0) atomicAdd(&wpath[k0], (unsigned long long)v0);
        s_path_key[q * kBlockMax + l] = kNoKey;
        s_path_sum[q * kBlockMax + l] = 0ull;
    }
    p.cn = 0;
}

// The packet stays in state s over [t0, t1): census counts and residence times.  With
// continuous dust weights (log-weight lw0 at t0, decay rate ka) the counts are the weights at
// the census times and the residences their integrals (2^-24 units both).
template <bool WGT>
__device__ __forceinline__ void census_add(Pk1 &p, const DevCloud &c, const uint8_t *__restrict__ tb,
                                           unsigned long long *__restrict__ tally, int64_t s, double t0, double t1,
                                           double lw0, double ka)
{
    const int n = c.n_census;
    if (p.ci > n) return;   // past the last census time: nothing to count
    unsigned long long *w = tally + c.tally_off;
    const uint64_t ns = c.n_states;
    if (t1 <= p.tn) {   // no census time in [t0, t1): the whole residence in interval ci - 1
        if (p.ci > 0 && t1 > t0) {
            const double r = (WGT && c.dust_weight) ? weight_integral(t0, t1, t0, lw0, ka) : t1 - t0;
            path_add(p, w + c.census_path_off, (uint64_t)(p.ci - 1) * ns + s, (uint64_t)rint(r * kPathFix));
        }
        return;
    }
    const double *ct = reinterpret_cast<const double *>(tb + c.off_census);
    int lo = p.ci;   // first census time >= t0: the packet's clock never goes back
    while (lo <= n && ct[lo] < t0) ++lo;
    p.ci = lo;
    p.tn = lo <= n ? ct[lo] : 0.0;
    for (int e = lo; e <= n && ct[e] < t1; ++e)
        atomicAdd(&w[c.census_bin_off + (uint64_t)e * ns + s],
                  (WGT && c.dust_weight) ? (unsigned long long)rint(exp(-(lw0 + ka * (ct[e] - t0))) * kPathFix) : 1ull);
    for (int i = lo > 0 ? lo - 1 : 0; i < n && ct[i] < t1; ++i) {
        const double a0 = fmax(t0, ct[i]), b0 = fmin(t1, ct[i + 1]);
        if (b0 > a0) {
            const double r = (WGT && c.dust_weight) ? weight_integral(a0, b0, t0, lw0, ka) : b0 - a0;
            path_add(p, w + c.census_path_off, (uint64_t)i * ns + s, (uint64_t)rint(r * kPathFix));
        }
    }
}

// Eq. 18: a leak of a step that stayed over [t0, t1) adds v times its residence in each census
// interval to `cell` (signed fixed point, 2^-24); with continuous dust weights, v times the
// weight's integral over the residence (the path correction).
// lo is the first census index whose time is >= t0 (the packet's index after census_add of
// the same residence).
template <bool WGT>
__device__ __forceinline__ void accel_add(const DevCloud &c, const uint8_t *__restrict__ tb, unsigned long long *__restrict__ tally,
                          int cell, double t0, double t1, double v, double lw0, double ka, int lo)
{
    const double *ct = reinterpret_cast<const double *>(tb + c.off_census);
    const int n = c.n_census;
    unsigned long long *w = tally + c.tally_off + c.census_accel_off;
    for (int i = lo > 0 ? lo - 1 : 0; i < n && ct[i] < t1; ++i) {
        const double a0 = fmax(t0, ct[i]), b0 = fmin(t1, ct[i + 1]);
        if (b0 > a0) {
            const double r = (WGT && c.dust_weight) ? weight_integral(a0, b0, t0, lw0, ka) : b0 - a0;
            atomicAdd(&w[(uint64_t)i * c.nc + cell], (unsigned long long)(long long)rint(v * r * kAccelFix));
        }
    }
}

// A weighted escape (continuous dust weights): weight and squared weight into slot q of the
// weighted spectra, w t and w t^2 into their 128-bit sums.
__device__ __forceinline__ void escape_weighted(const DevCloud &c, unsigned long long *w, uint64_t q, uint64_t nspec,
                                             double lw, double t)
{
    unsigned long long *ww = w + c.wspec_off;
    const double wt = exp(-lw);
    atomicAdd(&ww[4 + q], (unsigned long long)rint(wt * kWeightFix));
    atomicAdd(&ww[4 + nspec + q], (unsigned long long)rint(wt * wt * kWeightFix));
    const unsigned long long a1 = (unsigned long long)rint(wt * t * kWeightFix);
    if (atomicAdd(&ww[0], a1) + a1 < a1) atomicAdd(&ww[1], 1ull);
    const unsigned long long a2 = (unsigned long long)rint(wt * t * t * kTimeFix);
    if (atomicAdd(&ww[2], a2) + a2 < a2) atomicAdd(&ww[3], 1ull);
}

template <bool WGT, bool CEN>
__device__ __forceinline__ void finish1(Pk1 &p, const DevCloud &c, unsigned long long *__restrict__ tally, bool escaped, int row,
                        int slot, bool absorbed = false)
{
    unsigned long long *w = tally + c.tally_off;
    const uint64_t nspec = (uint64_t)c.n_rows * (c.nb + 2);
    if (absorbed) {
        atomicAdd(&w[TW_ABSORBED], 1ull);
    } else if (escaped) {
        atomicAdd(&w[TW_ESCAPED], 1ull);
        atomicAdd(&w[kTallyHeader + (uint64_t)row * (c.nb + 2) + slot], 1ull);
        atomicAdd(&w[TW_TSUM], (unsigned long long)rint(p.t * kTimeFix));
        const unsigned long long t2 = (unsigned long long)rint(p.t * p.t * kTimeFix);
        const unsigned long long old = atomicAdd(&w[TW_T2_LO], t2);
        if (old + t2 < old) atomicAdd(&w[TW_T2_HI], 1ull);
        atomicAdd(&w[kTallyHeader + nspec + time_bin1(p.t)], 1ull);
        if (WGT && c.dust_weight) escape_weighted(c, w, (uint64_t)row * (c.nb + 2) + slot, nspec, p.lw, p.t);
    } else {
        atomicAdd(&w[TW_CAPPED], 1ull);
    }
    if (CEN && c.n_census > 0) path_flush(p, w + c.census_path_off);
    atomicAdd(&w[kTallyHeader + nspec + RDDMC_TIME_BINS + 2 + step_bin1(p.steps)], 1ull);
    atomicAdd(&w[TW_STEPS], (unsigned long long)p.steps);
    atomicMax(&w[TW_STEPS_MAX], (unsigned long long)p.steps);
    if (p.mcs) atomicAdd(&w[TW_MC_STEPS], (unsigned long long)p.mcs);
    if (p.tomc) atomicAdd(&w[TW_TO_MC], (unsigned long long)p.tomc);
    if (p.toddmc) atomicAdd(&w[TW_TO_DDMC], (unsigned long long)p.toddmc);
    if (p.refl) atomicAdd(&w[TW_REFLECTED], (unsigned long long)p.refl);
    p.active = false;
}

// neighbour of `cell` through face f: -1 for vacuum (a sphere's r = 0 face has no leak)
__device__ __forceinline__ int neighbour1(const DevCloud &c, int cell, int f)
{
    if (f) return cell + 1 < c.nc ? cell + 1 : -1;
    return cell > 0 ? cell - 1 : -1;
}

// One DDMC step of a packet in a thick state.
template <bool SPH, bool WGT, bool CEN>
__device__ __forceinline__ void ddmc_step1(Pk1 &p, const DevCloud &c, const uint8_t *__restrict__ tb, const McArgs &a,
                           unsigned long long *__restrict__ tally)
{
    const int nb = c.nb;
    const int64_t s = (int64_t)p.cell * nb + p.j;
    const uint4 rec = reinterpret_cast<const uint4 *>(tb + c.off_hot)[s];
    const uint32_t tw = draw(p.r, a), ew = draw(p.r, a);
    const double dl = (double)ddmc_path(tw, __uint_as_float(rec.x));
    // continuous dust weights: the interaction distance dl carries optical depth k_a dl
    const double ka = (WGT && c.dust_weight) ? reinterpret_cast<const double *>(tb + c.off_dust)[2 * p.cell] : 0.0;
    const double lw0 = p.lw;
    if (CEN && c.n_census > 0) census_add<WGT>(p, c, tb, tally, s, p.t, p.t + dl, lw0, ka);
    const double t0 = p.t;
    p.t += dl;
    if (WGT && c.dust_weight) {
        p.lw = fma(ka, dl, p.lw);
        if (p.lw > kLogWMin) {   // negligible weight: eliminated
            finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
            return;
        }
    }
    int ev;
    bool have_lo = false;
    uint32_t lo_word = 0u;
    if (ew != rec.y && ew != rec.z) {
        ev = ew < rec.y ? 0 : (ew < rec.z ? 1 : 2);
    } else {   // the high words tie: compare the full u64
        const uint4 lw = reinterpret_cast<const uint4 *>(tb + c.off_lo_words)[s];
        lo_word = draw(p.r, a);
        have_lo = true;
        const uint64_t U = ((uint64_t)ew << 32) | lo_word;
        const uint64_t D = ((uint64_t)rec.y << 32) | lw.x;
        const uint64_t S = ((uint64_t)rec.z << 32) | lw.y;
        ev = U < D ? 0 : (U < S ? 1 : 2);
    }
    if (ev == 2 && c.dusty) {   // dust absorption band [A, 2^64) above the spatial leaks
        const uint4 lw = reinterpret_cast<const uint4 *>(tb + c.off_lo_words)[s];
        const uint64_t A = ((uint64_t)lw.w << 32) | lw.z;
        bool absorb;
        if (A == 0ull) {
            absorb = false;
        } else if (ew != lw.w) {
            absorb = ew > lw.w;
        } else {
            if (!have_lo) lo_word = draw(p.r, a);
            absorb = (((uint64_t)ew << 32) | lo_word) >= A;
        }
        if (absorb) {
            finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
            return;
        }
    }
    const double *fz = faces_of(c, tb, 0);
    if (ev < 2) {   // frequency leak (eq. 11)
        p.j += ev ? 1 : -1;
        if (rec.w & (ev ? kFlagUpThin : kFlagDnThin)) {   // into a thin bin: MC in this cell
            p.pos = cell_point<SPH>(fz, p.cell, p.r, a);
            p.n = iso_dir(p.r, a);
            p.left_inner = false;
            p.x = bin_x(c, tb, p.j, uf(draw(p.r, a)));
            p.mc = true;
            ++p.tomc;
        }
        return;
    }
    // spatial leak: face 0 or 1 from the state's split
    const uint32_t v = draw(p.r, a) >> 1;
    const int f = v >= reinterpret_cast<const uint32_t *>(tb + c.off_face_split)[s] ? 1 : 0;
    const double *kt = reinterpret_cast<const double *>(tb + c.off_k);
    const double dir = f ? 1.0 : -1.0;
    if (CEN && c.n_census > 0) accel_add<WGT>(c, tb, tally, p.cell, t0, p.t, dir * kt[s], lw0, ka, p.ci);   // outward leakage (eq. 18)
    const float xin = bin_x(c, tb, p.j, uf(draw(p.r, a)));
    const int nbc = neighbour1(c, p.cell, f);
    const float4 *mcell = reinterpret_cast<const float4 *>(tb + c.off_mcell);
    if (rec.w & (1u << (kFlagFaceShift + f))) {
        // interface leak into a thin state or vacuum: an MC packet leaving through face f
        p.pos = face_point<SPH>(fz, p.cell, f, p.r, a);
        p.n = hemi_about(p.r, a, face_normal<SPH>(f, p.pos));
        const float nu = n_dot_u<SPH>(mcell[2 * p.cell + 1].x, p.pos, p.n);
        if (nbc < 0) {
            const int slot = c.moving ? bin_of(c, tb, xin + nu) + 1 : p.j + 1;
            finish1<WGT, CEN>(p, c, tally, true, SPH ? 0 : f, slot);
            return;
        }
        const float4 m0 = mcell[2 * p.cell], m1 = mcell[2 * nbc];
        p.x = (xin + nu) * (m0.z / m1.z) - n_dot_u<SPH>(mcell[2 * nbc + 1].x, p.pos, p.n);
        p.cell = nbc;
        p.left_inner = f == 1;   // through the outer face of the old cell: the new one's inner
        p.mc = true;
        ++p.tomc;
        return;
    }
    // thick neighbour (vacuum faces always carry the interface bit); re-binned wherever the face's map
    // is not the identity, as the face flags and rates were built: in bin j itself the neighbour may
    // be thin, and its record empty
    float xs = xin;
    if (c.rebins) {
        const double *mp = reinterpret_cast<const double *>(tb + c.off_map) + 3 * (p.cell * 2 + f);
        const double rho = mp[0], sh = mp[1];
        if (rho != 1.0 || sh != 0.0) {
            xs = (float)fma(rho, (double)xin, sh);
            const int jn = bin_of(c, tb, xs);
            p.j = jn < 0 ? 0 : (jn > nb - 1 ? nb - 1 : jn);
        }
    }
    p.cell = nbc;
    bool ddmc_in = true;
    if (c.rebins) {
        const uint4 rn = reinterpret_cast<const uint4 *>(tb + c.off_hot)[(int64_t)p.cell * nb + p.j];
        if (!(rn.w & kFlagThick)) {   // re-binned into a thin state: MC in the new cell
            p.pos = cell_point<SPH>(fz, p.cell, p.r, a);
            p.n = iso_dir(p.r, a);
            p.left_inner = false;
            p.x = xs;
            p.mc = true;
            ++p.tomc;
            ddmc_in = false;
        }
    }
    if (CEN && c.n_census > 0 && ddmc_in)   // inward leakage into a DDMC state (eq. 18)
        accel_add<WGT>(c, tb, tally, p.cell, t0, p.t, dir * kt[(int64_t)p.cell * nb + p.j], lw0, ka, p.ci);
}

// One continuous-MC event (a scattering or a boundary crossing) of a packet in a thin state.
template <bool SPH, bool WGT, bool CEN>
__device__ __forceinline__ void mc_step1(Pk1 &p, const DevCloud &c, const uint8_t *__restrict__ tb, const McArgs &a,
                         unsigned long long *__restrict__ tally, const float *__restrict__ vtab,
                         const float *__restrict__ u0tab)
{
    ++p.mcs;
    const float4 *mcell = reinterpret_cast<const float4 *>(tb + c.off_mcell);
    const double *fz = faces_of(c, tb, 0);
    const float4 m0 = mcell[2 * p.cell];   // k0, a, sqrt(T), width
    const float4 m1c = mcell[2 * p.cell + 1];   // u, and with dust k_s, k_a
    const float uc = m1c.x;
    int fexit = 1;
    const float dwall = wall_distance<SPH>(fz[p.cell], fz[p.cell + 1], p.pos, p.n, p.left_inner, fexit);
    const float kl = m0.x * voigt_f32(m0.y, p.x, vtab);
    // dust absorption is an interaction, or (continuous weights) a decay of the weight
    const float kab = (WGT && c.dust_weight) ? 0.0f : m1c.z;
    const float kx = c.dusty ? kl + m1c.y + kab : kl;
    const float ds = -__logf(uf(draw(p.r, a))) / kx;
    const float u0 = n_dot_u<SPH>(uc, p.pos, p.n);
    const double fl = (double)fminf(ds, dwall);
    if (CEN && c.n_census > 0) {
        int jc = bin_of(c, tb, p.x);
        jc = jc < 0 ? 0 : (jc > c.nb - 1 ? c.nb - 1 : jc);
        census_add<WGT>(p, c, tb, tally, (int64_t)p.cell * c.nb + jc, p.t, p.t + fl, p.lw, (double)m1c.z);
    }
    if (WGT && c.dust_weight) {
        p.lw = fma((double)m1c.z, fl, p.lw);
        if (p.lw > kLogWMin) {   // negligible weight: eliminated
            finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
            return;
        }
    }
    if (ds < dwall) {   // an interaction
        p.pos.x = fmaf(ds, p.n.x, p.pos.x);
        p.pos.y = fmaf(ds, p.n.y, p.pos.y);
        p.pos.z = fmaf(ds, p.n.z, p.pos.z);
        p.t += (double)ds;
        if (SPH && c.moving) p.x += u0 - n_dot_u<SPH>(uc, p.pos, p.n);
        if (c.dusty) {   // which opacity interacted: dust absorption, dust scattering or Lya
            const float v = uf(draw(p.r, a)) * kx;
            if (v < kab) {
                finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
                return;
            }
            if (v < kab + m1c.y) {   // dust: isotropic, coherent in the comoving frame
                p.n = iso_dir(p.r, a);
                p.left_inner = false;
                return;
            }
        }
        float upar;
        if (!sample_upar(m0.y, p.x, u0tab, p.r, a, upar)) {
            finish1<WGT, CEN>(p, c, tally, false, 0, 0);   // counted with the step-capped packets
            return;
        }
        // perpendicular velocity in the scattering plane: sqrt(xc^2 - ln xi) cos(phi), a
        // N(0, 1/2) component without core-skipping (xc = 0)
        const float xc = (c.x_crit > 0.0f && fabsf(p.x) < c.x_crit) ? c.x_crit : 0.0f;
        const float uperp = sqrtf(fmaf(xc, xc, -__logf(uf(draw(p.r, a))))) * cosf(kTwoPi * uf(draw(p.r, a)));
        const float3 n2 = iso_dir(p.r, a);
        const float mu = dot3f(p.n, n2);
        p.x = p.x + upar * (mu - 1.0f) + uperp * sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
        p.n = n2;
        p.left_inner = false;
        const int jj = bin_of(c, tb, p.x);
        if (jj >= 0 && jj < c.nb &&
            (reinterpret_cast<const uint4 *>(tb + c.off_hot)[(int64_t)p.cell * c.nb + jj].w & kFlagThick)) {
            p.j = jj;
            p.mc = false;
            ++p.toddmc;
        }
        return;
    }
    // boundary crossing: put the point exactly on its plane or sphere
    p.pos.x = fmaf(dwall, p.n.x, p.pos.x);
    p.pos.y = fmaf(dwall, p.n.y, p.pos.y);
    p.pos.z = fmaf(dwall, p.n.z, p.pos.z);
    const float rf = (float)fz[p.cell + fexit];
    if (SPH) {
        const float3 e = radial(p.pos);
        p.pos = make_float3(rf * e.x, rf * e.y, rf * e.z);
    } else {
        p.pos.z = rf;
    }
    p.t += (double)dwall;
    const float nu = n_dot_u<SPH>(uc, p.pos, p.n);
    if (SPH && c.moving) p.x += u0 - nu;
    const int nbc = neighbour1(c, p.cell, fexit);
    if (nbc < 0) {
        finish1<WGT, CEN>(p, c, tally, true, SPH ? 0 : fexit, bin_of(c, tb, p.x + nu) + 1);
        return;
    }
    const float4 m1 = mcell[2 * nbc];
    const float xn = (p.x + nu) * (m0.z / m1.z) - n_dot_u<SPH>(mcell[2 * nbc + 1].x, p.pos, p.n);
    const int jn = bin_of(c, tb, xn);
    if (jn >= 0 && jn < c.nb &&
        (reinterpret_cast<const uint4 *>(tb + c.off_hot)[(int64_t)nbc * c.nb + jn].w & kFlagThick)) {
        const float kn = (float)reinterpret_cast<const double *>(tb + c.off_k)[(int64_t)nbc * c.nb + jn];
        const float mu = fabsf(dot3f(p.n, face_normal<SPH>(fexit, p.pos)));
        const float P = 2.0f / fmaf(kn, m1.w, 2.0f * (float)c.lambda) * (0.666666667f + mu);   // eq. 39
        if (uf(draw(p.r, a)) < P) {
            p.cell = nbc;
            p.j = jn;
            p.mc = false;
            ++p.toddmc;
            return;
        }
        // reflected: uniform point of the interface, isotropic direction back into the cell
        p.pos = face_point<SPH>(fz, p.cell, fexit, p.r, a);
        const float3 N = face_normal<SPH>(fexit, p.pos);
        p.n = hemi_about(p.r, a, make_float3(-N.x, -N.y, -N.z));
        p.left_inner = fexit == 0;   // back off the inner sphere, outward
        ++p.refl;
        return;
    }
    p.cell = nbc;
    p.left_inner = fexit == 1;
    p.x = xn;
}

// One frequency-group Monte Carlo event (Sec. 5.3) of a packet in a thin state of a static,
// isothermal cloud: the packet carries bin j; a flight meets the bin-averaged opacity k_ij
// (eq. 14) plus any dust; a scattering takes the outgoing bin from row j of the cloud's alias
// table of eq. 42 (two 32-bit words) and an isotropic direction.  Boundaries as in mc_step1,
// with the bin unchanged across faces (no velocities, one temperature).
// Bound by one wave's serial issue (about 8 cycles an instruction) and three dependent gathers: the
// opacity, the faces and, from its word of the stream, the alias entry are fetched before the next
// random block is generated, and the flags of the state entered only in clouds with thick states.
template <bool SPH, bool WGT, bool CEN>
__device__ __forceinline__ void grp_step1(Pk1 &p, const DevCloud &c, const uint8_t *__restrict__ tb, const McArgs &a,
                          unsigned long long *__restrict__ tally)
{
    ++p.mcs;
    const double *fz = faces_of(c, tb, 0);
    const double *kt = reinterpret_cast<const double *>(tb + c.off_k);
    const int64_t s = (int64_t)p.cell * c.nb + p.j;
    const double k64 = kt[s], lo = fz[p.cell], hi = fz[p.cell + 1];
    ready(p.r, a);
    uint32_t w[5];
    peek<5>(p.r, w);
    // words: flight, with dust the interaction, outgoing bin (two), direction (two)
    const uint32_t w1 = c.dusty ? w[2] : w[1], w2 = c.dusty ? w[3] : w[2];
    const int col = (int)(((uint64_t)w1 * (uint32_t)c.nb) >> 32);
    const uint2 ent = reinterpret_cast<const uint2 *>(tb + c.off_grp_alias)[(int64_t)p.j * c.nb + col];
    int fexit = 1;
    const float dwall = wall_distance<SPH>(lo, hi, p.pos, p.n, p.left_inner, fexit);
    const float kl = (float)k64;
    float ka = 0.0f, ks = 0.0f, kd = 0.0f;   // kd: dust absorption rate (either method)
    if (c.dusty) {
        const float4 m1c = reinterpret_cast<const float4 *>(tb + c.off_mcell)[2 * p.cell + 1];
        ks = m1c.y;
        kd = m1c.z;
        ka = (WGT && c.dust_weight) ? 0.0f : kd;
    }
    const float kx = kl + ks + ka;
    const float ds = -__logf(uf(w[0])) / kx;
    const double fl = (double)fminf(ds, dwall);
    if (CEN && c.n_census > 0) census_add<WGT>(p, c, tb, tally, s, p.t, p.t + fl, p.lw, (double)kd);
    if (WGT && c.dust_weight) {
        p.lw = fma((double)kd, fl, p.lw);
        if (p.lw > kLogWMin) {   // negligible weight: eliminated
            finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
            return;
        }
    }
    if (ds < dwall) {   // an interaction
        p.pos.x = fmaf(ds, p.n.x, p.pos.x);
        p.pos.y = fmaf(ds, p.n.y, p.pos.y);
        p.pos.z = fmaf(ds, p.n.z, p.pos.z);
        p.t += (double)ds;
        p.left_inner = false;
        if (c.dusty) {
            const float v = uf(w[1]) * kx;
            if (v < ka) {
                finish1<WGT, CEN>(p, c, tally, false, 0, 0, true);
                return;
            }
            if (v < ka + ks) {   // dust: isotropic, the bin unchanged
                p.n = direction(w[2], w[3]);
                advance(p.r, 4u);
                return;
            }
        }
        // eq. 42: the outgoing bin from the row's alias table
        const int jj = w2 < ent.x ? col : (int)ent.y;
        if (c.dusty) {
            advance(p.r, 4u);
            p.n = iso_dir(p.r, a);
        } else {
            p.n = direction(w[3], w[4]);
            advance(p.r, 5u);
        }
        p.j = jj;
        if (c.any_thick &&
            (reinterpret_cast<const uint4 *>(tb + c.off_hot)[(int64_t)p.cell * c.nb + jj].w & kFlagThick)) {
            p.mc = false;
            ++p.toddmc;
        }
        return;
    }
    advance(p.r, 1u);
    // boundary crossing: put the point exactly on its plane or sphere
    p.pos.x = fmaf(dwall, p.n.x, p.pos.x);
    p.pos.y = fmaf(dwall, p.n.y, p.pos.y);
    p.pos.z = fmaf(dwall, p.n.z, p.pos.z);
    const float rf = (float)(fexit ? hi : lo);
    if (SPH) {
        const float3 e = radial(p.pos);
        p.pos = make_float3(rf * e.x, rf * e.y, rf * e.z);
    } else {
        p.pos.z = rf;
    }
    p.t += (double)dwall;
    const int nbc = neighbour1(c, p.cell, fexit);
    if (nbc < 0) {
        finish1<WGT, CEN>(p, c, tally, true, SPH ? 0 : fexit, p.j + 1);
        return;
    }
    if (c.any_thick &&
        (reinterpret_cast<const uint4 *>(tb + c.off_hot)[(int64_t)nbc * c.nb + p.j].w & kFlagThick)) {
        const float4 m1 = reinterpret_cast<const float4 *>(tb + c.off_mcell)[2 * nbc];
        const float kn = (float)kt[(int64_t)nbc * c.nb + p.j];
        const float mu = fabsf(dot3f(p.n, face_normal<SPH>(fexit, p.pos)));
        const float P = 2.0f / fmaf(kn, m1.w, 2.0f * (float)c.lambda) * (0.666666667f + mu);   // eq. 39
        if (uf(draw(p.r, a)) < P) {
            p.cell = nbc;
            p.mc = false;
            ++p.toddmc;
            return;
        }
        // reflected: uniform point of the interface, isotropic direction back into the cell
        p.pos = face_point<SPH>(fz, p.cell, fexit, p.r, a);
        const float3 N = face_normal<SPH>(fexit, p.pos);
        p.n = hemi_about(p.r, a, make_float3(-N.x, -N.y, -N.z));
        p.left_inner = fexit == 0;
        ++p.refl;
        return;
    }
    p.cell = nbc;
    p.left_inner = fexit == 1;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src)
{
    const uint32_t lo = __shfl((int)(uint32_t)v, src);
    const uint32_t hi = __shfl((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// ---- cooperative walk of one packet ----------------------------------------------------------
// A DDMC step is one lane's chain of a few hundred dependent instructions and a gather, about
// 0.9 us for a lone lane, however few lanes of the wave are left.  Here the whole wave advances
// one packet: in a block, lane k draws the k-th pair of words of the packet's stream, the lanes
// hold the records of a window of states (2^(6-b) cells x 2^b bins, lane = (cell - wi) 2^b +
// (bin - wj)), and every lane computes where pair k would take a packet of its state, so that the
// packet's own position follows by one readlane per pair.  A step takes one pair {time, event},
// and a second {face, x} if its event is a spatial leak: a position with bit 6 set waits for its
// face pair.  Lane 63 is the stop: moves out of the window lead to it (the step is completed after
// the chain), and so do the steps a block does not take: ties, leaks into thin states or vacuum,
// dust absorption, spatial leaks of a cloud that re-bins on a non-uniform grid or out of the
// window, and a residence that crosses a census time.
// Those run in lane 0 with the step functions above, as do the continuous-MC events that follow
// a conversion, until the packet is in a DDMC state again.  The clock is that of the cooperative
// walk of pure clouds, census sums are integers: results do not depend on who walks a packet.
struct Window1 {
    int b, wi, wj;                        // shape and corner
    uint32_t lk, dhi, shi, ahi, split, flags;
    int dn, up, lo, hi, pend;             // where the events lead (63: stop)
    double ka;                            // continuous dust weights: absorption of the lane's cell
    double rho[2], sh[2];                 // clouds that re-bin: eq. 20 across the faces of the lane's cell
};

constexpr int kPend = 64;                 // position bit: the face pair comes next
__shared__ unsigned long long s_path_block[kBlockMax];   // a block's residence sums per position

// What the wave's lanes wrote to LDS before is seen by all of them after (the barrier alone holds the
// lanes together, but lets the compiler take a lane's own earlier store for its later load).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool WGT>
__device__ __forceinline__ void window_load(Window1 &w, const Pk1 &q, const DevCloud &c, const uint8_t *__restrict__ tb,
                                            int b, int lane)
{
    const int nb = c.nb, nc = c.nc;
    const int wjn = 1 << b, win = 64 >> b;
    int wi = q.cell - (win >> 1), wj = q.j - (wjn >> 1);
    if (wi > nc - win) wi = nc - win;
    if (wi < 0) wi = 0;
    if (wj > nb - wjn) wj = nb - wjn;
    if (wj < 0) wj = 0;
    if (((q.cell - wi) << b) + (q.j - wj) == 63) ++wj;   // the packet's own state needs a lane
    w.b = b;
    w.wi = wi;
    w.wj = wj;
    const int il = lane >> b, jl = lane & (wjn - 1);
    const bool in = wi + il < nc && wj + jl < nb;
    const int64_t s = in ? (int64_t)(wi + il) * nb + wj + jl : 0;
    const uint4 r = reinterpret_cast<const uint4 *>(tb + c.off_hot)[s];
    w.lk = r.x;
    w.dhi = r.y;
    w.shi = r.z;
    w.flags = r.w;
    w.split = reinterpret_cast<const uint32_t *>(tb + c.off_face_split)[s];
    w.ahi = 0xffffffffu;
    if (c.dusty) {   // the absorption band [A, 2^64), if any, belongs to lane 0
        const uint4 lw = reinterpret_cast<const uint4 *>(tb + c.off_lo_words)[s];
        if ((lw.w | lw.z) != 0u) w.ahi = lw.w;
    }
    if (WGT && c.dust_weight) w.ka = reinterpret_cast<const double *>(tb + c.off_dust)[2 * (in ? wi + il : 0)];
    const bool live = in && lane < 63;
    w.dn = live && jl > 0 && !(r.w & kFlagDnThin) ? lane - 1 : 63;
    w.up = live && jl < wjn - 1 && !(r.w & kFlagUpThin) ? lane + 1 : 63;
    w.lo = live && il > 0 && !(r.w & (1u << kFlagFaceShift)) ? lane - wjn : 63;
    w.hi = live && il < win - 1 && !(r.w & (2u << kFlagFaceShift)) ? lane + wjn : 63;
    // re-binning on non-uniform grids searches the edges: left to lane 0
    w.pend = live && (!c.rebins || c.uniform_bins) ? lane | kPend : 63;
    if (c.rebins) {
        const double *mp = reinterpret_cast<const double *>(tb + c.off_map) + 6 * (in ? wi + il : 0);
        w.rho[0] = mp[0];
        w.sh[0] = mp[1];
        w.rho[1] = mp[3];
        w.sh[1] = mp[4];
    }
}

// Pair K of the chain: an event pair, or the face pair of a spatial leak.
template <int K>
__device__ __forceinline__ void window_step(const Window1 &w, const DevCloud &c, uint32_t wa, uint32_t wb, int lane,
                                            int &p, int &post)
{
    if (p & kPend) {
        const bool upper = (rl(wa, K) >> 1) >= w.split;
        int nf = upper ? w.hi : w.lo;
        if (c.rebins) {   // ddmc_step1's re-binning: x uniform in the bin, moved to the neighbour's frame
            const int j = w.wj + (lane & ((1 << w.b) - 1));
            const float xin = fmaf((float)j + uf(rl(wb, K)), c.dx, c.x0);
            const double rho = upper ? w.rho[1] : w.rho[0], sh = upper ? w.sh[1] : w.sh[0];
            const float x = ((float)fma(rho, (double)xin, sh) - c.x0) * c.inv_dx;
            int jn = !(x >= 0.0f) ? 0 : (x >= (float)(c.nb - 1) ? c.nb - 1 : (int)x);
            if (rho == 1.0 && sh == 0.0) jn = j;
            const int to = nf + (jn - j);
            nf = nf == 63 || (unsigned)(jn - w.wj) >= (1u << w.b) ? 63 : to;
        }
        p = (int)rl((uint32_t)nf, p & 63);
        if (c.rebins && !(rl(w.flags, p) & kFlagThick)) p = 63;   // into a thin state: lane 0
    } else {
        const uint32_t e = rl(wb, K);
        const int f = e < w.dhi ? w.dn : w.up;
        const int x = e < w.ahi ? w.pend : 63;
        p = (int)rl((uint32_t)(e < w.shi ? f : x), p);
    }
    post = write_lane(p, K, post);
}

template <int G>
__device__ __forceinline__ void window_from(const Window1 &w, const DevCloud &c, uint32_t wa, uint32_t wb, int lane,
                                            int &p, int &post)
{
    window_step<8 * G + 0>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 1>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 2>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 3>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 4>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 5>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 6>(w, c, wa, wb, lane, p, post);
    window_step<8 * G + 7>(w, c, wa, wb, lane, p, post);
    if constexpr (G < 7) {
        if (p != 63) window_from<G + 1>(w, c, wa, wb, lane, p, post);
    }
}

__device__ __forceinline__ double shfl_f64(double v, int src)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)__shfl((int)(uint32_t)(b >> 32), src) << 32) |
                                            (uint32_t)__shfl((int)(uint32_t)b, src)));
}

// The log-weight after the residences of lanes K .. 63, added in order as the step functions do
// (lanes without one hold 0); with KEEP lane k keeps its value before residence k.
template <bool KEEP, int K>
__device__ __forceinline__ void log_weight(double &lw, double &lw0, double ka, double dd)
{
    if (KEEP) {
        const uint64_t b = (uint64_t)__double_as_longlong(lw), v = (uint64_t)__double_as_longlong(lw0);
        const int lo = write_lane((int)rl((uint32_t)b, 0), K, (int)(uint32_t)v);
        const int hi = write_lane((int)rl((uint32_t)(b >> 32), 0), K, (int)(uint32_t)(v >> 32));
        lw0 = __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
    }
    lw = fma(rl_f64(ka, K), rl_f64(dd, K), lw);
    if constexpr (K < 63) log_weight<KEEP, K + 1>(lw, lw0, ka, dd);
}

// Shape for the recent shares of spatial and frequency steps (as in the walk of pure clouds).
__device__ __forceinline__ int window_shape(const DevCloud &c, int nt, int ns)
{
    const int nf = nt - ns;
    int b = nf >= 256 * ns ? 6 : (nf >= 64 * ns ? 5 : (nf >= 4 * ns ? 4 : (4 * nf >= ns ? 3 : (64 * nf >= ns ? 2 : 1))));
    while (b > 1 && (1 << (b - 1)) >= c.nb) --b;
    while (b < 5 && (32 >> b) >= c.nc) ++b;
    return b;
}

// One block of steps of the wave-uniform packet q (word position wp, at least 64 steps below the
// step cap).  Returns true when it stopped at a step that lane 0 has to take.
template <bool WGT, bool CEN>
__device__ __forceinline__ bool window_block(Pk1 &q, uint64_t &wp, const DevCloud &c, const uint8_t *__restrict__ tb,
                                             const McArgs &a, unsigned long long *__restrict__ tally, int lane, int &nt,
                                             int &ns)
{
    Window1 w;
    window_load<WGT>(w, q, c, tb, window_shape(c, nt, ns), lane);
    // pair `lane` of the stream from wp on
    const uint64_t first = wp + 2ull * (uint64_t)lane;
    const uint64_t blk = first >> 2;
    const u32x4 r = philox4x32_10((uint32_t)blk, a.dom | (uint32_t)(blk >> 32), q.r.pid, q.r.key, a.key0, a.key1);
    const uint32_t after = (uint32_t)__shfl_down((int)r.x, 1);   // first word of the next lane's block
    const int ix = (int)(first & 3ull);
    const uint32_t wa = ix == 0 ? r.x : (ix == 1 ? r.y : (ix == 2 ? r.z : r.w));
    const uint32_t wb = ix == 0 ? r.y : (ix == 1 ? r.z : (ix == 2 ? r.w : after));
    const int m = (wp & 1ull) ? 63 : 64;
    const int p0 = (int)rl((uint32_t)(((q.cell - w.wi) << w.b) + (q.j - w.wj)), 0);
    int p = p0, post = 63;
    window_from<0>(w, c, wa, wb, lane, p, post);
    int pre = __shfl_up(post, 1);
    if (lane == 0) pre = p0;
    const bool face = (pre & kPend) != 0;      // this pair decides the face of the step before
    const int at = pre & 63;
    const uint32_t lk = (uint32_t)__shfl((int)w.lk, at), fl = (uint32_t)__shfl((int)w.flags, at);
    const uint32_t dh = (uint32_t)__shfl((int)w.dhi, at), sh = (uint32_t)__shfl((int)w.shi, at);
    const uint32_t ah = (uint32_t)__shfl((int)w.ahi, at), split = (uint32_t)__shfl((int)w.split, at);
    const bool spatial = wb >= sh;
    const int f = (wa >> 1) >= split ? 1 : 0;
    // the first pair a block leaves out: a step lane 0 takes (its event pair, also where its face
    // pair decides it), or the end
    // (in clouds that re-bin a leak out of the window too: where it ends is not known here)
    const bool hard = face ? (fl & (1u << (kFlagFaceShift + f))) != 0u || (c.rebins && post == 63)
                           : (wb == dh || wb == sh ||
                              (spatial ? wb >= ah || (c.rebins && !c.uniform_bins)
                                       : (fl & (wb < dh ? kFlagDnThin : kFlagUpThin)) != 0u));
    const uint64_t hm = __ballot(hard), fm = __ballot(face);
    uint64_t cutm = (hm & ~fm) | ((hm & fm) >> 1) | (m < 64 ? 1ull << 63 : 0ull);
    // a move out of the window completes its step: the block ends after its pair (the stop position
    // of a pair that lane 0 does not have to take)
    const uint64_t outm = __ballot(post == 63 && !hard);
    const int out = outm ? __ffsll((unsigned long long)outm) - 1 : 64;
    int done = cutm ? __ffsll((unsigned long long)cutm) - 1 : 64;
    bool stopped = done < m && done <= out;
    if (out < done) {
        done = out + 1;
        stopped = false;
    }
    // a last event pair whose face pair is not in the block waits for the next one
    if (!stopped && done > 0 && done <= 64) {
        const bool last_event = !((fm >> (done - 1)) & 1ull);
        const bool last_spatial = rl((spatial && !face) ? 1u : 0u, done - 1) != 0u;
        if (last_event && last_spatial) --done;
    }
    // residences of the event pairs
    const bool ev = lane < done && !face;
    double dd = ev ? (double)ddmc_path(wa, __uint_as_float(lk)) : 0.0;
    double t = q.t;
    double t0 = 0.0, t1 = 0.0;
    // continuous dust weights: the log-weight, step by step in order; lane k keeps it before step k
    const bool wgt = WGT && c.dust_weight;
    double lw0 = 0.0, ka = 0.0, lw = 0.0;
    if (wgt) {
        ka = shfl_f64(w.ka, at);
        lw = q.lw;
        log_weight<CEN, 0>(lw, lw0, ka, dd);
        if (lw > kLogWMin) return true;   // eliminated in this block: lane 0 finds the step
    }
    if (CEN && c.n_census > 0 && q.ci <= c.n_census) {
        // every step's own clock: the block's integer sum as a prefix sum
        double tt = q.t;
        if (!clock_parallel(tt, dd)) return true;
        const int e = (int)((((uint64_t)__double_as_longlong(q.t)) >> 52) & 0x7ffu) - 1023;
        double n = rint(ldexp(dd, 52 - e));
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double v = __shfl_up(n, o);
            if (lane >= o) n += v;
        }
        t1 = q.t + ldexp(n, e - 52);
        t0 = __shfl_up(t1, 1);
        if (lane == 0) t0 = q.t;
        const uint64_t cross = __ballot(ev && t1 > q.tn);
        if (cross) {   // that step, and what follows, is left to lane 0
            const int k = __ffsll((unsigned long long)cross) - 1;
            if (k < done) {
                done = k;
                stopped = true;
            }
        }
        t = done > 0 ? rl_f64(t1, done - 1) : q.t;
        if (q.ci > 0) {
            // the block's residences per position, then one add per visited state
            unsigned long long *acc = s_path_block + (threadIdx.x & ~63);
            acc[lane] = 0ull;
            wave_sync();
            if (lane < done && !face && t1 > t0) {
                const double r = wgt ? weight_integral(t0, t1, t0, lw0, ka) : t1 - t0;
                atomicAdd(&acc[at], (unsigned long long)rint(r * kPathFix));
            }
            wave_sync();
            const unsigned long long v = acc[lane];
            if (v) {
                const int64_t s = (int64_t)(w.wi + (lane >> w.b)) * c.nb + w.wj + (lane & ((1 << w.b) - 1));
                atomicAdd(&tally[c.tally_off + c.census_path_off + (uint64_t)(q.ci - 1) * c.n_states + s], v);
            }
        }
        // eq. 18: a leak's outward and inward terms over its step's residence
        const double ts = __shfl_up(t0, 1), ls = __shfl_up(lw0, 1);   // face pairs: the event pair before
        if (lane < done && face) {
            const double *kt = reinterpret_cast<const double *>(tb + c.off_k);
            const int i = w.wi + (at >> w.b), j = w.wj + (at & ((1 << w.b) - 1));
            const int i2 = f ? i + 1 : i - 1, j2 = post == 63 ? j : w.wj + (post & ((1 << w.b) - 1));
            const double dir = f ? 1.0 : -1.0;
            accel_add<WGT>(c, tb, tally, i, ts, t0, dir * kt[(int64_t)i * c.nb + j], ls, ka, q.ci);
            accel_add<WGT>(c, tb, tally, i2, ts, t0, dir * kt[(int64_t)i2 * c.nb + j2], ls, ka, q.ci);
        }
    } else if (done > 0 && !clock_parallel(t, dd)) {
        clock_from<0>(t, (uint32_t)__double_as_longlong(dd), (uint32_t)((uint64_t)__double_as_longlong(dd) >> 32), done);
    }
    if (done == 0) return stopped;
    // the state after the last pair: inside the window, or one move out of it
    const int l = done - 1;
    const int pl = (int)rl((uint32_t)post, l);
    if (pl != 63) {
        q.cell = w.wi + ((pl & 63) >> w.b);
        q.j = w.wj + (pl & 63 & ((1 << w.b) - 1));
    } else {
        const int al = (int)rl((uint32_t)at, l);
        q.cell = w.wi + (al >> w.b);
        q.j = w.wj + (al & ((1 << w.b) - 1));
        if ((fm >> l) & 1ull)
            q.cell += rl((uint32_t)f, l) ? 1 : -1;
        else
            q.j += rl(wb < dh ? 1u : 0u, l) ? -1 : 1;
    }
    q.t = t;
    // (only a census time cuts a block after its residences were laid out)
    if (wgt) q.lw = CEN && done < 64 ? rl_f64(lw0, done) : lw;
    wp += 2ull * (uint64_t)done;
    const int steps = __popcll(__ballot(lane < done && !face));
    q.steps += (uint64_t)steps;
    nt += steps;
    ns += __popcll(__ballot(lane < done && face));
    if (nt > 512) {   // forget older steps
        nt >>= 1;
        ns >>= 1;
    }
    return stopped;
}

// The fields of lane l's packet that a DDMC state carries, wave-uniform.
__device__ __forceinline__ void share_ddmc(Pk1 &q, const Pk1 &p, int l)
{
    q.cell = (int)rl((uint32_t)p.cell, l);
    q.j = (int)rl((uint32_t)p.j, l);
    q.active = rl(p.active ? 1u : 0u, l) != 0u;
    q.t = rl_f64(p.t, l);
    q.ci = (int)rl((uint32_t)p.ci, l);
    q.tn = rl_f64(p.tn, l);
    q.steps = rl64(p.steps, l);
    q.mcs = rl(p.mcs, l);
    q.tomc = rl(p.tomc, l);
    q.toddmc = rl(p.toddmc, l);
    q.refl = rl(p.refl, l);
}

// One packet handed over by the lane walk (its census sums flushed).
struct Tail1 {             // 104 bytes
    uint32_t cl, pid;
    int32_t cell, j;
    uint64_t steps, words;
    double t;
    uint32_t mcs, tomc, toddmc, refl;
    int32_t ci;
    uint32_t flags;        // bit 0 continuous MC, bit 1 left_inner
    float pos[3], n[3];
    float x;
    uint32_t pad;
    double lw;
};
static_assert(sizeof(Tail1) == 104, "export slots are sized by the work-area query");
// Work area (u64 words): [0] packet queue, [8] export slots handed out, [16] slots walked; slots
// from byte 256 on.
constexpr int kWGiven = 8, kWTaken = 16;

__device__ __forceinline__ Tail1 *slots_of(unsigned long long *work)
{
    return reinterpret_cast<Tail1 *>(reinterpret_cast<uint8_t *>(work) + 256);
}

// Walk the packet of an export slot to its end with the whole wave.
template <bool SPH, bool WGT, bool CEN>
__device__ __forceinline__ void coop_walk1(const Tail1 &k, const DevCloud *__restrict__ clouds,
                                           const uint8_t *__restrict__ tb, const McArgs &a,
                                           unsigned long long *__restrict__ tally, const float *__restrict__ vtab,
                                           const float *__restrict__ u0tab, int lane)
{
    Pk1 q;                                    // the packet, wave-uniform (DDMC fields)
    q.cl = (int)rl(k.cl, 0);
    const DevCloud &c = clouds[q.cl];
    q.cell = (int)rl((uint32_t)k.cell, 0);
    q.j = (int)rl((uint32_t)k.j, 0);
    q.active = true;
    q.t = rl_f64(k.t, 0);
    q.ci = (int)rl((uint32_t)k.ci, 0);
    q.tn = -__builtin_inf();                  // found again by the first residence
    q.steps = rl64(k.steps, 0);
    q.mcs = rl(k.mcs, 0);
    q.tomc = rl(k.tomc, 0);
    q.toddmc = rl(k.toddmc, 0);
    q.refl = rl(k.refl, 0);
    q.lw = WGT ? rl_f64(k.lw, 0) : 0.0;
    q.r.pid = rl(k.pid, 0);
    q.r.key = c.stream;
    uint64_t wp = rl64(k.words, 0);
    Pk1 s = q;                                // lane 0's own copy, with the continuous-MC fields
    s.mc = (k.flags & 1u) != 0u;
    s.left_inner = (k.flags & 2u) != 0u;
    s.pos = make_float3(k.pos[0], k.pos[1], k.pos[2]);
    s.n = make_float3(k.n[0], k.n[1], k.n[2]);
    s.x = k.x;
    s.cn = 0u;
    bool alone = true;
    int singles = 1, nt = 64, ns = 2;
    while (q.active) {
        if (!alone && a.max_steps - q.steps < 64ull) {   // near the cap
            alone = true;
            singles = 64;
        }
        if (alone) {
            if (lane == 0) {
                s.cell = q.cell;
                s.j = q.j;
                s.t = q.t;
                s.ci = q.ci;
                s.tn = q.tn;
                s.steps = q.steps;
                s.lw = q.lw;
                set_words(s.r, wp, a);
                do {
                    if (s.steps >= a.max_steps) {
                        finish1<WGT, CEN>(s, c, tally, false, 0, 0);
                        break;
                    }
                    ++s.steps;
                    if (!s.mc)
                        ddmc_step1<SPH, WGT, CEN>(s, c, tb, a, tally);
                    else if (c.groups)
                        grp_step1<SPH, WGT, CEN>(s, c, tb, a, tally);
                    else
                        mc_step1<SPH, WGT, CEN>(s, c, tb, a, tally, vtab, u0tab);
                } while (s.active && (s.mc || --singles > 0));
                wp = word_pos(s.r);
            }
            share_ddmc(q, s, 0);
            if (WGT) q.lw = rl_f64(s.lw, 0);
            wp = rl64(wp, 0);
            alone = false;
            singles = 1;
            continue;
        }
        alone = window_block<WGT, CEN>(q, wp, c, tb, a, tally, lane, nt, ns);
    }
}

// The packets the lane walk handed over, each by a whole wave.
template <bool SPH, bool WGT, bool CEN>
__global__ __launch_bounds__(256) void walk1dh_coop(const uint8_t *__restrict__ tb, McArgs a,
                                                    unsigned long long *__restrict__ tally,
                                                    unsigned long long *__restrict__ work)
{
    const uint64_t given = work[kWGiven];
    const uint64_t n = given < a.slots ? given : a.slots;
    if (n == 0) return;
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    const float *vtab = reinterpret_cast<const float *>(tb + H->off_voigt);
    const float *u0tab = reinterpret_cast<const float *>(tb + H->off_u0);
    const int lane = threadIdx.x & 63;
    if (CEN) path_init();
    for (;;) {
        uint64_t i = 0;
        if (lane == 0) i = atomicAdd(&work[kWTaken], 1ull);
        i = rl64(i, 0);
        if (i >= n) break;
        coop_walk1<SPH, WGT, CEN>(slots_of(work)[i], clouds, tb, a, tally, vtab, u0tab, lane);
    }
}

// Whether the cooperative walk should take the n live packets of a wave, of st steps and mc
// continuous-MC events together.  A side-by-side step costs ~2000 cycles whatever the lanes (a wave or
// two per SIMD are left by then), a cooperative one ~50-70, and an MC event ~4000 either way: with a share
// f of MC events the hand-over pays below (2000 + 4000 f) / (60 + 4000 f) lanes.  A packet that leaves for
// an MC state now and then costs a block and lane 0's steps each time: above f = 1/10 the walk in the lanes
// is the faster one (slab of 2^18 packets, f = 0.06: 667 ms in the lanes, 638 so; sphere, f = 0.07: 416
// and 395, f = 0.14: 377 and 417 if handed over).  All live packets go or none, by the wave's own share: the
// wave goes on for those that stay, and the cooperative walk starts when the last wave has ended.
// (By each packet's own share, at 1/32, half the packets of a 24 x 40 sphere at f = 0.032 left:
// 2^17 packets 336 ms, 2^20 737 ms; 275 and 652 without the hand-over; 228 and 600 so.)
// (At 1000 / 48 the dusty census slab, 16 packets to a wave, took 407 ms: most waves stayed just
// above the limit.)
__host__ __device__ constexpr bool coop_pays(float n, float st, float mc)
{
    return st >= 64.0f * n && 10.0f * mc < st && n * (60.0f * st + 4000.0f * mc) < 2000.0f * st + 4000.0f * mc;
}
static_assert(coop_pays(33, 33e4f, 0) && !coop_pays(34, 34e4f, 0), "pure DDMC packets");
static_assert(coop_pays(11, 11e4f, 3.5e3f) && !coop_pays(12, 12e4f, 3.84e3f), "an MC event in 31 steps");
static_assert(!coop_pays(1, 1e4f, 1.1e3f) && !coop_pays(1, 63, 0), "mostly MC, or just emitted");

__device__ __forceinline__ uint64_t hand_over(const Pk1 &p)
{
    const uint64_t m = __ballot(p.active);
    float st = p.active ? (float)p.steps : 0.0f, mc = p.active ? (float)p.mcs : 0.0f;
    for (int o = 32; o > 0; o >>= 1) {
        st += __shfl_xor(st, o);
        mc += __shfl_xor(mc, o);
    }
    return coop_pays((float)__popcll(m), st, mc) ? m : 0ull;
}

// Packet g of the batch's flattened packet space at its source.
template <bool SINGLE>
__device__ __forceinline__ void emit1(Pk1 &p, uint64_t g, const uint8_t *__restrict__ tb,
                                      const DevCloud *__restrict__ clouds, const uint64_t *__restrict__ prefix,
                                      const McArgs &a, unsigned long long *__restrict__ tally)
{
    int cl = 0;
    if (!SINGLE) {
        int lo = 0, hi = a.n_clouds;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (g >= prefix[mid]) lo = mid; else hi = mid;
        }
        cl = lo;
    }
    const DevCloud &c = clouds[cl];
    p.cl = cl;
    p.r = Rng{0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 4u, false, 0u, 0u, (uint32_t)(g - prefix[cl]),
              c.stream};
    // emission (Sec. 2.3): a source entry drawn by its probability
    const double u = ud(draw(p.r, a));
    const double *cdf = reinterpret_cast<const double *>(tb + c.off_src_cdf);
    int lo = 0, hi = c.n_src - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (u < cdf[mid]) hi = mid; else lo = mid + 1;
    }
    const int64_t st = reinterpret_cast<const int32_t *>(tb + c.off_src_state)[lo];
    p.cell = (int)(st / c.nb);
    p.j = (int)(st - (int64_t)p.cell * c.nb);
    p.t = 0.0;
    p.lw = 0.0;
    p.ci = 0;
    p.tn = -__builtin_inf();
    if (c.off_src_t) {   // emission uniform over the source's window
        const double *tw = reinterpret_cast<const double *>(tb + c.off_src_t) + 2 * lo;
        p.t = tw[0] + (tw[1] - tw[0]) * ud(draw(p.r, a));
    }
    p.steps = 0;
    p.mcs = p.tomc = p.toddmc = p.refl = 0u;
    p.active = true;
    const uint4 rec = reinterpret_cast<const uint4 *>(tb + c.off_hot)[st];
    p.mc = !(rec.w & kFlagThick);
    if (p.mc) {   // a thin source state starts as an MC packet at the source
        const float4 sp = reinterpret_cast<const float4 *>(tb + c.off_src_pos)[lo];
        p.pos = make_float3(0.f, 0.f, sp.z);
        p.x = sp.w;
        p.n = iso_dir(p.r, a);
        p.left_inner = false;
    }
    atomicAdd(&tally[c.tally_off + TW_LAUNCHED], 1ull);
}

// Pure frequency-group Monte Carlo: batches whose clouds all carry groups and have no thick state
// (and neither census nor weights).  The events are grp_step1's, with nothing else in the loop, and
// what the next event will gather is fetched as soon as it is known: the opacity with the outgoing
// bin, the alias entry once the next words are there, the faces when the cell changes; the new
// direction is computed while they are on their way.  A lone lane's event took 1.7 us with the
// gathers one after another between the draws, 0.8 us here (tau0 = 3e3 slab, 64 x 128), about 250
// vector instructions that one wave issues one every 4 to 8 cycles.
template <bool SPH, bool SINGLE>
__global__ __launch_bounds__(256) void walk1dg(const uint8_t *__restrict__ tb, McArgs a,
                                               unsigned long long *__restrict__ tally,
                                               unsigned long long *__restrict__ work)
{
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    const uint64_t *prefix = reinterpret_cast<const uint64_t *>(tb + H->off_prefix);
    const int lane = threadIdx.x & 63;
    Pk1 p;
    p.active = false;
    p.mc = true;
    p.left_inner = false;
    p.cl = p.cell = p.j = 0;
    p.pos = make_float3(0.f, 0.f, 0.f);
    p.n = make_float3(0.f, 0.f, 1.f);
    p.t = 0.0;
    p.steps = 0;
    p.mcs = p.tomc = p.toddmc = p.refl = 0u;
    p.r = Rng{0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 4u, false, 0u, 0u, 0u, 0u};
    double lo = 0.0, hi = 1.0, k64 = 1.0;
    uint2 ent = make_uint2(0u, 0u);
    uint32_t w0 = 0u, w1 = 0u, w2 = 0u, w3 = 0u, w4 = 0u;   // the next five words
    auto take = [&]() {
        uint32_t w[5];
        ready(p.r, a);
        peek<5>(p.r, w);
        w0 = w[0];
        w1 = w[1];
        w2 = w[2];
        w3 = w[3];
        w4 = w[4];
    };
    bool exhausted = false;
    for (;;) {
        if (!exhausted) {
            const uint64_t need = __ballot(!p.active && lane < a.lanes);
            if (need) {
                const int leader = __ffsll((unsigned long long)need) - 1;
                const int cnt = __popcll(need);
                uint64_t base = 0;
                if (lane == leader) base = atomicAdd(work, (unsigned long long)cnt);
                base = shfl64(base, leader);
                if (base + cnt >= a.count || a.one_round) exhausted = true;
                const uint64_t q = base + __popcll(need & ((1ull << lane) - 1ull));
                if (!p.active && lane < a.lanes && q < a.count) {
                    emit1<SINGLE>(p, a.first + q, tb, clouds, prefix, a, tally);
                    const DevCloud &c = clouds[SINGLE ? 0 : p.cl];
                    const double *fz = faces_of(c, tb, 0);
                    lo = fz[p.cell];
                    hi = fz[p.cell + 1];
                    k64 = reinterpret_cast<const double *>(tb + c.off_k)[(int64_t)p.cell * c.nb + p.j];
                    take();
                    const int col = (int)(((uint64_t)(c.dusty ? w2 : w1) * (uint32_t)c.nb) >> 32);
                    ent = reinterpret_cast<const uint2 *>(tb + c.off_grp_alias)[(int64_t)p.j * c.nb + col];
                }
            }
        }
        if (!__any(p.active)) break;
        const DevCloud &c = clouds[SINGLE ? 0 : p.cl];
        const double *fz = faces_of(c, tb, 0);
        const double *kt = reinterpret_cast<const double *>(tb + c.off_k);
        const uint2 *alias = reinterpret_cast<const uint2 *>(tb + c.off_grp_alias);
        const int nb = c.nb, nc = c.nc;
        const bool dusty = c.dusty != 0;
        for (int k = 0; k < a.chunk; ++k) {
            if (p.active && p.steps >= a.max_steps) finish1<false, false>(p, c, tally, false, 0, 0);
            if (!__any(p.active)) break;
            if (p.active) {
                ++p.steps;
                ++p.mcs;
                int fexit = 1;
                const float dwall = wall_distance<SPH>(lo, hi, p.pos, p.n, p.left_inner, fexit);
                float ka = 0.0f, ks = 0.0f;
                if (dusty) {
                    const float4 m1c = reinterpret_cast<const float4 *>(tb + c.off_mcell)[2 * p.cell + 1];
                    ks = m1c.y;
                    ka = m1c.z;
                }
                const float kx = (float)k64 + ks + ka;
                const float ds = -__logf(uf(w0)) / kx;
                const bool inter = ds < dwall;
                const float dl = inter ? ds : dwall;
                p.pos.x = fmaf(dl, p.n.x, p.pos.x);
                p.pos.y = fmaf(dl, p.n.y, p.pos.y);
                p.pos.z = fmaf(dl, p.n.z, p.pos.z);
                p.t += (double)dl;
                // words of a new direction (at 3, 4; at 2, 3 after a dust scattering; a dusty cloud's
                // last one follows the five)
                uint32_t d0 = w3, d1 = w4;
                bool turn = inter;
                uint32_t used = 1u;
                if (inter) {
                    p.left_inner = false;
                    used = 5u;
                    bool lya = true;
                    if (dusty) {
                        const float v = uf(w1) * kx;
                        if (v < ka) {
                            finish1<false, false>(p, c, tally, false, 0, 0, true);
                            turn = lya = false;
                        } else if (v < ka + ks) {   // dust: isotropic, the bin unchanged
                            d0 = w2;
                            d1 = w3;
                            used = 4u;
                            lya = false;
                        } else {
                            d0 = w4;
                        }
                    }
                    if (lya) {   // eq. 42: the outgoing bin from the row's alias table
                        const int col = (int)(((uint64_t)(dusty ? w2 : w1) * (uint32_t)nb) >> 32);
                        p.j = (dusty ? w3 : w2) < ent.x ? col : (int)ent.y;
                        k64 = kt[(int64_t)p.cell * nb + p.j];
                        if (dusty) {
                            advance(p.r, 5u);
                            d1 = draw(p.r, a);
                            used = 0u;
                        }
                    }
                } else {   // boundary crossing: put the point exactly on its plane or sphere
                    const float rf = (float)(fexit ? hi : lo);
                    if (SPH) {
                        const float3 e = radial(p.pos);
                        p.pos = make_float3(rf * e.x, rf * e.y, rf * e.z);
                    } else {
                        p.pos.z = rf;
                    }
                    const int nbc = fexit ? p.cell + 1 : p.cell - 1;
                    if (nbc < 0 || nbc >= nc) {
                        finish1<false, false>(p, c, tally, true, SPH ? 0 : fexit, p.j + 1);
                    } else {
                        p.cell = nbc;
                        p.left_inner = fexit == 1;
                        lo = fz[nbc];
                        hi = fz[nbc + 1];
                        k64 = kt[(int64_t)nbc * nb + p.j];
                    }
                }
                if (used) advance(p.r, used);
                take();
                const int col = (int)(((uint64_t)(dusty ? w2 : w1) * (uint32_t)nb) >> 32);
                ent = alias[(int64_t)p.j * nb + col];
                if (turn) p.n = direction(d0, d1);
            }
        }
    }
}

// Four waves per SIMD, three with census estimators or weights, two with both: the registers of the
// hand-over and of the five words of a group event had taken one wave from ten of the sixteen (2^20 packets
// of eight slabs: weights 1340 -> 1134 ms, census 1226 -> 1125, plain 925 -> 865, four spilled registers).
template <bool SPH, bool SINGLE, bool WGT, bool CEN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WGT && CEN ? 2 : (WGT || CEN ? 3 : 4)))) void walk1dh(const uint8_t *__restrict__ tb, McArgs a,
                                               unsigned long long *__restrict__ tally,
                                               unsigned long long *__restrict__ work)
{
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    const uint64_t *prefix = reinterpret_cast<const uint64_t *>(tb + H->off_prefix);
    const float *vtab = reinterpret_cast<const float *>(tb + H->off_voigt);
    const float *u0tab = reinterpret_cast<const float *>(tb + H->off_u0);
    const int lane = threadIdx.x & 63;

    Pk1 p;
    p.active = false;
    p.mc = false;
    p.left_inner = false;
    p.cl = 0;
    p.cell = 0;
    p.j = 0;
    p.pos = make_float3(0.f, 0.f, 0.f);
    p.n = make_float3(0.f, 0.f, 1.f);
    p.x = 0.f;
    p.t = 0.0;
    p.lw = 0.0;
    if (CEN) path_init();
    p.cn = 0;
    p.ci = 0;
    p.tn = -__builtin_inf();
    p.steps = 0;
    p.mcs = p.tomc = p.toddmc = p.refl = 0u;
    p.r = Rng{0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u, 4u, false, 0u, 0u, 0u, 0u};
    bool exhausted = false;

    for (;;) {
        if (!exhausted) {
            const uint64_t need = __ballot(!p.active && lane < a.lanes);
            if (need) {
                const int leader = __ffsll((unsigned long long)need) - 1;
                const int cnt = __popcll(need);
                uint64_t base = 0;
                if (lane == leader) base = atomicAdd(work, (unsigned long long)cnt);
                base = shfl64(base, leader);
                if (base + cnt >= a.count || a.one_round) exhausted = true;
                if (!p.active && lane < a.lanes) {
                    const uint64_t q = base + __popcll(need & ((1ull << lane) - 1ull));
                    if (q < a.count) {
                        emit1<SINGLE>(p, a.first + q, tb, clouds, prefix, a, tally);
                    }
                }
            }
        }
        if (!__any(p.active)) break;
        // few packets left: handed over to the cooperative walk
        const uint64_t go = a.slots && exhausted ? hand_over(p) : 0ull;
        if (go) {
            const int leader = __ffsll((unsigned long long)go) - 1;
            uint64_t base = 0;
            if (lane == leader) base = atomicAdd(&work[kWGiven], (unsigned long long)__popcll(go));
            base = shfl64(base, leader) + __popcll(go & ((1ull << lane) - 1ull));
            if (((go >> lane) & 1ull) && base < a.slots) {
                const DevCloud &c = clouds[p.cl];
                if (CEN && c.n_census > 0) path_flush(p, tally + c.tally_off + c.census_path_off);
                Tail1 k;
                k.cl = (uint32_t)p.cl;
                k.pid = p.r.pid;
                k.cell = p.cell;
                k.j = p.j;
                k.steps = p.steps;
                k.words = word_pos(p.r);
                k.t = p.t;
                k.mcs = p.mcs;
                k.tomc = p.tomc;
                k.toddmc = p.toddmc;
                k.refl = p.refl;
                k.ci = p.ci;
                k.flags = (p.mc ? 1u : 0u) | (p.left_inner ? 2u : 0u);
                k.pos[0] = p.pos.x;
                k.pos[1] = p.pos.y;
                k.pos[2] = p.pos.z;
                k.n[0] = p.n.x;
                k.n[1] = p.n.y;
                k.n[2] = p.n.z;
                k.x = p.x;
                k.pad = 0u;
                k.lw = p.lw;
                slots_of(work)[base] = k;
                p.active = false;
            }
            if (!__any(p.active)) continue;   // (packets that found no slot walk on here)
        }

        // Mode-batched passes, as on 3D grids: DDMC lanes take up to two steps, or MC lanes
        // one event; every packet's own sequence of steps and draws is unchanged by this.
        const DevCloud &c = clouds[SINGLE ? 0 : p.cl];
        for (int k = 0; k < a.chunk; ++k) {
            if (p.active && p.steps >= a.max_steps) finish1<WGT, CEN>(p, c, tally, false, 0, 0);
            const uint64_t bm = __ballot(p.active && p.mc);
            const uint64_t bd = __ballot(p.active && !p.mc);
            if (!(bm | bd)) break;
            const int nm = __popcll(bm), nd = __popcll(bd);
            const bool mc_pass = nm > 0 && (4 * nm >= nd || (k & 7) == 7);
            if (p.active && p.mc == mc_pass) {
                ++p.steps;
                if (mc_pass) {
                    if (c.groups) {
                        grp_step1<SPH, WGT, CEN>(p, c, tb, a, tally);
                    } else {
                        prefetch(p.r, a);
                        mc_step1<SPH, WGT, CEN>(p, c, tb, a, tally, vtab, u0tab);
                    }
                } else {
                    prefetch(p.r, a);
                    ddmc_step1<SPH, WGT, CEN>(p, c, tb, a, tally);
                    if (p.active && !p.mc && p.steps < a.max_steps) {
                        ++p.steps;
                        ddmc_step1<SPH, WGT, CEN>(p, c, tb, a, tally);
                    }
                }
            }
        }
    }
}

__global__ void reset_queue1(unsigned long long *work)
{
    if (blockIdx.x == 0 && threadIdx.x < 32) work[threadIdx.x] = 0ull;
}

}  // namespace

hipError_t launch_walk1dh(const uint8_t *d_tables, const DevHeader &h, bool any_thick, bool all_groups, const rddmc_run &run,
                          uint64_t first, uint64_t count, unsigned long long *d_tally, unsigned long long *d_work,
                          uint64_t work_bytes, hipStream_t s)
{
    McArgs a{};
    a.first = first;
    a.count = count;
    a.max_steps = run.max_steps;
    a.key0 = (uint32_t)run.seed;
    a.key1 = (uint32_t)(run.seed >> 32);
    a.chunk = run.chunk > 0 ? run.chunk : 64;
    a.n_clouds = h.n_clouds;
    a.dom = kDom1DH;
    const int block = run.block > 0 ? run.block : 256;
    uint64_t grid = run.grid > 0 ? (uint64_t)run.grid : 0;
    // The cooperative walk suits DDMC steps: not where no state is thick, and not asked for with
    // tail_lanes < 0.  Jobs of less than a wave per SIMD spread over the device, fewer lanes to a
    // wave: the lanes do not wait longer, and the cooperative walk finds the packets where it has
    // issue slots.
    const bool coop = any_thick && run.tail_lanes >= 0;
    a.slots = coop && work_bytes > 256 ? (work_bytes - 256) / sizeof(Tail1) : 0;
    a.lanes = 64;
    if (grid == 0) {
        const uint64_t waves = 4ull * (uint64_t)device_cu_count();
        const uint64_t per = (count + waves - 1) / waves;
        a.lanes = per < 64 ? (int)per : 64;
    }
    if (grid == 0) {
        const uint64_t want = (count + (uint64_t)a.lanes * (block / 64) - 1) / ((uint64_t)a.lanes * (block / 64));
        const uint64_t cap = (uint64_t)device_cu_count() * 8;
        grid = want < cap ? want : cap;
        if (grid < 1) grid = 1;
    }
    a.one_round = queue_in_one_round(grid * (uint64_t)(block / 64), (uint64_t)a.lanes, count, (uint64_t)device_cu_count()) ? 1 : 0;
    reset_queue1<<<1, 64, 0, s>>>(d_work);
    const bool sph = h.geometry == RDDMC_SPHERE;
    const bool single = h.n_clouds == 1;
    if (all_groups && !any_thick && !h.dust_weight1d && !h.census1d) {
        if (sph && single)
            walk1dg<true, true><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else if (sph)
            walk1dg<true, false><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else if (single)
            walk1dg<false, true><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else
            walk1dg<false, false><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        return hipGetLastError();
    }
    // batches with continuous dust weights or census estimators take instantiations of their
    // own, so that the others keep the registers (and occupancy) of a walk without them
    auto go = [&](auto wgt, auto cen) {
        constexpr bool W = decltype(wgt)::value, C = decltype(cen)::value;
        if (sph && single)
            walk1dh<true, true, W, C><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else if (sph)
            walk1dh<true, false, W, C><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else if (single)
            walk1dh<false, true, W, C><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        else
            walk1dh<false, false, W, C><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
        if (!a.slots) return;
        const unsigned blocks = (unsigned)std::min<uint64_t>((count + 3) / 4, 4ull * (uint64_t)device_cu_count());
        if (sph)
            walk1dh_coop<true, W, C><<<blocks, 256, 0, s>>>(d_tables, a, d_tally, d_work);
        else
            walk1dh_coop<false, W, C><<<blocks, 256, 0, s>>>(d_tables, a, d_tally, d_work);
    };
    if (h.dust_weight1d && h.census1d)
        go(std::true_type{}, std::true_type{});
    else if (h.dust_weight1d)
        go(std::true_type{}, std::false_type{});
    else if (h.census1d)
        go(std::false_type{}, std::true_type{});
    else
        go(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

}  // namespace rddmc
