// Persistent rDDMC walk (Sec. 2.3, eqs. 15-16; Sec. 2.5 for moving media).
//
// Every lane carries one packet in registers: cloud, packet id, cell, bin, FP64 clock
// and step count.  A step reads the state's 16-byte hot record and two 32-bit words of
// a Philox4x32-10 block keyed by (seed) and counted by (step pair, packet, cloud); one
// block serves two consecutive steps:
//   time word  -> exponential path length dl = -ln(xi) / K (xi in (0,1), f32 log2),
//   event word -> high word of a u64 uniform U compared with the state's categorical
//                 thresholds D = P(lower bin) 2^64 and S = (1 - P(spatial)) 2^64.
// When the high word decides (all but ~2^-31 of steps) the step is a frequency move;
// otherwise an auxiliary block supplies U's low word, the face choice and any
// re-binning draws.  This samples the same law as taking the smallest of independent
// exponential distances for every possible leak: the minimum is Exp(K) and the winner
// is X with probability k_X / K, independently -- exact to 2^-64 per event, which
// matters because spatial leaks from line-core bins have probabilities ~1e-10.
//
// Every `chunk` steps the wave refills lanes whose packet has finished from a global
// counter (one atomic per wave).  Escapes and step-capped packets add to exact int64
// tallies with device atomics; results depend only on (seed, cloud, packet id).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "philox.h"
#include "rddmc_internal.h"
#include "surrogate_dev.h"
#include "wave_dev.h"

namespace rddmc {

namespace {

struct WalkArgs {
    uint64_t first;        // first flattened packet index of this run
    uint64_t count;        // number of packets in this run
    uint64_t max_steps;
    uint32_t key0, key1;
    int32_t chunk;
    int32_t n_clouds;
    int32_t tail_lanes;    // export a wave's packets once the queue is empty and <= this many remain
    int32_t ahead;         // few waves per SIMD: records are fetched ahead of the step that needs them
    int32_t one_round;     // the queue is empty after one refill
    uint64_t tail_capacity;
    const uint8_t *surr;   // learned escape surrogate (windows and records) or null
    uint32_t producer_blocks;   // blocks [0, producer_blocks) walk packets from the queue;
    uint32_t producer_waves;    // later blocks walk handed-over packets cooperatively
    uint32_t consumer_waves;
    int32_t share;              // consumer waves that may be busy before a wave's last packets leave
};

// Work area (u64 words, the polled ones on their own 128-byte lines): [0] packet queue
// counter, [8] export slots handed out, [16] tickets taken by consumer waves of the
// lane-walk launch, [24] producer waves finished, [25] slots claimed by the closing
// cooperative kernel; export slots start at byte kWorkHeaderBytes.
constexpr uint64_t kWorkHeaderBytes = 256;
constexpr int kWGiven = 8, kWClaimed = 16, kWDone = 24, kWSweep = 25;

// One exported packet.  `flag` moves empty -> ready (published by the exporting lane) ->
// taken (claimed by a walking wave), or empty -> abandoned (a consumer claimed the slot
// before its packet was published and moved on) -> ready again (the exporter leaves the packet to
// the closing kernel) -> taken.
struct TailPacket {        // 48 bytes
    uint32_t cl, pid;
    int32_t i, j;
    uint64_t steps;
    double t;
    uint32_t flag, surr_calls;   // slot state; surrogate exits the packet took before
    uint64_t pad1;
};
constexpr uint32_t kSlotEmpty = 0u, kSlotReady = 1u, kSlotTaken = 2u, kSlotAbandoned = 3u;
// Polls of one export slot before a consumer wave gives up on it (about 100 s); in normal
// operation it leaves much earlier, as soon as every producer wave has finished.
constexpr int kConsumerPolls = 2000000;

// Domain tags in the second counter word (high bits of the step index never reach them).
constexpr uint32_t kDomAux = 0x80000000u;   // extra draws inside step k (re-binning, escape)
constexpr uint32_t kDomEmit = 0xC0000000u;  // emission draw
constexpr uint32_t kDomSurr = 0x40000000u;  // surrogate exit draws (per pair slot)
constexpr uint32_t kDomSub = 0x20000000u;   // sub-walk data: exit frequency inside the exit bin

__device__ __forceinline__ double u01_open_low(uint32_t r)
{   // (r + 0.5) / 2^32 in (0, 1)
    return ((double)r + 0.5) * 2.3283064365386962890625e-10;
}

__device__ __forceinline__ int locate_bin(const double *e, int nb, double x)
{   // j with e[j] <= x < e[j+1]; -1 below the grid, nb at or above the top edge
    if (x < e[0]) return -1;
    if (x >= e[nb]) return nb;
    int lo = 0, hi = nb;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (x >= e[mid]) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int time_bin(double t)
{
    if (!(t >= 1e-3)) return 0;
    const double u = (log10(t) + 3.0) * (RDDMC_TIME_BINS / 9.0);
    if (u >= (double)RDDMC_TIME_BINS) return RDDMC_TIME_BINS + 1;
    return 1 + (int)u;
}

__device__ __forceinline__ int step_bin(uint64_t n)
{
    return n <= 1 ? 0 : 63 - __clzll((long long)n);
}

__device__ void tally_finish(unsigned long long *tally, const DevCloud &c, bool escaped, int row,
                             int slot, double t, uint64_t steps)
{
    unsigned long long *w = tally + c.tally_off;
    if (escaped) {
        atomicAdd(&w[TW_ESCAPED], 1ull);
        atomicAdd(&w[kTallyHeader + (uint64_t)row * (c.nb + 2) + slot], 1ull);
        const unsigned long long tf = (unsigned long long)rint(t * kTimeFix);
        atomicAdd(&w[TW_TSUM], tf);
        const unsigned long long t2 = (unsigned long long)rint(t * t * kTimeFix);
        const unsigned long long old = atomicAdd(&w[TW_T2_LO], t2);
        if (old + t2 < old) atomicAdd(&w[TW_T2_HI], 1ull);
        const uint64_t spec_words = (uint64_t)c.n_rows * (c.nb + 2);
        atomicAdd(&w[kTallyHeader + spec_words + time_bin(t)], 1ull);
    } else {
        atomicAdd(&w[TW_CAPPED], 1ull);
    }
    const uint64_t spec_words = (uint64_t)c.n_rows * (c.nb + 2);
    atomicAdd(&w[kTallyHeader + spec_words + RDDMC_TIME_BINS + 2 + step_bin(steps)], 1ull);
    atomicAdd(&w[TW_STEPS], (unsigned long long)steps);
    atomicMax(&w[TW_STEPS_MAX], (unsigned long long)steps);
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src)
{
    const uint32_t lo = __shfl((int)(uint32_t)v, src);
    const uint32_t hi = __shfl((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// Path length of one step in length units: -ln(xi) / K with xi = (tw + 1/2) / 2^32, as
// -log2(xi) * (ln2 / K).  Written with explicit round-to-nearest operations so that the
// lane walk and the cooperative walk produce the same bits.
__device__ __forceinline__ float path_length(uint32_t tw, float ln2_over_K)
{
    const float xi = __fmul_rn(__fadd_rn((float)tw, 0.5f), 2.3283064365386963e-10f);
    return __fmul_rn(-__log2f(xi), ln2_over_K);
}

// Per-lane packet state of the 1D walk.
struct Packet1D {
    int cl, nb, nc, geom;
    uint32_t pid, key;         // packet id within its cloud; the cloud's stream key
    int i, j;
    double t;
    uint64_t steps;
    const uint4 *hot;          // HotRecord viewed as 4 words
    const float4 *cmap;        // per-cell Doppler maps {rho0, shift0, rho1, shift1}
    float x0, dx, inv_dx;      // uniform bin grid
    bool uniform;
    bool moving;               // the cloud re-bins: bulk velocity or temperatures that differ (one
                               // Philox block per step)
    bool active;
    uint32_t surr_calls;       // exits taken from the learned surrogate
};

// The cloud's surrogate window.
struct SurrWin {
    int i_lo, i_hi, j_lo, j_hi;
    uint64_t rec_off;
};

// The windows are tested by unsigned differences, in which an empty one (i_hi < i_lo) would hold
// every state: it becomes one of a cell that no cloud has.
constexpr SurrWin kNoWindow{0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff, 0ull};
__device__ __forceinline__ SurrWin surr_window(const uint8_t *__restrict__ surr, int cl)
{
    const SurrHeader *SH = reinterpret_cast<const SurrHeader *>(surr);
    const SurrCloud *c = reinterpret_cast<const SurrCloud *>(surr + SH->off_clouds) + cl;
    if (c->i_hi < c->i_lo || c->j_hi < c->j_lo) return kNoWindow;
    return SurrWin{c->i_lo, c->i_hi, c->j_lo, c->j_hi, c->rec_off};
}

__device__ __forceinline__ bool in_window(const Packet1D &p, const SurrWin &w)
{
    return (unsigned)(p.i - w.i_lo) <= (unsigned)(w.i_hi - w.i_lo) &&
           (unsigned)(p.j - w.j_lo) <= (unsigned)(w.j_hi - w.j_lo);
}

// Replace the rest of the packet's walk inside its cell by one exit drawn from the learned
// law of the state: mixture component, face, then (y1, y2) from the component's correlated
// Gaussian; x_out = S sinh(y1) in the cell's frame, dt = w exp(y2).  The exit crosses the
// face like a spatial leak (Doppler map of eq. 20 applied to x_out).  It takes a whole
// Philox pair slot (the step count is rounded up to even, then advanced by 2), drawn in
// its own counter domain.
template <bool MOVING>
__device__ __forceinline__ void mdn_exit(Packet1D &p, const SurrWin &sw, const float *__restrict__ recs,
                         const uint8_t *__restrict__ tb, const DevCloud &c, const WalkArgs &a)
{
    p.steps = (p.steps + 1ull) & ~1ull;
    const uint64_t pair = p.steps >> 1;
    const u32x4 r = philox4x32_10((uint32_t)pair, kDomSurr | (uint32_t)(pair >> 32), p.pid, p.key, a.key0, a.key1);
    const int64_t idx = (int64_t)sw.rec_off + (int64_t)(p.i - sw.i_lo) * (sw.j_hi - sw.j_lo + 1) + (p.j - sw.j_lo);
    const float *q = recs + idx * kSurrRec;
    const float u0 = ((float)(r.x >> 8) + 0.5f) * 5.9604644775390625e-8f;
    int k = 0;
    while (k < 15 && u0 >= q[kRecCdf + k]) ++k;
    const float uf = ((float)(r.y >> 8) + 0.5f) * 5.9604644775390625e-8f;
    const int face = uf < q[kRecPf0 + k] ? 0 : 1;
    const float ua = ((float)(r.z >> 8) + 0.5f) * 5.9604644775390625e-8f;
    const float ub = ((float)(r.w >> 8) + 0.5f) * 5.9604644775390625e-8f;
    const float rad = sqrtf(-2.0f * __logf(ua));
    float sn, cs;
    sincosf(6.28318530717959f * ub, &sn, &cs);
    const float n1 = rad * cs, n2 = rad * sn;
    const float rho = q[kRecRho + k];
    float y1 = fmaf(q[kRecSg1 + k], n1, q[kRecMu1 + k]);
    float y2 = q[kRecMu2 + k] + q[kRecSg2 + k] * fmaf(rho, n1, sqrtf(fmaxf(0.0f, 1.0f - rho * rho)) * n2);
    y1 = fminf(fmaxf(y1, -20.0f), 20.0f);
    y2 = fminf(y2, 80.0f);
    const float xo = q[kRecS] * sinhf(y1);
    p.t += (double)(q[kRecW] * __expf(y2));
    float xn = xo;
    if (MOVING && p.moving) {
        const float4 cm = p.cmap[p.i];
        xn = fmaf(face ? cm.z : cm.x, xo, face ? cm.w : cm.y);
    }
    int jn;
    if (p.uniform) {
        const float fj = (xn - p.x0) * p.inv_dx;
        jn = !(fj >= 0.0f) ? 0 : (fj >= (float)(p.nb - 1) ? p.nb - 1 : (int)fj);
    } else {
        jn = locate_bin(reinterpret_cast<const double *>(tb + c.off_edges), p.nb, (double)xn);
        jn = jn < 0 ? 0 : (jn > p.nb - 1 ? p.nb - 1 : jn);
    }
    p.j = jn;
    p.i += face ? 1 : -1;
    p.steps += 2ull;
    ++p.surr_calls;
}

// Random words of one step.  Static clouds: one Philox block serves two steps (time and
// event words); clouds that re-bin: one block per step (time, event, re-binning, escape mu).
// The layout is a property of the cloud, so a cloud's packets draw the same numbers in
// whichever kernel variant walks them.
struct StepWords {
    uint32_t t, e, z, w;
};

// Comoving re-binning across face `face` (Sec. 2.5, eq. 20): x uniform in bin j, mapped to
// the neighbour's frame x' = rho x + shift, re-binned and clamped to the grid.
// The neighbour's bin on a uniform grid (before clamping), with explicit rounding so that
// every walker computes the same bits.
__device__ __forceinline__ int rebin_uniform(const Packet1D &p, float rho, float sh, uint32_t zw)
{
    const float u = __fmul_rn(__fadd_rn((float)(zw >> 8), 0.5f), 5.9604644775390625e-8f);   // 24-bit uniform
    const float x = __fmaf_rn(__fadd_rn((float)p.j, u), p.dx, p.x0);
    return (int)floorf(__fmul_rn(__fsub_rn(__fmaf_rn(rho, x, sh), p.x0), p.inv_dx));
}

__device__ __forceinline__ void rebin(Packet1D &p, int face, float4 cm, uint32_t zw,
                                      const DevCloud &c, const uint8_t *__restrict__ tb)
{
    const float rho = face ? cm.z : cm.x;
    const float sh = face ? cm.w : cm.y;
    if (rho == 1.0f && sh == 0.0f) return;
    int jn;
    if (p.uniform) {
        jn = rebin_uniform(p, rho, sh, zw);
    } else {
        const double *e = reinterpret_cast<const double *>(tb + c.off_edges);
        const double x = e[p.j] + (e[p.j + 1] - e[p.j]) * u01_open_low(zw);
        jn = locate_bin(e, p.nb, (double)rho * x + (double)sh);
    }
    p.j = jn < 0 ? 0 : (jn > p.nb - 1 ? p.nb - 1 : jn);
}

// Replace the rest of the packet's walk inside its cell by one exit drawn from the exact law of
// its in-cell walk (the exact exit kernel, same window and check points as the learned
// surrogate): (face, exit bin) from the state's row CDF with a 32-bit uniform, then the spatial
// leak from the exit bin exactly as a walk step takes it (x uniform in the bin and the Doppler
// map of eq. 20 in moving clouds).  The time has the exact conditional mean m1 and squared
// coefficient of variation c2: m1 (1 - sqrt(c2)) + m1 sqrt(c2) E for c2 <= 1, else a balanced
// mixture of two exponentials (probabilities q and 1 - q, means m1 / 2q and m1 / 2(1 - q),
// q = 1 / ((1 + c2)(1 + sqrt((c2 - 1) / (c2 + 1))))), with q on the 2^-24 grid of the uniform
// that picks the branch so that the mean stays m1 exactly.  E = -ln u with u a 24-bit uniform
// (its largest value, 17.3, leaves out 6e-7 of an exponential's mean).  One Philox block in the
// surrogate's counter domain per exit: x for the CDF, y for the branch, z for the re-binning, w
// for E.
template <bool MOVING>
__device__ __forceinline__ void exact_exit(Packet1D &p, const SurrWin &sw, const uint8_t *__restrict__ tb, const DevCloud &c,
                           const WalkArgs &a)
{
    p.steps = (p.steps + 1ull) & ~1ull;
    const uint64_t pair = p.steps >> 1;
    const u32x4 r = philox4x32_10((uint32_t)pair, kDomSurr | (uint32_t)(pair >> 32), p.pid, p.key, a.key0, a.key1);
    const SurrHeader *SH = reinterpret_cast<const SurrHeader *>(a.surr);
    const int64_t idx = (int64_t)sw.rec_off + (int64_t)(p.i - sw.i_lo) * (sw.j_hi - sw.j_lo + 1) + (p.j - sw.j_lo);
    const ExitRec er = reinterpret_cast<const ExitRec *>(a.surr + SH->off_records)[idx];
    const double *cdf = reinterpret_cast<const double *>(a.surr + SH->off_rows + er.row_off);
    const double u = (double)r.x * 2.3283064365386962890625e-10;   // [0, 1) on the 2^-32 grid
    int lo = 0, hi = 2 * er.m - 1;   // first outcome whose CDF exceeds u (the last is 1)
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (u < cdf[mid]) hi = mid; else lo = mid + 1;
    }
    const int face = lo >= er.m ? 1 : 0;
    const int k = lo - face * er.m;
    const float2 tp = reinterpret_cast<const float2 *>(cdf + 2 * er.m)[k];   // {m1, c2}
    const float ex = -__logf(((float)(r.w >> 8) + 0.5f) * 5.9604644775390625e-8f);
    float dt;
    if (tp.y <= 1.0f) {
        const float b = tp.x * sqrtf(tp.y);
        dt = fmaf(b, ex, tp.x - b);
    } else {
        const float q = 1.0f / ((1.0f + tp.y) * (1.0f + sqrtf((tp.y - 1.0f) / (tp.y + 1.0f))));
        const uint32_t nq = (uint32_t)fminf(fmaxf(rintf(q * 16777216.0f), 1.0f), 8388608.0f);
        const float qk = (float)nq * 5.9604644775390625e-8f;
        dt = ((r.y >> 8) < nq ? tp.x / (2.0f * qk) : tp.x / (2.0f * (1.0f - qk))) * ex;
    }
    p.t += (double)dt;
    p.j = er.j_lo + k;
    if (MOVING && p.moving) rebin(p, face, p.cmap[p.i], r.z, c, tb);
    p.i += face ? 1 : -1;
    p.steps += 2ull;
    ++p.surr_calls;
}

// A cell exit from the surrogate buffer: the learned law or the exact kernel.
template <bool MOVING>
__device__ __forceinline__ void surrogate_exit(Packet1D &p, const SurrWin &sw, const float *__restrict__ recs,
                                               const uint8_t *__restrict__ tb, const DevCloud &c, const WalkArgs &a)
{
    if (reinterpret_cast<const SurrHeader *>(a.surr)->kind == kSurrExact)
        exact_exit<MOVING>(p, sw, tb, c, a);
    else
        mdn_exit<MOVING>(p, sw, recs, tb, c, a);
}

// Rare path of a step: the event word tied with a threshold's high word (resolved with an
// auxiliary low word) or an escape.  Returns false when the packet escaped.
template <bool MOVING>
__device__ __forceinline__ bool slow_step(Packet1D &p, StepWords w, uint4 rec, float4 cm,
                                          const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                                          const WalkArgs &a, unsigned long long *__restrict__ tally)
{
    const DevCloud &c = clouds[p.cl];
    const int s = p.i * p.nb + p.j;
    const u32x4 aux = philox4x32_10((uint32_t)p.steps, kDomAux | (uint32_t)(p.steps >> 32), p.pid, p.key,
                                    a.key0, a.key1);
    const uint4 lw = reinterpret_cast<const uint4 *>(tb + c.off_lo_words)[s];
    const uint64_t U = ((uint64_t)w.e << 32) | aux.x;
    const uint64_t D = ((uint64_t)rec.y << 32) | lw.x;
    const uint64_t S = ((uint64_t)rec.z << 32) | lw.y;
    const uint64_t F = ((uint64_t)rec.w << 32) | lw.z;
    if (U < D) { --p.j; ++p.steps; return true; }
    if (U < S) { ++p.j; ++p.steps; return true; }
    // spatial leak: face 0 (lower / inner) or face 1 (upper / outer)
    const int face = (U < F) ? 0 : 1;
    const int ni = face ? p.i + 1 : p.i - 1;
    ++p.steps;
    if (ni < 0 || ni >= p.nc) {
        int slot = p.j + 1;
        if (MOVING && p.moving) {   // lab frame: x uniform in the bin, outward mu uniform in (0, 1]
            const double *e = reinterpret_cast<const double *>(tb + c.off_edges);
            const double un = reinterpret_cast<const double *>(tb + c.off_map)[3 * (p.i * 2 + face) + 2];
            if (un != 0.0) {
                const double x = e[p.j] + (e[p.j + 1] - e[p.j]) * u01_open_low(w.z);
                slot = locate_bin(e, p.nb, x + u01_open_low(w.w) * un) + 1;
            }
        }
        tally_finish(tally, c, true, (p.geom == RDDMC_SLAB) ? face : 0, slot, p.t, p.steps);
        p.active = false;
        return false;
    }
    if (MOVING && p.moving) rebin(p, face, cm, w.z, c, tb);
    p.i = ni;
    return true;
}

// One step with its random words, the state's hot record and (moving media) the cell's
// Doppler map.  Returns -1 / +1 for a frequency move and 2 for a spatial move decided on
// the fast path, 0 for a step that took the slow path.
template <bool MOVING>
__device__ __forceinline__ int one_step(Packet1D &p, StepWords w, uint4 rec, float4 cm,
                                        const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                                        const WalkArgs &a, unsigned long long *__restrict__ tally)
{
    p.t += (double)path_length(w.t, __uint_as_float(rec.x));
    const uint32_t ew = w.e;
    const bool tie = (ew == rec.y) | (ew == rec.z) | (ew == rec.w);
    if (__builtin_expect(!tie, 1)) {
        if (ew < rec.z) {
            const int d = (ew < rec.y) ? -1 : 1;
            p.j += d;
            ++p.steps;
            return d;
        }
        const int face = (ew < rec.w) ? 0 : 1;
        const int ni = face ? p.i + 1 : p.i - 1;
        if ((unsigned)ni < (unsigned)p.nc) {
            if (MOVING && p.moving) rebin(p, face, cm, w.z, clouds[p.cl], tb);
            p.i = ni;
            ++p.steps;
            return 2;
        }
    }
    slow_step<MOVING>(p, w, rec, cm, tb, clouds, a, tally);
    return 0;
}

template <bool MOVING>
__device__ __forceinline__ StepWords words_of_step(const Packet1D &p, uint64_t step, const WalkArgs &a)
{
    if (MOVING && p.moving) {
        const u32x4 r = philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), p.pid, p.key, a.key0, a.key1);
        return {r.x, r.y, r.z, r.w};
    }
    const uint64_t pr = step >> 1;
    const u32x4 r = philox4x32_10((uint32_t)pr, (uint32_t)(pr >> 32), p.pid, p.key, a.key0, a.key1);
    return (step & 1) ? StepWords{r.z, r.w, 0u, 0u} : StepWords{r.x, r.y, 0u, 0u};
}

// One step's fast path as selects (no branches): the clock advances for every enabled lane;
// a frequency move or a spatial move inside the grid is applied; returns true when the step
// needs the slow path (a tie with a threshold's high word, or a leak out of the grid), which
// the caller runs.  Disabled lanes change nothing.  The arithmetic is that of one_step.
__device__ __forceinline__ bool select_step(Packet1D &p, bool en, uint32_t tw, uint32_t ew, uint4 rec, int &d)
{
    const double tn = p.t + (double)path_length(tw, __uint_as_float(rec.x));
    p.t = en ? tn : p.t;
    const bool tie = (ew == rec.y) | (ew == rec.z) | (ew == rec.w);
    const bool freq = ew < rec.z;
    const int dj = ew < rec.y ? -1 : 1;
    const int ni = ew < rec.w ? p.i - 1 : p.i + 1;
    const bool inside = (unsigned)ni < (unsigned)p.nc;
    const bool slow = en & (tie | (!freq & !inside));
    const bool fast = en & !slow;
    p.j = (fast & freq) ? p.j + dj : p.j;
    p.i = (fast & !freq) ? ni : p.i;
    p.steps += fast ? 1ull : 0ull;
    d = slow ? 0 : (freq ? dj : 2);
    return slow;
}

// Whether the surrogate exits of a pass are taken now: an exit is a search of dependent gathers that
// the wave's other lanes wait for, so lanes due for one wait until they are a third of the live
// ones (or every eighth pass, or nobody else steps).  Which pass takes a packet's exit does not
// change its steps.  (Exit kernel, tau0 = 1e7 sphere, 2^18 packets: 273 ms with an exit pass
// whenever a lane is due, 262 ms so, both before the present hand-over.)
__device__ __forceinline__ bool exits_due(bool sx, bool step, int k)
{
    const uint64_t x = __ballot(sx), o = __ballot(step);
    return x != 0ull && (2 * __popcll(x) >= __popcll(o) || (k & 7) == 7);
}

// Pairs of static-medium steps: the lanes that step share one masked region per pair, in which the
// common moves are selects; ties and escapes run under a mask of their own.  Where waves fill the
// SIMDs, each step's record is gathered when its state is known, one gather a step: other waves
// cover its latency, and gathers ahead cost more than they save (2^20 packets of the efficient-grid
// tau0 = 1e7 sphere: 154 ms with three gathers ahead and a fourth after a spatial move, 109 ms so, with
// the tail thresholds below).  With AHEAD, for grids of a few waves per SIMD, the neighbouring bins'
// records are fetched with the pair's first, so that a frequency move does not wait (2^12 packets of
// the tau0 = 1e5 slab 530 ms, 600 without).
// Same records, random words and arithmetic as one_step, so the same bits.
template <bool MOVING, bool SURR, bool AHEAD>
__device__ __forceinline__ void static_pairs(Packet1D &p, int budget, int last_state, const uint8_t *__restrict__ tb,
                                             const DevCloud *__restrict__ clouds, const WalkArgs &a,
                                             unsigned long long *__restrict__ tally, const SurrWin *sw,
                                             const float *__restrict__ recs)
{
    const float4 nomap = make_float4(1.f, 0.f, 1.f, 0.f);
    for (int k = 0; k < a.chunk; ++k) {
        bool en = p.active && k < budget && (!SURR || p.steps < a.max_steps);
        if (!__any(en)) break;
        if (SURR) {   // a pair that starts in the surrogate window is replaced by one exit
            const bool sx = en && p.steps + 3ull <= a.max_steps && in_window(p, *sw);
            en = en && !sx;
            if (exits_due(sx, en, k)) {
                if (sx) surrogate_exit<MOVING>(p, *sw, recs, tb, clouds[p.cl], a);
            }
        }
        if (en) {
            const int s = p.i * p.nb + p.j;
            const uint4 r0 = p.hot[s];
            uint4 rm, rp;
            if (AHEAD) {
                rm = p.hot[s > 0 ? s - 1 : 0];
                rp = p.hot[s < last_state ? s + 1 : s];
            }
            const uint64_t pair = p.steps >> 1;
            const u32x4 r = philox4x32_10((uint32_t)pair, (uint32_t)(pair >> 32), p.pid, p.key, a.key0, a.key1);
            int d;
            const bool s1 = select_step(p, true, r.x, r.y, r0, d);
            if (s1) slow_step<MOVING>(p, StepWords{r.x, r.y, 0u, 0u}, r0, nomap, tb, clouds, a, tally);
            if (p.active && p.steps < a.max_steps) {
                uint4 r1;
                if (AHEAD) {
                    r1 = d == -1 ? rm : rp;
                    if (d == 0 || d == 2) r1 = p.hot[p.i * p.nb + p.j];   // after a spatial move or a slow step
                } else {
                    r1 = p.hot[p.i * p.nb + p.j];
                }
                const bool s2 = select_step(p, true, r.z, r.w, r1, d);
                if (s2) slow_step<MOVING>(p, StepWords{r.z, r.w, 0u, 0u}, r1, nomap, tb, clouds, a, tally);
            }
        }
    }
}

// One moving-medium step as selects: like select_step, with the Doppler re-binning of a
// spatial move (eq. 20) computed inline on uniform grids; on other grids the lanes that
// moved spatially re-bin under a mask.  The arithmetic is that of one_step.
__device__ __forceinline__ bool select_step_moving(Packet1D &p, bool en, StepWords w, uint4 rec, float4 cm,
                                                   const DevCloud *__restrict__ clouds,
                                                   const uint8_t *__restrict__ tb)
{
    const double tn = p.t + (double)path_length(w.t, __uint_as_float(rec.x));
    p.t = en ? tn : p.t;
    const uint32_t ew = w.e;
    const bool tie = (ew == rec.y) | (ew == rec.z) | (ew == rec.w);
    const bool freq = ew < rec.z;
    const int dj = ew < rec.y ? -1 : 1;
    const bool up = ew >= rec.w;   // face 1 (upper / outer)
    const int ni = up ? p.i + 1 : p.i - 1;
    const bool inside = (unsigned)ni < (unsigned)p.nc;
    const bool slow = en & (tie | (!freq & !inside));
    const bool fast = en & !slow;
    const bool spatial = fast & !freq;
    const float rho = up ? cm.z : cm.x;
    const float sh = up ? cm.w : cm.y;
    const bool ident = (rho == 1.0f) & (sh == 0.0f);
    int jn = rebin_uniform(p, rho, sh, w.z);
    jn = jn < 0 ? 0 : (jn > p.nb - 1 ? p.nb - 1 : jn);
    const bool other_grid = spatial & !ident & !p.uniform;
    p.j = (fast & freq) ? p.j + dj : ((spatial & !ident & p.uniform) ? jn : p.j);
    if (__any(other_grid)) {
        if (other_grid) rebin(p, up ? 1 : 0, cm, w.z, clouds[p.cl], tb);
    }
    p.i = spatial ? ni : p.i;
    p.steps += fast ? 1ull : 0ull;
    return slow;
}

// Moving-medium steps (one Philox block each): at most `lim` iterations, lanes past their own
// `budget` left out; with the surrogate, a step that starts in the window is replaced by one exit.
template <bool SURR = false>
__device__ __forceinline__ void moving_steps(Packet1D &p, int budget, int lim, const uint8_t *__restrict__ tb,
                                             const DevCloud *__restrict__ clouds, const WalkArgs &a,
                                             unsigned long long *__restrict__ tally, const SurrWin *sw = nullptr,
                                             const float *__restrict__ recs = nullptr)
{
    for (int k = 0; k < lim; ++k) {
        bool en = p.active && k < budget && (!SURR || p.steps < a.max_steps);
        if (!__any(en)) break;
        if (SURR) {
            const bool sx = en && p.steps + 3ull <= a.max_steps && in_window(p, *sw);
            en = en && !sx;
            if (exits_due(sx, en, k)) {
                if (sx) surrogate_exit<true>(p, *sw, recs, tb, clouds[p.cl], a);
            }
        }
        if (en) {
            const uint4 rec = p.hot[p.i * p.nb + p.j];
            const float4 cm = p.cmap[p.i];
            const u32x4 r = philox4x32_10((uint32_t)p.steps, (uint32_t)(p.steps >> 32), p.pid, p.key, a.key0, a.key1);
            const StepWords w{r.x, r.y, r.z, r.w};
            const bool slow = select_step_moving(p, true, w, rec, cm, clouds, tb);
            if (slow) slow_step<true>(p, w, rec, cm, tb, clouds, a, tally);
        }
    }
}

// 1D walk (slab or sphere), pure DDMC; MOVING enables Doppler re-binning and lab-frame
// escape frequencies.  Static media take one Philox block per pair of steps ((x, y) for the
// even step and (z, w) for the odd one; all active lanes of a wave are at even step counts
// between pairs); moving media take one block per step.
template <bool MOVING, bool SURR, bool SUB = false>
__device__ int coop_walk(Packet1D &q, const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                         const WalkArgs &a, unsigned long long *__restrict__ tally, int lane);

__device__ __forceinline__ TailPacket *slots_of(unsigned long long *work)
{
    return reinterpret_cast<TailPacket *>(reinterpret_cast<uint8_t *>(work) + kWorkHeaderBytes);
}

// The packet's copies of its cloud's fields.
__device__ __forceinline__ void set_cloud(Packet1D &p, const uint8_t *__restrict__ tb, const DevCloud &c)
{
    p.key = c.stream;
    p.nb = c.nb;
    p.nc = c.nc;
    p.geom = c.geometry;
    p.hot = reinterpret_cast<const uint4 *>(tb + c.off_hot);
    p.cmap = reinterpret_cast<const float4 *>(tb + c.off_cmap);
    p.x0 = c.x0;
    p.dx = c.dx;
    p.inv_dx = c.inv_dx;
    p.uniform = c.uniform_bins != 0;
    p.moving = c.rebins != 0u;
}

// The packet of an export slot as a wave-uniform state.
__device__ Packet1D load_slot(const TailPacket *ts, const uint8_t *__restrict__ tb,
                              const DevCloud *__restrict__ clouds)
{
    const TailPacket tk = *ts;
    Packet1D q;
    q.cl = (int)rl(tk.cl, 0);
    set_cloud(q, tb, clouds[q.cl]);
    q.pid = rl(tk.pid, 0);
    q.i = (int)rl((uint32_t)tk.i, 0);
    q.j = (int)rl((uint32_t)tk.j, 0);
    q.steps = ((uint64_t)rl((uint32_t)(tk.steps >> 32), 0) << 32) | rl((uint32_t)tk.steps, 0);
    const uint64_t tb64 = ((uint64_t)rl((uint32_t)(__double_as_longlong(tk.t) >> 32), 0) << 32) |
                          rl((uint32_t)__double_as_longlong(tk.t), 0);
    q.t = __longlong_as_double((long long)tb64);
    q.active = true;
    q.surr_calls = rl(tk.surr_calls, 0);
    return q;
}

// A consumer wave (a block past the producers) walks handed-over packets cooperatively, one after
// another.  It takes a ticket, the index of the export slot it will walk next, with one atomic
// add, and polls that slot alone: claiming the next published slot by compare-and-swap on a
// shared counter let a few thousand waves fail against one that succeeded, ~25 us per claim.
// (The efficient-grid sphere of 64 shells, 6e4 packets: 390 ms with the shared claim, 5.5 ms with
// tickets.)  Polls start about 1 us apart and double to about 50 us; they are relaxed (an acquire would
// invalidate the compute unit's vector cache under the waves that still walk there).  Before every poll the wave reads how
// many producer waves have finished: once all have, a slot that was never handed out ends the
// wave, and one that was is already published.  After kConsumerPolls polls of one slot the wave
// marks it abandoned and leaves; what is left, the closing kernel walks.
template <bool MOVING, bool SURR>
__device__ void consume_exported(const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                                 const WalkArgs &a, unsigned long long *__restrict__ tally,
                                 unsigned long long *__restrict__ work, int lane)
{
    TailPacket *slots = slots_of(work);
    for (;;) {
        uint64_t idx = 0;
        uint32_t got = 0u;
        if (lane == 0) {
            idx = __hip_atomic_fetch_add(&work[kWClaimed], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (idx < a.tail_capacity) {
                uint32_t *f = &slots[idx].flag;
                int nap = 1;
                for (int poll = 0; poll < kConsumerPolls; ++poll) {
                    const bool over = __hip_atomic_load(&work[kWDone], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >=
                                      (unsigned long long)a.producer_waves;
                    if (over) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kSlotReady) {
                        got = 1u;
                        break;
                    }
                    if (over) break;
                    for (int z = 0; z < nap; ++z) __builtin_amdgcn_s_sleep(32);
                    nap = nap < 64 ? 2 * nap : 64;
                }
                uint32_t expect = got ? kSlotReady : kSlotEmpty;
                if (__hip_atomic_compare_exchange_strong(f, &expect, got ? kSlotTaken : kSlotAbandoned, __ATOMIC_ACQ_REL,
                                                         __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == false)
                    got = 0u;
            }
        }
        if (rl(got, 0) == 0u) return;
        idx = ((uint64_t)rl((uint32_t)(idx >> 32), 0) << 32) | rl((uint32_t)idx, 0);
        Packet1D q = load_slot(slots + idx, tb, clouds);
        coop_walk<MOVING, SURR>(q, tb, clouds, a, tally, lane);
    }
}

template <bool MOVING, bool SURR>
__global__ __launch_bounds__(256) void walk1d(const uint8_t *__restrict__ tb, WalkArgs a,
                                              unsigned long long *__restrict__ tally,
                                              unsigned long long *__restrict__ work)
{
    const SurrHeader *SH = SURR ? reinterpret_cast<const SurrHeader *>(a.surr) : nullptr;
    const float *recs = SURR ? reinterpret_cast<const float *>(a.surr + SH->off_records) : nullptr;
    SurrWin sw = kNoWindow;
    int last_state = 0;
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    const uint64_t *prefix = reinterpret_cast<const uint64_t *>(tb + H->off_prefix);
    const int lane = threadIdx.x & 63;
    if (blockIdx.x >= a.producer_blocks) {   // a consumer block
        consume_exported<MOVING, SURR>(tb, clouds, a, tally, work, lane);
        return;
    }

    Packet1D p;
    p.active = false;
    p.cl = 0; p.nb = 1; p.nc = 1; p.geom = 0; p.pid = 0; p.key = 0; p.i = 0; p.j = 0; p.t = 0.0; p.steps = 0;
    p.hot = nullptr;
    p.cmap = nullptr;
    p.x0 = 0.f; p.dx = 1.f; p.inv_dx = 1.f; p.uniform = false; p.moving = false;
    p.surr_calls = 0u;
    bool exhausted = false;       // wave-uniform: the queue is empty

    for (;;) {
        // ---- refill finished lanes (one atomic per wave) -----------------------------
        if (!exhausted) {
            const uint64_t need = __ballot(!p.active);
            if (need) {
                const int leader = __ffsll((unsigned long long)need) - 1;
                const int cnt = __popcll(need);
                uint64_t base = 0;
                if (lane == leader) base = atomicAdd(work, (unsigned long long)cnt);
                base = shfl_u64(base, leader);
                if (base + cnt >= a.count || a.one_round) exhausted = true;
                if (!p.active) {
                    const int rank = __popcll(need & ((1ull << lane) - 1ull));
                    const uint64_t q = base + rank;
                    if (q < a.count) {
                        const uint64_t g = a.first + q;
                        int lo = 0, hi = a.n_clouds;      // prefix[lo] <= g < prefix[hi]
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (g >= prefix[mid]) lo = mid; else hi = mid;
                        }
                        p.cl = lo;
                        const DevCloud &c = clouds[lo];
                        p.pid = (uint32_t)(g - prefix[lo]);
                        set_cloud(p, tb, c);
                        last_state = (int)c.n_states - 1;
                        // emission (Sec. 2.3): a source state drawn by its probability
                        const u32x4 r = philox4x32_10(0u, kDomEmit, p.pid, p.key, a.key0, a.key1);
                        const double u = u01_open_low(r.x);
                        const int32_t *ss = reinterpret_cast<const int32_t *>(tb + c.off_src_state);
                        const double *cdf = reinterpret_cast<const double *>(tb + c.off_src_cdf);
                        int k = 0;
                        while (k < c.n_src - 1 && u >= cdf[k]) ++k;
                        const int32_t st = ss[k];
                        p.i = st / p.nb;
                        p.j = st - p.i * p.nb;
                        p.t = 0.0;
                        p.steps = 0;
                        p.active = true;
                        p.surr_calls = 0u;
                        if (SURR) sw = surr_window(a.surr, lo);
                        atomicAdd(&tally[c.tally_off + TW_LAUNCHED], 1ull);
                    }
                }
            }
        }
        if (!__any(p.active)) break;

        // ---- tail: hand packets of this wave to the cooperative walk ------------------------------
        // The last few of the wave all at once; before that, where producers leave SIMDs idle, as many
        // as the consumer waves there are free to take (a wave waiting on its ticket is free).
        if (exhausted && a.tail_lanes > 0) {
            const uint64_t live = __ballot(p.active);
            const int n = __popcll(live);
            int give = n <= a.tail_lanes ? n : 0;
            if (give == 0 && a.share > 0) {
                int room = 0;
                if (lane == 0) {
                    const int64_t waiting =
                        (int64_t)(__hip_atomic_load(&work[kWClaimed], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) -
                                  __hip_atomic_load(&work[kWGiven], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    const int64_t busy = (int64_t)a.consumer_waves - waiting;
                    room = busy < a.share ? (int)((a.share - busy) / (int64_t)a.producer_waves) + 1 : 0;
                }
                room = (int)rl((uint32_t)room, 0);
                give = room < n ? room : n;
            }
            if (give > 0) {
                const int leader = __ffsll((unsigned long long)live) - 1;
                const int rank = __popcll(live & ((1ull << lane) - 1ull));
                uint64_t base = 0;
                if (lane == leader) base = atomicAdd(&work[kWGiven], (unsigned long long)give);
                base = shfl_u64(base, leader);
                if (p.active && rank < give) {
                    TailPacket *tp = slots_of(work) + base + rank;
                    tp->cl = (uint32_t)p.cl;
                    tp->pid = p.pid;
                    tp->i = p.i;
                    tp->j = p.j;
                    tp->steps = p.steps;
                    tp->t = p.t;
                    tp->surr_calls = p.surr_calls;
                    __threadfence();
                    uint32_t expect = kSlotEmpty;
                    // a slot its consumer gave up on before it was published (the ticket is spent, so no
                    // other consumer looks at it): published again for the closing kernel
                    if (!__hip_atomic_compare_exchange_strong(&tp->flag, &expect, kSlotReady, __ATOMIC_RELEASE,
                                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                        __hip_atomic_store(&tp->flag, kSlotReady, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                    p.active = false;
                }
                if (give == n) break;
            }
        }

        // ---- walk up to `chunk` pairs of steps ---------------------------------------
        const bool was_active = p.active;
        const uint64_t left = p.active ? (a.max_steps - p.steps) : 0ull;
        if (!(MOVING && p.moving)) {
            const uint64_t pairs = (left + 1) >> 1;
            const int budget = pairs < (uint64_t)a.chunk ? (int)pairs : a.chunk;
            if (!SURR && a.ahead)
                static_pairs<MOVING, false, true>(p, budget, last_state, tb, clouds, a, tally, &sw, recs);
            else
                static_pairs<MOVING, SURR, false>(p, budget, last_state, tb, clouds, a, tally, &sw, recs);
        }
        if (MOVING && p.moving) {
            const uint64_t lim = 2ull * (uint64_t)a.chunk;
            const int budget = left < lim ? (int)left : (int)lim;
            moving_steps<SURR>(p, budget, (int)lim, tb, clouds, a, tally, &sw, recs);
        }
        if (p.active && p.steps >= a.max_steps) {
            tally_finish(tally, clouds[p.cl], false, 0, 0, p.t, p.steps);
            p.active = false;
        }
        if (SURR && was_active && !p.active && p.surr_calls)
            atomicAdd(&tally[clouds[p.cl].tally_off + TW_SURR_CALLS], (unsigned long long)p.surr_calls);
    }
    if (lane == 0) __hip_atomic_fetch_add(&work[kWDone], 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Cooperative walk of ONE packet by a whole wave (the packet state is wave-uniform).
//   * The 64 lanes hold the hot records of 64 consecutive bins of the packet's cell (the
//     band); each block of up to 128 steps walks a 30-bin window of it.
//   * Lane l draws the words of two steps (in static media one Philox pair).  A frequency step
//     changes the parity of the position, so the first of a lane's steps starts at an even and
//     the second at an odd window position: 15 each, which a table of 4-bit fields in two
//     registers holds (field m: the next position's index, 15 out of the window).  The tables of
//     a lane's two steps are composed by shifts and selects of whole words, and so are those of
//     an even lane and the next.
//   * The sequential part is a scalar chain of two instructions per four steps (a 4-bit field
//     extract addressed by the position, a shift-add back to an address); even lanes receive the
//     position their steps start from, the others derive theirs.
//   * Each lane then looks at its two steps' thresholds: the first leak, tie, surrogate exit or
//     move out of the window (or the step cap) ends the block; a move completes, the others run in
//     lane 0 with the lane walk's arithmetic.
// The clock gives the bits of the lane walk's ordered FP64 additions (clock_parallel, else
// in order), so every tally is bit-identical to walking the packet in a single lane.
// Bound: dependent instructions of one wave, ~660 a block.  One packet of the tau0 = 1e5 slab (64 x
// 128) takes 22 ns per step and one of a 3 x 300 slab 29 ns; with one step per lane, 15-bin windows
// and all stops in the tables (58 instead of 102 steps a block) it was 30 and 37.
constexpr int kCoopWin = 30;
// scan state: 4 x position index in bits 0..5, field width 4 in bits 16..22 (the operand
// layout of s_bfe_u64); kScanStop is the state of the stop position
constexpr uint32_t kScanWidth = 4u << 16;
constexpr uint32_t kScanStop = kScanWidth | (15u << 2);

// Step L of the chain: hand lane L its starting state, then move to the next position.
template <int L>
__device__ __forceinline__ void scan_step(uint32_t &st, int &vst, uint32_t tlo, uint32_t thi)
{
    const uint64_t tab = ((uint64_t)rl(thi, L) << 32) | rl(tlo, L);
    uint64_t f;
    asm("v_writelane_b32 %0, %1, %2" : "+v"(vst) : "s"(st), "n"(L));
    asm("s_bfe_u64 %0, %1, %2" : "=s"(f) : "s"(tab), "s"(st) : "scc");
    asm("s_lshl2_add_u32 %0, %1, %2" : "=s"(st) : "s"((uint32_t)f), "s"(kScanWidth) : "scc");
}

// The chain over four-step tables held by the even lanes, sixteen steps per group, leaving once
// the stop is reached.
template <int G>
__device__ __forceinline__ void scan_from(uint32_t &st, int &vst, uint32_t tlo, uint32_t thi)
{
    scan_step<8 * G + 0>(st, vst, tlo, thi);
    scan_step<8 * G + 2>(st, vst, tlo, thi);
    scan_step<8 * G + 4>(st, vst, tlo, thi);
    scan_step<8 * G + 6>(st, vst, tlo, thi);
    if constexpr (G < 7) {
        if (st != kScanStop) scan_from<G + 1>(st, vst, tlo, thi);
    }
}

// The packet as lane 0 left it, made wave-uniform again.
template <bool SURR>
__device__ __forceinline__ void take_lane0(Packet1D &q, const Packet1D &s1)
{
    q.i = (int)rl((uint32_t)s1.i, 0);
    q.j = (int)rl((uint32_t)s1.j, 0);
    q.steps = ((uint64_t)rl((uint32_t)(s1.steps >> 32), 0) << 32) | rl((uint32_t)s1.steps, 0);
    const uint64_t tbits = (uint64_t)__double_as_longlong(s1.t);
    q.t = __longlong_as_double((long long)(((uint64_t)rl((uint32_t)(tbits >> 32), 0) << 32) | rl((uint32_t)tbits, 0)));
    q.active = rl(s1.active ? 1u : 0u, 0) != 0u;
    if (SURR) q.surr_calls = rl(s1.surr_calls, 0);
}

// ---- blocks of mixed steps -------------------------------------------------------------------
// Where spatial leaks are frequent the table scan above stops after a few steps.  A mixed block
// holds a window of states around the packet instead, one state per lane: 2^(6-b) cells x 2^b
// bins, lane = (cell - wi) 2^b + (bin - wj).  For step k every lane computes where that step
// would take a packet of ITS state (the event word is wave-uniform), and the packet's position
// follows by one readlane: p <- next[p].  Lane 63 is the stop: its own next position is 63, and
// a move out of the window or the grid, and (with the surrogate) a step that starts in the
// surrogate window at a check point, lead to it.  Ties with a threshold's high word are found
// after the chain, when lane k holds step k's position and its records, and cut the block.
// The step a block stops at is taken with the lane walk's arithmetic.
// Bound: instruction issue of one wave, 9 vector instructions per step (about 25 with a Doppler
// re-binning; done for the packet's own state alone, behind a branch on its position, it is a
// serial chain: the moving 24 x 64 sphere took 64 ms instead of 30), and per block ~250 for the
// words, the window and the clock.  The static slab of 9 cells x 17 bins (tau0 = 300, 3e4 packets) takes 5.0 ms where lane 0 walking such runs alone took
// 157 ms (with the claims below); the slowest packet of a 40 x 50 sphere (3.1e5 steps) 58 ns per step.
struct MixWindow {
    int b, wi, wj;                             // shape and corner
    uint32_t lk, dhi, shi, fhi;                // the lane's record
    int dn, up, lo, hi;                        // where the four moves lead (63: stop)
    float4 cm;                                 // the Doppler map of the lane's cell
    bool id0, id1;                             // identity across face 0 / face 1
};

template <bool MOVING>
__device__ __forceinline__ void mix_load(MixWindow &w, const Packet1D &q, int b, int lane)
{
    const int wjn = 1 << b, win = 64 >> b;
    int wi = q.i - (win >> 1), wj = q.j - (wjn >> 1);
    if (wi > q.nc - win) wi = q.nc - win;
    if (wi < 0) wi = 0;
    if (wj > q.nb - wjn) wj = q.nb - wjn;
    if (wj < 0) wj = 0;
    if (((q.i - wi) << b) + (q.j - wj) == 63) ++wj;   // the packet's own state needs a lane
    w.b = b;
    w.wi = wi;
    w.wj = wj;
    const int il = lane >> b, jl = lane & (wjn - 1);
    const int i = wi + il, j = wj + jl;
    const bool in = i < q.nc && j < q.nb;
    const uint4 r = q.hot[in ? i * q.nb + j : 0];
    w.lk = r.x;
    w.dhi = r.y;
    w.shi = r.z;
    w.fhi = r.w;
    const bool live = in && lane < 63;
    w.dn = live && jl > 0 ? lane - 1 : 63;
    w.up = live && jl < wjn - 1 && j + 1 < q.nb ? lane + 1 : 63;
    w.lo = live && il > 0 ? lane - wjn : 63;
    w.hi = live && il < win - 1 && i + 1 < q.nc ? lane + wjn : 63;
    if (MOVING && q.moving) {
        w.cm = q.cmap[in ? i : 0];
        w.id0 = w.cm.x == 1.0f && w.cm.y == 0.0f;
        w.id1 = w.cm.z == 1.0f && w.cm.w == 0.0f;
    }
}

// Step k of the chain: every lane's next position, then the packet's.
template <bool MOVING, bool SURR>
__device__ __forceinline__ void mix_step(const MixWindow &w, const Packet1D &q, bool rebins, int k, uint32_t ew, float u,
                                         bool stop_here, int lane, int &p, int &post)
{
    const uint32_t e = rl(ew, k);
    const int f = e < w.dhi ? w.dn : w.up;
    const bool inner = e < w.fhi;
    int x = inner ? w.lo : w.hi;
    if (MOVING && rebins) {
        const float uk = __uint_as_float(rl(__float_as_uint(u), k));
        const int j = w.wj + (lane & ((1 << w.b) - 1));
        const float xj = __fmaf_rn(__fadd_rn((float)j, uk), q.dx, q.x0);
        const float rho = inner ? w.cm.x : w.cm.z, sh = inner ? w.cm.y : w.cm.w;
        int jn = (int)floorf(__fmul_rn(__fsub_rn(__fmaf_rn(rho, xj, sh), q.x0), q.inv_dx));
        jn = jn < 0 ? 0 : (jn > q.nb - 1 ? q.nb - 1 : jn);
        const int moved = x + (jn - j);   // x: the same bin of the neighbour
        const bool out = x == 63 || (unsigned)(jn - w.wj) >= (1u << w.b) || moved == 63;
        x = (inner ? w.id0 : w.id1) ? x : (out ? 63 : moved);
    }
    int n = e < w.shi ? f : x;
    if (SURR) n = stop_here ? 63 : n;
    p = (int)rl((uint32_t)n, p);
    post = write_lane(p, k, post);
}

template <bool MOVING, bool SURR, int G>
__device__ __forceinline__ void mix_from(const MixWindow &w, const Packet1D &q, bool rebins, uint32_t ew, float u,
                                         bool stop_even, bool stop_odd, int lane, int &p, int &post)
{
#pragma unroll
    for (int k = 0; k < 8; ++k)
        mix_step<MOVING, SURR>(w, q, rebins, 8 * G + k, ew, u, (k & 1) ? stop_odd : stop_even, lane, p, post);
    if constexpr (G < 7) {
        if (p != 63) mix_from<MOVING, SURR, G + 1>(w, q, rebins, ew, u, stop_even, stop_odd, lane, p, post);
    }
}

// The window's shape for the recent share of spatial leaks: a walk leaves a window of W cells
// and V bins after about W^2 / 4s or V^2 / 4f steps (s, f the shares of spatial and frequency
// steps), equal at V / W = sqrt(f / s); of the shapes V / W = 16, 4, 1, 1/4, 1/16 the nearest,
// no dimension more than needed to cover the grid.
__device__ __forceinline__ int mix_shape(const Packet1D &q, int nt, int ns)
{
    const int nf = nt - ns;
    int b = nf >= 64 * ns ? 5 : (nf >= 4 * ns ? 4 : (4 * nf >= ns ? 3 : (64 * nf >= ns ? 2 : 1)));
    while (b > 1 && (1 << (b - 1)) >= q.nb) --b;
    while (b < 5 && (32 >> b) >= q.nc) ++b;
    return b;
}

// One mixed block of up to 64 steps (at least 68 steps below the step cap).  Adds the block's
// steps and spatial leaks to `nt` and `ns`.
template <bool MOVING, bool SURR>
__device__ __forceinline__ void mix_block(Packet1D &q, int b, const SurrWin &sw, const float *__restrict__ recs,
                                          const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                                          const WalkArgs &a, unsigned long long *__restrict__ tally, int lane,
                                          int &nt, int &ns)
{
    MixWindow w;
    mix_load<MOVING>(w, q, b, lane);
    const bool mv = MOVING && q.moving;
    const StepWords wl = words_of_step<MOVING>(q, q.steps + (uint64_t)lane, a);
    const float u = __fmul_rn(__fadd_rn((float)(wl.z >> 8), 0.5f), 5.9604644775390625e-8f);   // as rebin_uniform
    bool stop_even = false, stop_odd = false;
    if (SURR) {   // surrogate exits: every step in moving media, even step counts in static ones
        const int i = w.wi + (lane >> b), j = w.wj + (lane & ((1 << b) - 1));
        const bool in = (unsigned)(i - sw.i_lo) <= (unsigned)(sw.i_hi - sw.i_lo) &&
                        (unsigned)(j - sw.j_lo) <= (unsigned)(sw.j_hi - sw.j_lo);
        stop_even = in && (mv || !(q.steps & 1ull));
        stop_odd = in && (mv || (q.steps & 1ull));
    }
    const int p0 = ((q.i - w.wi) << b) + (q.j - w.wj);
    int p = (int)rl((uint32_t)p0, 0), post = 63;
    if (mv)   // on a uniform grid (the caller's choice)
        mix_from<MOVING, SURR, 0>(w, q, true, wl.e, u, stop_even, stop_odd, lane, p, post);
    else
        mix_from<MOVING, SURR, 0>(w, q, false, wl.e, u, stop_even, stop_odd, lane, p, post);
    // lane k: the position step k starts from, and that state's record
    int pre = __shfl_up(post, 1);
    if (lane == 0) pre = p0;
    const uint32_t lk = (uint32_t)__shfl((int)w.lk, pre);
    const uint32_t dh = (uint32_t)__shfl((int)w.dhi, pre), sh = (uint32_t)__shfl((int)w.shi, pre);
    const uint32_t fh = (uint32_t)__shfl((int)w.fhi, pre);
    const bool tie = wl.e == dh || wl.e == sh || wl.e == fh;
    const uint64_t stops = __ballot(post == 63 || tie);
    const int done = stops ? __ffsll((unsigned long long)stops) - 1 : 64;
    const int pos = done < 64 ? (int)rl((uint32_t)pre, done) : (int)rl((uint32_t)post, 63);
    const double dd = lane < done ? (double)path_length(wl.t, __uint_as_float(lk)) : 0.0;
    double t = q.t;                    // the lane walk's FP64 additions, same bits
    if (done > 0 && !clock_parallel(t, dd))
        clock_from<0>(t, (uint32_t)__double_as_longlong(dd), (uint32_t)((uint64_t)__double_as_longlong(dd) >> 32), done);
    q.t = t;
    q.steps += (uint64_t)done;
    q.i = w.wi + (pos >> b);
    q.j = w.wj + (pos & ((1 << b) - 1));
    nt += done;
    ns += __popcll(__ballot(lane < done && wl.e >= sh));
    if (done == 64) return;
    // the step the block stopped at, taken by the whole wave with the lane walk's selects; a
    // surrogate exit, a tie or an escape runs in lane 0
    Packet1D s1 = q;
    bool exits = false;
    if (SURR) {
        const bool chk = mv || !(q.steps & 1ull);
        if (chk && in_window(q, sw)) {
            exits = true;
            if (lane == 0) surrogate_exit<MOVING>(s1, sw, recs, tb, clouds[s1.cl], a);
        }
    }
    if (!exits) {
        const StepWords ws = {rl(wl.t, done), rl(wl.e, done), rl(wl.z, done), rl(wl.w, done)};
        const uint4 rec = make_uint4(rl(w.lk, pos), rl(w.dhi, pos), rl(w.shi, pos), rl(w.fhi, pos));
        float4 cm = make_float4(1.f, 0.f, 1.f, 0.f);
        bool slow;
        int d;
        if (mv) {
            cm = make_float4(__uint_as_float(rl(__float_as_uint(w.cm.x), pos)),
                             __uint_as_float(rl(__float_as_uint(w.cm.y), pos)),
                             __uint_as_float(rl(__float_as_uint(w.cm.z), pos)),
                             __uint_as_float(rl(__float_as_uint(w.cm.w), pos)));
            slow = select_step_moving(s1, true, ws, rec, cm, clouds, tb);
        } else {
            slow = select_step(s1, true, ws.t, ws.e, rec, d);
        }
        ++nt;
        ns += ws.e >= rec.z ? 1 : 0;
        if (__any(slow)) {
            if (lane == 0) slow_step<MOVING>(s1, ws, rec, cm, tb, clouds, a, tally);
        }
    }
    take_lane0<SURR>(q, s1);
}

// The fields of four that hold 15, all others zero.
__device__ __forceinline__ uint32_t full_fields(uint32_t v)
{
    v &= v >> 1;
    v &= v >> 2;
    v &= 0x11111111u;
    return (v << 4) - v;
}

// Each of eight bits spread to a field of four.
__device__ __forceinline__ uint32_t nibbles(uint32_t m)
{
    m = (m | (m << 12)) & 0x000f000fu;
    m = (m | (m << 6)) & 0x03030303u;
    m = (m | (m << 3)) & 0x11111111u;
    return (m << 4) - m;
}

// With SUB the walk is a sub-walk: it ends with the first spatial leak, of which it returns the
// bin (-1 if the step cap came first), and tallies nothing.
template <bool MOVING, bool SURR, bool SUB>
__device__ int coop_walk(Packet1D &q, const uint8_t *__restrict__ tb, const DevCloud *__restrict__ clouds,
                         const WalkArgs &a, unsigned long long *__restrict__ tally, int lane)
{
    // the cloud's surrogate window: a step that starts in it is replaced by one exit, at the
    // same points as in the lane walk (every step in moving media, even step counts in
    // static media, and only with room for three more steps)
    SurrWin sw = kNoWindow;
    const float *recs = nullptr;
    if (SURR) {
        const SurrHeader *SH = reinterpret_cast<const SurrHeader *>(a.surr);
        recs = reinterpret_cast<const float *>(a.surr + SH->off_records);
        sw = surr_window(a.surr, q.cl);
    }
    int wi = -1, jb = 0;
    int short_run = 0;   // consecutive table blocks stopped by a slow-path step within 16 steps
    bool mixed = false;
    int nt = 0, ns = 0;  // recent steps and spatial leaks (mixed blocks)
    uint32_t v_lk = 0u, v_dhi = 0u, v_shi = 0u, v_fhi = 0u;
    int jw = 0;
    uint32_t w_dh[kCoopWin];   // the window's lower thresholds, halved
    while (q.active) {
        const uint64_t left = a.max_steps - q.steps;
        if (left == 0) {
            if (!SUB && lane == 0) tally_finish(tally, clouds[q.cl], false, 0, 0, q.t, q.steps);
            q.active = false;
            break;
        }
        if (mixed && left >= 68 && MOVING && q.moving && !q.uniform) {
            // re-binning on other grids searches the bin edges: lane 0 walks on alone for a while
            Packet1D s1 = q;
            const int n = left < 1024 ? (int)left : 1024;
            if (lane == 0) moving_steps<SURR>(s1, n, n, tb, clouds, a, tally, &sw, recs);
            take_lane0<SURR>(q, s1);
            mixed = false;
            continue;
        }
        if (mixed && left >= 68) {
            mix_block<MOVING, SURR>(q, mix_shape(q, nt, ns), sw, recs, tb, clouds, a, tally, lane, nt, ns);
            if (nt > 256) {   // forget older steps; back to table blocks where leaks are rare
                mixed = 64 * ns > nt;
                nt >>= 1;
                ns >>= 1;
            }
            continue;
        }
        // band of 64 bins around the packet (reloaded on a new cell or near its edges)
        const bool fresh = q.i != wi || (q.j - jb <= kCoopWin / 2 && jb > 0) ||
                           (q.j - jb > 63 - kCoopWin / 2 && jb < q.nb - 64);
        if (fresh) {
            jb = q.j - 32;
            if (jb > q.nb - 64) jb = q.nb - 64;
            if (jb < 0) jb = 0;
            wi = q.i;
            // bins beyond the grid: every event there is "slow" (never reached)
            v_lk = 0u;
            v_dhi = 0u;
            v_shi = 0u;
            v_fhi = 0u;
            if (jb + lane < q.nb) {
                const uint4 r = q.hot[q.i * q.nb + jb + lane];
                v_lk = r.x;
                v_dhi = r.y;
                v_shi = r.z;
                v_fhi = r.w;
            }
        }
        // The window stays where it is while the packet keeps off its edges.  A static walk pairs its
        // steps by count: the packet is at an even position of the window before the first of a pair.
        const bool mv = MOVING && q.moving;
        if (fresh || (unsigned)(q.j - jw - 5) > (unsigned)(kCoopWin - 11) || (!mv && ((q.j - jw) ^ (int)q.steps) & 1)) {
            jw = q.j - kCoopWin / 2;
            if (jw > jb + 64 - kCoopWin) jw = jb + 64 - kCoopWin;
            if (jw < jb) jw = jb;
            if (!mv && ((q.j - jw) ^ (int)q.steps) & 1) jw += jw == jb + 64 - kCoopWin ? 1 : -1;   // off the grid at most
#pragma unroll
            for (int b = 0; b < kCoopWin; ++b) w_dh[b] = rl(v_dhi, (jw - jb + b) & 63) >> 1;
        }
        const int wb = jw - jb;   // band lane of window position 0
        // each lane's two steps, from an even and an odd position; a packet at an odd one starts with
        // the second step of lane 0
        const int odd = (q.j - jw) & 1;
        StepWords wa, wc;
        if (mv) {
            wa = words_of_step<MOVING>(q, q.steps + 2ull * (uint64_t)lane - (uint64_t)odd, a);
            wc = words_of_step<MOVING>(q, q.steps + 2ull * (uint64_t)lane - (uint64_t)odd + 1ull, a);
        } else {
            const uint64_t pr = (q.steps >> 1) + (uint64_t)lane;
            const u32x4 r = philox4x32_10((uint32_t)pr, (uint32_t)(pr >> 32), q.pid, q.key, a.key0, a.key1);
            wa = StepWords{r.x, r.y, 0u, 0u};
            wc = StepWords{r.z, r.w, 0u, 0u};
        }
        const bool none = lane == 0 && odd != 0;   // the step taken before
        // bit m: the first step from position 2m, the second from 2m + 1 goes down (the sign of a
        // difference of halves; equal halves count as ties below)
        const uint32_t ea = wa.e >> 1, ec = wc.e >> 1;
        uint32_t da = 0u, dc = 0u;
#pragma unroll
        for (int m = kCoopWin / 2 - 1; m >= 0; --m) {
            da = __funnelshift_l(ea - w_dh[2 * m], da, 1);
            dc = __funnelshift_l(ec - w_dh[2 * m + 1], dc, 1);
        }
        // tables of next positions, one 4-bit field per position (15: out of the window).  The second
        // step leads from 2m + 1 to m or m + 1, both together from 2m to where the second leads from
        // 2 (m - 1) + 1 or 2m + 1
        const uint32_t da_lo = nibbles(da & 0xffu), da_hi = nibbles(da >> 8);
        const uint32_t dc_lo = nibbles(dc & 0xffu), dc_hi = nibbles(dc >> 8);
        const uint32_t b_lo = (0x76543210u & dc_lo) | (0x87654321u & ~dc_lo);
        const uint32_t b_hi = (0xfedcba98u & dc_hi) | (0xffedcba9u & ~dc_hi);
        uint32_t c_lo = ((b_lo << 4 | 0xfu) & da_lo) | (b_lo & ~da_lo);
        uint32_t c_hi = (__funnelshift_l(b_lo, b_hi, 4) & da_hi) | (b_hi & ~da_hi) | 0xf0000000u;
        if (none) {
            c_lo = b_lo;
            c_hi = b_hi;
        }
        // even lanes: the table of four steps (this lane's, then the next lane's): the two steps of a
        // lane go one field down, nowhere or one up; the one step of `none` nowhere or up
        const uint32_t n_lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c_lo, 0xf5, 0xf, 0xf, false);
        const uint32_t n_hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c_hi, 0xf5, 0xf, 0xf, false);
        const uint32_t dd_lo = none ? 0u : da_lo & (dc_lo << 4);
        const uint32_t dd_hi = none ? 0u : da_hi & __funnelshift_l(dc_lo, dc_hi, 4);
        const uint32_t uu_lo = ~((none ? 0u : da_lo) | dc_lo), uu_hi = ~((none ? 0u : da_hi) | dc_hi);
        uint32_t f_lo = ((n_lo << 4) & dd_lo) | (__funnelshift_r(n_lo, n_hi, 4) & uu_lo) | (n_lo & ~(dd_lo | uu_lo));
        uint32_t f_hi = (__funnelshift_l(n_lo, n_hi, 4) & dd_hi) | ((n_hi >> 4) & uu_hi) | (n_hi & ~(dd_hi | uu_hi));
        f_lo |= full_fields(c_lo);
        f_hi |= full_fields(c_hi);
        // sequential part: the chain of positions, in scalar registers, four steps at a time
        uint32_t st = rl(kScanWidth | ((uint32_t)(q.j - jw) >> 1 << 2), 0);
        int vst = (int)kScanStop;
        scan_from<0>(st, vst, f_lo, f_hi);
        // each lane's starting position (odd lanes: two steps from the even lane before); what its
        // steps do there
        const uint32_t p4 = (uint32_t)vst & 63u;
        const uint32_t after = (p4 < 32u ? c_lo >> p4 : c_hi >> (p4 - 32u)) & 15u;
        const uint32_t from_even = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)after, 0xa0, 0xf, 0xf, false);
        const int ma = (lane & 1) ? (int)from_even : (int)(p4 >> 2);
        const int mc = ma - (none ? 0 : (int)((da >> ma) & 1u));
        const int pa = 2 * ma, pc = 2 * mc + 1;
        const int pd = pc + 1 - 2 * (int)((dc >> (mc & 31)) & 1u);
        const int la = (wb + pa) & 63, lc = (wb + pc) & 63;
        const uint32_t lk_a = (uint32_t)__shfl((int)v_lk, la), lk_c = (uint32_t)__shfl((int)v_lk, lc);
        const uint32_t dh_a = (uint32_t)__shfl((int)v_dhi, la), dh_c = (uint32_t)__shfl((int)v_dhi, lc);
        const uint32_t sh_a = (uint32_t)__shfl((int)v_shi, la), sh_c = (uint32_t)__shfl((int)v_shi, lc);
        // stops: leaks, ties, surrogate exits, the step cap
        bool slow_a = !none && (wa.e >= sh_a || ea == dh_a >> 1), slow_c = wc.e >= sh_c || ec == dh_c >> 1;
        bool exit_a = false, exit_c = false;
        if (SURR && (unsigned)(q.i - sw.i_lo) <= (unsigned)(sw.i_hi - sw.i_lo)) {
            const uint64_t k = 2ull * (uint64_t)lane - (uint64_t)odd;
            exit_a = !none && k + 3ull <= left && (unsigned)(jw + pa - sw.j_lo) <= (unsigned)(sw.j_hi - sw.j_lo);
            exit_c = mv && k + 4ull <= left && (unsigned)(jw + pc - sw.j_lo) <= (unsigned)(sw.j_hi - sw.j_lo);
            slow_a |= exit_a;
            slow_c |= exit_c;
        }
        if (left < 128ull) {
            slow_a |= 2 * lane - odd >= (int)left;
            slow_c |= 2 * lane + 1 - odd >= (int)left;
        }
        const bool end_a = slow_a || (unsigned)pc >= (unsigned)kCoopWin;
        const bool end_c = slow_c || (unsigned)pd >= (unsigned)kCoopWin;
        // the first step that stops: one that leaves the window is done, any other is not
        const uint64_t sb = __ballot(ma != 15 && (end_a || end_c));
        int done = 128, pos = (int)((st & 63u) >> 1);
        bool special = false, surr_stop = false;
        StepWords ws = {0u, 0u, 0u, 0u};
        if (sb) {
            const int ls = __ffsll((unsigned long long)sb) - 1;
            const uint32_t kind = (end_a ? 0u : 1u) | ((end_a ? slow_a : slow_c) ? 2u : 0u) |
                                  ((end_a ? exit_a : exit_c) ? 4u : 0u);
            const uint32_t kd = rl(kind, ls);
            special = (kd & 2u) != 0u;
            done = 2 * ls + (int)(kd & 1u) + (special ? 0 : 1);
            pos = (int)rl((uint32_t)(special ? (end_a ? pa : pc) : (end_a ? pc : pd)), ls);
            surr_stop = SURR && (kd & 4u) != 0u;
            if (special) {
                ws.t = (kd & 1u) ? rl(wc.t, ls) : rl(wa.t, ls);
                ws.e = (kd & 1u) ? rl(wc.e, ls) : rl(wa.e, ls);
                ws.z = (kd & 1u) ? rl(wc.z, ls) : rl(wa.z, ls);
                ws.w = (kd & 1u) ? rl(wc.w, ls) : rl(wa.w, ls);
            }
        }
        const double ta = 2 * lane < done && !none ? (double)path_length(wa.t, __uint_as_float(lk_a)) : 0.0;
        const double tc = 2 * lane + 1 < done ? (double)path_length(wc.t, __uint_as_float(lk_c)) : 0.0;
        double t = q.t;                    // the lane walk's FP64 additions, same bits
        if (!clock_parallel(t, ta, tc)) {
            for (int l = 0; 2 * l < done; ++l) {
                t += rl_f64(ta, l);
                t += rl_f64(tc, l);
            }
        }
        done -= odd;
        special = special && (uint64_t)done < left;
        q.t = t;
        q.steps += (uint64_t)done;
        const int jj = jw + pos;
        q.j = jj;
        short_run = special && done < 16 ? short_run + 1 : 0;
        if (special) {
            // the step at `done` in lane 0 with the lane walk's arithmetic; several blocks in a
            // row that stopped early (spatial leaks are frequent here) hand over to mixed blocks
            const int b = (jj - jb) & 63;
            const uint4 rec = make_uint4(rl(v_lk, b), rl(v_dhi, b), rl(v_shi, b), rl(v_fhi, b));
            Packet1D s1 = q;
            if (lane == 0 && SURR && surr_stop) {
                surrogate_exit<MOVING>(s1, sw, recs, tb, clouds[s1.cl], a);
            } else if (lane == 0) {
                const float4 cm = (MOVING && s1.moving) ? s1.cmap[s1.i] : make_float4(1.f, 0.f, 1.f, 0.f);
                one_step<MOVING>(s1, ws, rec, cm, tb, clouds, a, tally);
            }
            const int i0 = q.i;
            take_lane0<SURR>(q, s1);
            if (SUB && q.i != i0) return jj;
            if (!SUB && short_run >= 2) {
                mixed = true;
                short_run = 0;
                wi = -1;
                nt = 64;
                ns = 8;
            }
        }
    }
    if (SURR && lane == 0 && q.surr_calls)
        atomicAdd(&tally[clouds[q.cl].tally_off + TW_SURR_CALLS], (unsigned long long)q.surr_calls);
    return -1;
}

template <bool MOVING, bool SURR>
__global__ __launch_bounds__(64) void walk1d_coop(const uint8_t *__restrict__ tb, WalkArgs a,
                                                  unsigned long long *__restrict__ tally,
                                                  unsigned long long *__restrict__ work)
{
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    const int lane = threadIdx.x & 63;
    const uint64_t n = work[kWGiven] < a.tail_capacity ? work[kWGiven] : a.tail_capacity;
    TailPacket *slots = slots_of(work);
    for (;;) {   // the packets still published once the lane-walk launch has ended
        uint64_t idx = 0;
        if (lane == 0) idx = atomicAdd(&work[kWSweep], 1ull);
        idx = shfl_u64(idx, 0);
        if (idx >= n) break;
        uint32_t got = 0u;
        if (lane == 0) {
            uint32_t expect = kSlotReady;
            got = __hip_atomic_compare_exchange_strong(&slots[idx].flag, &expect, kSlotTaken, __ATOMIC_ACQ_REL,
                                                       __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT)
                      ? 1u
                      : 0u;
        }
        if (rl(got, 0) == 0u) continue;
        Packet1D q = load_slot(slots + idx, tb, clouds);
        coop_walk<MOVING, SURR>(q, tb, clouds, a, tally, lane);
    }
}

// An event whose word ties with the high word of a threshold, decided by the full u64 with the
// low word of the step's auxiliary block: 0 / 1 a lower / upper bin, 2 / 3 a leak through face 0 / 1.
__device__ int tied_event(const Packet1D &p, uint32_t ew, uint4 rec, const uint8_t *__restrict__ tb, const DevCloud &c,
                          const WalkArgs &a)
{
    const u32x4 aux = philox4x32_10((uint32_t)p.steps, kDomAux | (uint32_t)(p.steps >> 32), p.pid, p.key, a.key0,
                                    a.key1);
    const uint4 lw = reinterpret_cast<const uint4 *>(tb + c.off_lo_words)[p.i * p.nb + p.j];
    const uint64_t U = ((uint64_t)ew << 32) | aux.x;
    if (U < (((uint64_t)rec.y << 32) | lw.x)) return 0;
    if (U < (((uint64_t)rec.z << 32) | lw.y)) return 1;
    return U < (((uint64_t)rec.w << 32) | lw.z) ? 2 : 3;
}

// Live lanes of a sub-walk wave at which it turns to walking them one by one: a side-by-side step
// of the whole wave costs as much issue as ~14 cooperative ones (a lone lane 0.75 us per step, a
// cooperative packet ~0.04).
constexpr int kSubTail = 14;

// Sub-walks for the surrogate's training data: sample q starts in state s_state[q] of
// cloud s_cloud[q] (a cell with two neighbours) and takes DDMC steps until its first
// spatial leak.  Writes the state's features X[q, 16] and the exit Y[q] = (face, y1, y2),
// face -1 when max_steps ran out first, and the number of steps.
template <bool MOVING>
__global__ __launch_bounds__(256) void subwalk1d(const uint8_t *__restrict__ tb, WalkArgs a,
                                                 const int32_t *__restrict__ s_cloud,
                                                 const int32_t *__restrict__ s_state, int64_t n, int per_wave,
                                                 float *__restrict__ X, float *__restrict__ Y,
                                                 unsigned long long *__restrict__ steps_out)
{
    const int lane = threadIdx.x & 63;
    int64_t q = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per_wave + lane;
    const bool mine = lane < per_wave && q < n;
    if (!mine) q = n - 1;
    const DevHeader *H = reinterpret_cast<const DevHeader *>(tb);
    const DevCloud *clouds = reinterpret_cast<const DevCloud *>(tb + H->off_clouds);
    Packet1D p;
    p.cl = s_cloud[q];
    const DevCloud &c = clouds[p.cl];
    set_cloud(p, tb, c);
    p.pid = (uint32_t)q;
    p.i = s_state[q] / c.nb;
    p.j = s_state[q] - p.i * c.nb;
    p.t = 0.0;
    p.steps = 0;
    p.active = mine;
    p.surr_calls = 0u;
    float f[kSurrIn], S, w;
    surr_features(c, tb, p.i, p.j, f, S, w);
    if (mine)
        for (int k = 0; k < kSurrIn; ++k) X[q * kSurrIn + k] = f[k];
    int face = -1, jexit = p.j;
    // lanes walk side by side until few are left ...
    while (__popcll(__ballot(p.active)) > kSubTail) {
        for (int k = 0; k < 32; ++k) {
            if (p.active) {
                const uint4 rec = p.hot[p.i * p.nb + p.j];
                const StepWords w = words_of_step<MOVING>(p, p.steps, a);
                p.t += (double)path_length(w.t, __uint_as_float(rec.x));
                int ev = w.e < rec.y ? 0 : (w.e < rec.z ? 1 : (w.e < rec.w ? 2 : 3));   // bins -, +, faces 0, 1
                if (w.e == rec.y || w.e == rec.z || w.e == rec.w) ev = tied_event(p, w.e, rec, tb, c, a);
                ++p.steps;
                if (ev >= 2) {
                    face = ev - 2;
                    jexit = p.j;
                }
                p.j += ev == 0 ? -1 : (ev == 1 ? 1 : 0);
                p.active = ev < 2 && p.steps < a.max_steps;
            }
        }
    }
    // ... and the wave takes those one after another, cooperatively
    for (uint64_t left = __ballot(p.active); left;) {
        const int l = __ffsll((unsigned long long)left) - 1;
        left &= left - 1ull;
        Packet1D u;   // that lane's packet, the same in every lane
        u.active = true;
        u.surr_calls = 0u;
        u.cl = (int)rl((uint32_t)p.cl, l);
        u.pid = rl(p.pid, l);
        u.i = (int)rl((uint32_t)p.i, l);
        u.j = (int)rl((uint32_t)p.j, l);
        u.steps = ((uint64_t)rl((uint32_t)(p.steps >> 32), l) << 32) | rl((uint32_t)p.steps, l);
        u.t = rl_f64(p.t, l);
        set_cloud(u, tb, clouds[u.cl]);
        const int i0 = u.i;
        const int j = coop_walk<MOVING, false, true>(u, tb, clouds, a, nullptr, lane);
        if (lane == l) {
            p.t = u.t;
            p.steps = u.steps;
            if (j >= 0) {   // a walk the cap cut keeps its entry bin, as one cut side by side
                face = u.i > i0 ? 1 : 0;
                jexit = j;
            }
        }
    }
    if (!mine) return;
    const double *e = reinterpret_cast<const double *>(tb + c.off_edges);
    const u32x4 r = philox4x32_10((uint32_t)q, kDomSub | (uint32_t)((uint64_t)q >> 32), p.pid, p.key, a.key0, a.key1);
    const double xo = e[jexit] + (e[jexit + 1] - e[jexit]) * u01_open_low(r.x);
    Y[3 * q] = (float)face;
    Y[3 * q + 1] = (float)asinh(xo / (double)S);
    Y[3 * q + 2] = (float)log(p.t / (double)w);
    steps_out[q] = p.steps;
}

__global__ void philox_fill_kernel(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                                   uint32_t c3, uint64_t n, uint32_t *out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const u32x4 r = philox4x32_10(c0 + (uint32_t)i, c1, c2, c3, k0, k1);
    out[4 * i + 0] = r.x;
    out[4 * i + 1] = r.y;
    out[4 * i + 2] = r.z;
    out[4 * i + 3] = r.w;
}

// Clears the counters and every export slot's flag (a kernel, so that the call can be
// captured in a graph).
__global__ void reset_work(unsigned long long *work, uint64_t capacity)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kWorkHeaderBytes / 8) work[i] = 0ull;
    if (i < capacity) slots_of(work)[i].flag = kSlotEmpty;
}

}  // namespace

int device_cu_count()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
    return n > 0 ? n : 256;
}

hipError_t launch_walk(const uint8_t *d_tables, const DevHeader &h, const DevCloud *host_clouds,
                       const rddmc_run &run, uint64_t first, uint64_t count,
                       unsigned long long *d_tally, unsigned long long *d_work, uint64_t work_bytes,
                       hipStream_t s)
{
    WalkArgs a;
    a.first = first;
    a.count = count;
    a.max_steps = run.max_steps;
    a.key0 = (uint32_t)run.seed;
    a.key1 = (uint32_t)(run.seed >> 32);
    // in pairs of steps; bounded, so that neither the pairs of the largest chunk nor their steps leave an int
    a.chunk = run.chunk > 0 ? (int)((std::min<int64_t>(run.chunk, 1 << 21) + 1) / 2) : 32;
    a.n_clouds = h.n_clouds;
    a.tail_lanes = run.tail_lanes < 0 ? 0 : run.tail_lanes;
    a.tail_capacity = work_bytes > kWorkHeaderBytes ? (work_bytes - kWorkHeaderBytes) / sizeof(TailPacket) : 0;
    if (a.tail_capacity == 0) a.tail_lanes = 0;
    a.one_round = 0;
    const int block = run.block > 0 ? run.block : 256;
    uint64_t grid = run.grid > 0 ? (uint64_t)run.grid : 0;
    if (grid == 0) {
        const uint64_t want = (count + block - 1) / block;
        const uint64_t cap = (uint64_t)device_cu_count() * 8;   // 8 blocks of 256 per CU
        grid = want < cap ? want : cap;
        if (grid < 1) grid = 1;
    }
    const uint64_t lanes = grid * (uint64_t)block;
    a.share = 0;
    if (run.tail_lanes == 0 && a.tail_capacity > 0) {
        // A SIMD's issue slots take a lane walk one step per live lane in ~500 cycles and a cooperative
        // walk one step in 50-60, however many waves share it: a wave's packets all leave once ten or
        // so are left.  8 from four waves per SIMD on (2^20 packets of the efficient-grid tau0 = 1e7 sphere:
        // 109 ms, 120 at 16), 16 below two, whose last packets wait on latency (2^16 packets of moving
        // spheres: 108 ms, 115 at 8), 12 between (2^17 packets of a moving 6 x 131 sphere: 279 ms, 326 at 8, 261
        // at 16; the efficient-grid sphere there 3 % slower than at 8).  SIMDs without a producer wave work cooperatively from the start, on
        // up to four packets each, handed over as consumers become free (2^14 packets of the tau0 = 1e5
        // slab, 256 producer waves, with the table blocks of that time: 626 ms, 1006 at 16 alone, 675 at
        // 64 per wave; 530 ms with the present ones).
        const uint64_t simds = 4ull * (uint64_t)device_cu_count(), waves = (lanes + 63) / 64;
        a.tail_lanes = waves >= 4 * simds ? 8 : (waves >= 2 * simds ? 12 : 16);
        a.share = waves < simds ? (int)(4 * (simds - waves)) : 0;
    }
    a.one_round = queue_in_one_round(grid * (uint64_t)(block / 64), 64, count, (uint64_t)device_cu_count()) ? 1 : 0;
    a.ahead = (lanes + 63) / 64 <= 8ull * (uint64_t)device_cu_count() ? 1 : 0;
    if (a.tail_lanes > 0 && (lanes < count ? lanes : count) > a.tail_capacity) {
        // every exported packet (at most one per lane, at most `count`) needs a slot
        grid = a.tail_capacity / block;
        if (grid < 1) {
            grid = 1;
            a.tail_lanes = 0;
        }
        a.one_round = queue_in_one_round(grid * (uint64_t)(block / 64), 64, count, (uint64_t)device_cu_count()) ? 1 : 0;
    }
    bool moving = false;
    for (int c = 0; c < h.n_clouds; ++c) moving |= host_clouds[c].rebins != 0u;
    a.surr = static_cast<const uint8_t *>(run.surrogate);
    a.producer_blocks = (uint32_t)grid;
    a.producer_waves = (uint32_t)(grid * (uint64_t)(block / 64));
    // consumer blocks after the producers: 16 waves per CU walk handed-over packets as soon
    // as lane-walk blocks finish and free their slots
    const uint64_t consumers = a.tail_lanes > 0 ? ((uint64_t)device_cu_count() * 16 * 64 + block - 1) / block : 0;
    a.consumer_waves = (uint32_t)(consumers * (uint64_t)(block / 64));
    {
        const uint64_t n = a.tail_capacity > kWorkHeaderBytes / 8 ? a.tail_capacity : kWorkHeaderBytes / 8;
        reset_work<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(d_work, a.tail_capacity);
    }
    grid += consumers;
    if (moving && a.surr)
        walk1d<true, true><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
    else if (moving)
        walk1d<true, false><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
    else if (a.surr)
        walk1d<false, true><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
    else
        walk1d<false, false><<<(unsigned)grid, block, 0, s>>>(d_tables, a, d_tally, d_work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.tail_lanes == 0) return e;
    const unsigned cgrid = (unsigned)device_cu_count() * 16;   // one wave per block
    if (moving && a.surr)
        walk1d_coop<true, true><<<cgrid, 64, 0, s>>>(d_tables, a, d_tally, d_work);
    else if (moving)
        walk1d_coop<true, false><<<cgrid, 64, 0, s>>>(d_tables, a, d_tally, d_work);
    else if (a.surr)
        walk1d_coop<false, true><<<cgrid, 64, 0, s>>>(d_tables, a, d_tally, d_work);
    else
        walk1d_coop<false, false><<<cgrid, 64, 0, s>>>(d_tables, a, d_tally, d_work);
    return hipGetLastError();
}

hipError_t launch_subwalk(const uint8_t *d_tables, bool moving, uint64_t seed, uint64_t max_steps,
                          const int32_t *d_cloud, const int32_t *d_state, int64_t n, float *d_x, float *d_y,
                          unsigned long long *d_steps, hipStream_t s)
{
    WalkArgs a{};
    a.max_steps = max_steps;
    a.key0 = (uint32_t)seed;
    a.key1 = (uint32_t)(seed >> 32);
    // as many waves as fill the device four times over before a wave takes more than a few samples:
    // the last of them are walked one after another (13 320 samples of 35 000 steps: 414 ms at 64
    // per wave, 107 spread out)
    const int64_t fill = 16ll * device_cu_count();
    const int64_t per = (n + fill - 1) / fill;
    const int per_wave = per < 4 ? 4 : (per > 64 ? 64 : (int)per);
    const int64_t waves = (n + per_wave - 1) / per_wave;
    const unsigned grid = (unsigned)((waves + 3) / 4);
    if (moving)
        subwalk1d<true><<<grid, 256, 0, s>>>(d_tables, a, d_cloud, d_state, n, per_wave, d_x, d_y, d_steps);
    else
        subwalk1d<false><<<grid, 256, 0, s>>>(d_tables, a, d_cloud, d_state, n, per_wave, d_x, d_y, d_steps);
    return hipGetLastError();
}

hipError_t launch_philox_fill(uint32_t k0, uint32_t k1, uint32_t c0, uint32_t c1, uint32_t c2,
                              uint32_t c3, uint64_t n, uint32_t *d_out, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    philox_fill_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(k0, k1, c0, c1, c2, c3, n, d_out);
    return hipGetLastError();
}

}  // namespace rddmc
