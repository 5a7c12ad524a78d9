// kt_trace.hip -- gfx950 kernels of the Kerr backward ray tracer.
//
// trace_kernel<METHOD>: one ray per lane.  Each lane holds its ray's state
// (r, theta, phi, p_r, p_theta), its constants (E, L) and its step control in
// VGPRs and advances one integrator step per loop iteration; all busy lanes
// of a wave evaluate the six (DP45) or four (RK4) right-hand sides together.
// When a ray ends, the lane writes that ray's outputs and takes the next
// slot from its wave's queue, a contiguous range of slots that the wave
// refills in batches from a global atomic ticket (persistent mode).  A slot
// names a ray through the dispatch order (ring first: rays near the photon
// ring, which take the most steps, go out first), through the compacted list
// of the FP64 re-run pass, or directly.  A wave exits once the ticket has
// passed the last slot and all its lanes are idle.
//
// Event location (disk plane, source sphere) reuses the same loop: a lane in
// LOCATE mode takes trial steps of size h' from the step's start state, so
// trial steps run in lockstep with other lanes' ordinary steps.
#include <hip/hip_runtime.h>

#include "kt_device.h"
#include "kt_internal.h"
#include "kt_ray.h"
#include "kt_sort.h"

// The file is compiled twice.  As itself it defines every kernel of the
// render in namespace kt, with the trace kernels built for 2 waves per SIMD.
// kt_trace_w3.hip includes it again with KT_TRACE_ONLY set: only the trace
// kernels and their launchers, in namespace kt_w3, built for 3 waves per SIMD
// and compiled without machine loop-invariant code motion (see there).
#ifndef KT_WAVES_PER_EU
#define KT_WAVES_PER_EU 2
#endif
#ifndef KT_TRACE_NS
#define KT_TRACE_NS kt
#endif
#ifndef KT_TRACE_ONLY
#define KT_TRACE_ONLY 0
#endif

namespace KT_TRACE_NS {
using namespace kt;

// Great-circle angle between the directions (theta1, phi1) and
// (theta2, phi1 + dphi), given sin/cos of the thetas: atan2(|n1 x n2|, n1.n2).
__device__ __forceinline__ double arc_angle(double s1, double c1, double s2, double c2, double dphi) {
    double sd, cd;
    sincos_fast(dphi, &sd, &cd);
    // frame rotated so that phi1 = 0: n1 = (s1, 0, c1), n2 = (s2 cd, s2 sd, c2)
    const double cx = -c1 * s2 * sd;
    const double cy = fma(c1 * s2, cd, -s1 * c2);
    const double cz = s1 * s2 * sd;
    const double cr = sqrt(fma(cx, cx, fma(cy, cy, cz * cz)));
    const double dt = fma(s1 * s2, cd, c1 * c2);
    return atan2_upper(cr, dt);
}

// The same angle for the short arcs of single steps: 2 asin(|n2 - n1| / 2)
// with the small-angle series, where
// |n2 - n1|^2 = (s2 - s1)^2 + (c2 - c1)^2 + 4 s1 s2 sin^2(dphi / 2).
// *in_range is false when the arc is outside the range of the series
// (|dphi| > 1/2 or chord/2 > 1/16); the caller then takes arc_angle.
__device__ __forceinline__ double arc_angle_short(double s1, double c1, double s2, double c2, double dphi,
                                                  bool* in_range) {
    // sin x, |x| <= 1/4, through x^11 (truncation below 1e-17 relative)
    const double x = 0.5 * dphi, x2 = x * x;
    double p = -1.0 / 39916800.0;
    p = fma_k(p, x2, 1.0 / 362880.0);
    p = fma_k(p, x2, -1.0 / 5040.0);
    p = fma_k(p, x2, 1.0 / 120.0);
    p = fma_k(p, x2, -1.0 / 6.0);
    const double sh = fma(p * x2, x, x);
    const double ds = s2 - s1, dc = c2 - c1;
    const double q = (4.0 * s1) * s2;
    const double h = 0.5 * sqrt_fast(fma(q * sh, sh, fma(ds, ds, dc * dc)));
    *in_range = (fabs(dphi) <= 0.5) & (h <= 0.0625);
    return 2.0 * asin_small(h);
}

// Celestial-sphere code of the direction (theta, phi) (Sect. 4.1).  theta is
// folded into [0, pi] (past the polar axis a ray continues on the meridian
// phi + pi) and phi into [0, 2 pi); then the graticule test (distance to the
// nearest multiple of grid_deg in either angle) and the quadrant.
__device__ __forceinline__ uint8_t sky_code(double th, double ph, double grid_deg, double line_deg) {
    constexpr double PI = 3.14159265358979323846, TWO_PI = 6.28318530717958647692;
    constexpr double DEG = 180.0 / PI;
    double t = th - TWO_PI * floor(th * (1.0 / TWO_PI));
    if (t > PI) {
        t = TWO_PI - t;
        ph += PI;
    }
    double p = ph - TWO_PI * floor(ph * (1.0 / TWO_PI));
    if (p >= TWO_PI) p -= TWO_PI;
    if (grid_deg > 0.0) {
        const double td = t * DEG, pd = p * DEG;
        const double dt = fabs(td - grid_deg * rint(td / grid_deg));
        const double dp = fabs(pd - grid_deg * rint(pd / grid_deg));
        if (dt <= line_deg || dp <= line_deg) return KT_SKY_LINE;
    }
    if (t < HALF_PI) return p < PI ? KT_SKY_GREEN : KT_SKY_RED;
    return p < PI ? KT_SKY_BLUE : KT_SKY_YELLOW;
}

// Index of the image that ray id `ray` belongs to (binary search over the
// images' first ray ids).
__device__ __forceinline__ int find_image(const Params& P, int64_t ray) {
    int lo = 0, hi = P.n_images - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (P.images[mid].first <= ray)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The cold parameters, in constant address space so that uniform reads are
// scalar loads (the copy is written before the launch and not during it).
// The empty asm keeps the compiler from moving those loads out of the rare
// paths that need them into scalar registers that live across the step loop.
__device__ __forceinline__ const Params& cold_params(const Params* p) {
    using Const = const __attribute__((address_space(4))) Params;
    Const* q = (Const*)p;
    asm volatile("" : "+s"(q));
    return *(const Params*)q;
}

// The per-image values the step loop needs.  For a single image they come
// from kernel arguments (wave-uniform); for a batch they are loaded per ray.
// The radii of events are read where an event is looked at: event_radii.
struct LaneImg {
    Spacetime st;
    int32_t feat;  // FEAT_* bits
    int32_t k;     // image index
};

__device__ __forceinline__ LaneImg lane_img(const Image& im, int k) {
    LaneImg li;
    li.st = Spacetime{im.M, im.a, im.a2, im.two_a2};
    li.feat = image_features(im);
    li.k = k;
    return li;
}

struct Radii {
    double r_cap, r_esc, r_src, r_in, r_out;
};

template <bool BATCH>
__device__ __forceinline__ Radii event_radii(const Params* cold, int k) {
    const Params& P = cold_params(cold);
    const Image& im = BATCH ? P.images[k] : P.img0;
    return Radii{im.r_cap, im.r_esc, im.r_src, im.r_in, im.r_out};
}

// Lane flags, packed in one int.
enum : int {
    F_LOCATE = 1 << 2,    // taking trial steps to locate an event
    F_RETAKE = 1 << 4,    // re-taking an accepted step after locating an event in it
    F_SKIPDISK = 1 << 5,  // disk crossing of the re-taken step already handled
    F_SRCDONE = 1 << 6,   // source sphere crossed
    F_EVSRC = 1 << 7,     // event being located is the source sphere
    F_USED32 = 1 << 24,   // mixed pass: some step used the FP32 mass part
    F_EVESC = 1 << 25,    // event being located is the celestial sphere
    F_EV32 = 1 << 26,     // mixed pass: the step whose event is being located (and
                          // then retaken) ran with the FP32 mass part
};
constexpr int NCROSS_SHIFT = 8;   // 8 bits: equatorial crossings outside the disk
constexpr int EVIT_SHIFT = 16;    // 8 bits: trial steps of the current event

// Per-lane state that only events touch lives in LDS, laid out
// [field][thread] so a wave's accesses are consecutive words: the size of
// the step an event lies in, the regula falsi's bracket, and once the source
// sphere is crossed the deflection and the angle to the source.
enum : int { C_H = 0, C_EVA, C_EVFA, C_EVB, C_EVFB, C_DEFL, C_SRCPSI, C_LAM, C_SWEPT, C_MAXH2, C_RELK, C_RELD, N_COLD };
// METRIC_SCHWARZSCHILD is Kerr with a = 0: single images by DP45 in FP64.
enum : int { METRIC_KERR = KT_METRIC_KERR, METRIC_Q = KT_METRIC_Q, METRIC_SCHWARZSCHILD = 2 };
constexpr int BLOCK_MAX = 256;

template <int METHOD, class ST, class EL>
__device__ __forceinline__ void take_step(const ST& st, const RayConst& rc, const double y[5],
                                          const double k1[5], double s0, double c0, double h, double yn[5],
                                          double kn[5], double er[5], Diag* dg, const EL& el) {
    if constexpr (METHOD == KT_DP45) {
        dp45_step(st, rc, y, k1, s0, c0, h, yn, kn, er, dg, nullptr, el);
    } else if constexpr (METHOD == KT_RKF45) {
        erk6_step<Fehlberg45>(st, rc, y, k1, s0, c0, h, yn, kn, er, dg, el);
    } else if constexpr (METHOD == KT_CK45) {
        erk6_step<CashKarp45>(st, rc, y, k1, s0, c0, h, yn, kn, er, dg, el);
    } else if constexpr (METHOD == KT_BS) {
        bs_step<false>(st, rc, y, k1, h, yn, kn, er, dg, el);
    } else if constexpr (METHOD == KT_BS_RAT) {
        bs_step<true>(st, rc, y, k1, h, yn, kn, er, dg, el);
    } else {
        rk4s_step(st, rc, y, k1, h, yn, kn, dg, el);
#pragma unroll
        for (int i = 0; i < 5; ++i) er[i] = 0.0;
    }
}

// A value that is the same in all lanes, in a scalar register.
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}

// The number of lanes below this one in a mask of the wave.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// The sum over the wave's lanes (all of them active), lane by lane: run once
// at a wave's end, where shuffles would hold their address registers through
// the step loop.
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
    unsigned long long sum = 0ull;
    for (int l = 0; l < 64; ++l) {
        const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
        const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), l));
        sum += (static_cast<unsigned long long>(hi) << 32) | lo;
    }
    return sum;
}

// max(|a|, |b|) in one instruction (fmax makes each operand canonical first,
// a vector instruction apiece); the other operand where one is NaN.
__device__ __forceinline__ double max_abs(double a, double b) {
    double r;
    asm("v_max_f64 %0, |%1|, |%2|" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// A ray's state (r, theta, phi, p_r, p_theta), or the field, as it is kept
// across steps: named members, so that each lives in a register pair of its
// own.  (An array that lives across the loop becomes one 16-register vector,
// three pairs of it unused and all of it copied at every commit.)
struct Vec5 {
    double r, th, ph, pr, pth;
    static __device__ __forceinline__ Vec5 of(const double z[5]) { return Vec5{z[0], z[1], z[2], z[3], z[4]}; }
    __device__ __forceinline__ void to(double z[5]) const {
        z[0] = r;
        z[1] = th;
        z[2] = ph;
        z[3] = pr;
        z[4] = pth;
    }
};

// STORE: the end of a ray that took more steps than its forward render.  It
// and the rays that end without a step or out of their budget are left to the
// one-lane path (status ADJ_OVERFLOW), whose budget is one of attempts alone
// and whose word on failures is the one that counts.
constexpr int FATE_NO_ROOM = 8;
constexpr uint32_t NO_RECORD = 0xffffffffu;

// The running maxima of |2H| and of |H|_rel = Kabs / D, the latter as its two
// parts (ratios compared by cross products): no quotient per step.  Inside the
// horizon, where a ray of a fixed step or without a capture buffer gets to, D may
// be negative; rel_k carries the ratio's sign, so that the cross products compare
// the ratios themselves there too (SIGNED; the q-metric's terms are positive).
template <bool SIGNED>
__device__ __forceinline__ void keep_max(const Diag& dg, double* max_h2, double* rel_k, double* rel_d) {
    *max_h2 = max_abs(dg.H2, *max_h2);
    if (dg.Kabs * (SIGNED ? fabs(*rel_d) : *rel_d) > *rel_k * dg.D) {
        *rel_k = SIGNED ? __builtin_copysign(dg.Kabs, dg.D) : dg.Kabs;
        *rel_d = dg.D;
    }
}

// STORE: the backward sweeps, a step VJP per iteration from the step's entry in
// the store (the next one's is fetched meanwhile).  First launch: a wave with no
// forward ray left sweeps the rays that its own lanes stored, longest first, while
// other waves still run the longest rays' forward passes, chains of up to 1700
// steps that keep few lanes busy (512x512 fit: 2.9 ms for 0.8 ms of work, and 2.0
// ms of sweeps after it).  A lane reads only what it has written itself, so
// nothing has to be waited for.  Once no wave has a forward ray, the rest of the
// work is dealt out anew: what a lane has left it puts on a list, also the middle
// of a sweep, and the second launch's lanes take that list's sweeps and the split
// rays' segment items from a ticket.  Both launches run this one loop, so the
// gradients do not depend on where a sweep was cut.
//
// Bound by the FP64 vector issue rate: ~1300 vector instructions per step of
// a wave, 40 bytes read per lane and step.
__device__ __forceinline__ void sweep(const Hot& hp, uint32_t own) {
    const AdjStore& A = cold_params(hp.cold).adj;
    const double M = hp.M, a = hp.a;
    const bool second = hp.sweep_only != 0;
    const bool overlap = uniform(A.counters[ADJ_C_OVERLAP]) != 0u;
    if (!second && !overlap) return;
    const uint32_t n_split = uniform(A.counters[ADJ_C_SPLIT]);
    const uint32_t waves = (gridDim.x * blockDim.x) >> 6;
    uint32_t n_left = 0, total = 0, done = 0, seen = 0;
    if (second) {
        n_left = uniform(overlap ? A.counters[ADJ_C_LEFT] : A.counters[ADJ_C_END] - A.counters[ADJ_C_FIRST] - n_split);
        total = n_left + min(A.counters[ADJ_C_ITEMS], A.item_cap);
    } else {
        if (__lane_id() == 0u) atomicAdd(A.counters + ADJ_C_DONE, 1u);
        const double r_in = cold_params(hp.cold).img0.r_in;
        for (uint32_t k = own; k != NO_RECORD; k = A.recs[k].next) {
            AdjLong& o = A.recs[k];
            double zb[5], gr;
            adj::ParBar q;
            adj::seed(A.dm, a, r_in, o.zb[0], o.zb[1], o.zb[2], o.E, o.L, A.cot[o.ray], zb, &q, &gr);
            o.zb[0] = zb[0];
            o.zb[1] = zb[1];
            o.zb[2] = o.zb[3] = 0.0;
            o.pb[0] = q.E;
            o.pb[1] = q.L;
            o.pb[2] = q.a;
            o.gr = gr;
        }
    }
    bool more = second;
    uint32_t rec = 0, item = 0;
    int left = -1;  // steps still to do, after the current one; -1: idle
    const double* e = nullptr;  // the current step's entry
    double y0 = 0.0, y1 = 0.0, y3 = 0.0, y4 = 0.0, h = 0.0, E = 0.0, L = 0.0;
    double b0 = 0.0, b1 = 0.0, b3 = 0.0, b4 = 0.0;
    adj::ParBar pb{0.0, 0.0, 0.0};
    const auto begin = [&](int first, int last) {
        const AdjLong& o = A.recs[rec];
        E = o.E;
        L = o.L;
        left = last - first;
        e = A.store + (static_cast<size_t>(o.base) + static_cast<size_t>(last)) * ADJ_ENTRY;
        y0 = e[0];
        y1 = e[1];
        y3 = e[2];
        y4 = e[3];
        h = e[4];
    };
    const auto begin_ray = [&]() {
        const AdjLong& o = A.recs[rec];
        b0 = o.zb[0];
        b1 = o.zb[1];
        b3 = o.zb[2];
        b4 = o.zb[3];
        pb = adj::ParBar{o.pb[0], o.pb[1], o.pb[2]};
        begin(0, o.n);
    };
    const auto put_ray = [&]() {
        AdjLong& o = A.recs[rec];
        o.zb[0] = b0;
        o.zb[1] = b1;
        o.zb[2] = b3;
        o.zb[3] = b4;
        o.pb[0] = pb.E;
        o.pb[1] = pb.L;
        o.pb[2] = pb.a;
    };
    for (;;) {
        unsigned long long idle = __ballot(left < 0);
        while (idle != 0ull && more) {
            const uint32_t want = static_cast<uint32_t>(__popcll(idle));
            const int leader = __ffsll(idle) - 1;
            uint32_t base = 0;
            if (static_cast<int>(__lane_id()) == leader) base = atomicAdd(A.counters + ADJ_C_SWEEP, want);
            base = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(base), leader));
            more = base < total;
            item = left < 0 ? base + lanes_below(idle) : item;
            if (left < 0 && item < n_left) {
                rec = overlap ? A.recs[item].left : n_split + item;
                if (A.recs[rec].status == ADJ_OK) begin_ray();
            } else if (left < 0 && item < total) {
                rec = A.owner[item - n_left];
                const AdjLong& o = A.recs[rec];
                if (o.status == ADJ_OK) {
                    const uint32_t local = item - n_left - o.item_base, b = local & 3u;
                    const int first = static_cast<int>(local >> 2) * ADJ_SEG;
                    b0 = b == 0u ? 1.0 : 0.0;
                    b1 = b == 1u ? 1.0 : 0.0;
                    b3 = b == 2u ? 1.0 : 0.0;
                    b4 = b == 3u ? 1.0 : 0.0;
                    pb = adj::ParBar{0.0, 0.0, 0.0};
                    begin(first, min(o.n, first + ADJ_SEG - 1));
                }
            }
            idle = __ballot(left < 0);
        }
        if (!second && done != waves) {
            // the count as it was one iteration ago, so that its load is not waited for
            done = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(seen)));
            seen = __hip_atomic_load(A.counters + ADJ_C_DONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (left < 0 && own != NO_RECORD) {
                rec = own;
                own = A.recs[rec].next;
                begin_ray();
            }
        } else if (!second) {
            // no wave has a forward ray left
            if (left >= 0) {
                put_ray();
                A.recs[rec].n = left;
                A.recs[atomicAdd(A.counters + ADJ_C_LEFT, 1u)].left = rec;
            }
            for (; own != NO_RECORD; own = A.recs[own].next)
                A.recs[atomicAdd(A.counters + ADJ_C_LEFT, 1u)].left = own;
            break;
        }
        if (__ballot(left >= 0) == 0ull) break;
        if (left < 0) continue;
        const double y[5] = {y0, y1, 0.0, y3, y4}, hs = h;
        double yb[5] = {b0, b1, 0.0, b3, b4};
        if (left > 0) {
            e -= ADJ_ENTRY;
            y0 = e[0];
            y1 = e[1];
            y3 = e[2];
            y4 = e[3];
            h = e[4];
        }
        adj::dp_step_vjp<false>(M, a, E, L, y, hs, yb, &pb);
        b0 = yb[0];
        b1 = yb[1];
        b3 = yb[3];
        b4 = yb[4];
        if (--left < 0) {
            if (!second || item < n_left) {
                put_ray();
            } else {
                double* o = A.items + static_cast<size_t>(item - n_left) * 8u;
                o[0] = b0;
                o[1] = b1;
                o[2] = b3;
                o[3] = b4;
                o[4] = pb.E;
                o[5] = pb.L;
                o[6] = pb.a;
            }
        }
    }
}

// FEAT >= 0 fixes the image's features (FEAT_* bits) at compile time, so the
// event tests of absent features vanish from the step loop; FEAT_DYN reads
// them from the launch (single images) or the lane's image (batches).
constexpr int FEAT_DYN = -1;

// The step loop has one straight path that every busy lane of the wave takes
// together: the step, its error and step-size factor, and one predicate that
// names the lanes for which anything else than an ordinary accepted or
// rejected step may have happened (a window of r, the disk plane, the source
// arc's range, a non-finite error, event location under way, the step
// budget).  Ordinary lanes commit or shrink their step there; the others go
// through the long form of the same decisions after it, and only then does
// the wave look for ended rays to replace.  What the predicate may not miss
// is listed at each test; a lane it names without need takes the long form
// and ends up with the same bits.
//
// The kernel is bound by the FP64 vector issue rate (the step alone is ~570
// FP64 instructions), so everything that is not that arithmetic counts:
// with each test in a branch of its own, and the per-ray scalars in LDS, an
// attempt took ~830 vector and ~215 scalar instructions, and a wave alone on
// its SIMD, as in small images, needed 2.5 us for it.  It takes 615 and ~40 now
// (a Kerr disk, 2-wave build; 583 of them FP64; 580 without spin) and 1.45 us:
// 512x512 lensing 4.9 -> 3.1 ms, 1024x1024 ring 18.1 -> 15.3.
//
// STORE: the adjoint's forward pass.  The rays come from its work list, every
// accepted step and the located partial step go to the ray's range of the
// step store, and its end to its record instead of the outputs; then the wave
// sweeps (see sweep).
template <int METHOD, int PREC, bool BATCH, int METRIC = METRIC_KERR, int FEAT = FEAT_DYN, bool STORE = false>
__global__ void __launch_bounds__(BLOCK_MAX) __attribute__((amdgpu_waves_per_eu(KT_WAVES_PER_EU)))
trace_kernel(const Hot hp) {
    constexpr bool QMET = METRIC == METRIC_Q;
    static_assert(!(QMET && (BATCH || METHOD == KT_RK4_S || PREC != KT_FP64)),
                  "the q-metric runs single images with the adaptive FP64 schemes");
    static_assert(FEAT == FEAT_DYN || !BATCH, "batches read each image's features");
    constexpr int EVALS_PER_STEP = evals_per_step<METHOD>();
    constexpr bool ADAPTIVE = (METHOD != KT_RK4_S);
    constexpr bool S_TIME = (METHOD == KT_RK4_S);
    constexpr bool MIXED = (PREC == KT_MIXED) && (METHOD == KT_DP45) && !QMET;
    constexpr bool LONG_STEPS = METHOD == KT_BS || METHOD == KT_BS_RAT;
    constexpr bool PIN_SHIFT = !LONG_STEPS && METHOD != KT_RK4_S;
    constexpr bool PIN_THETA = METHOD == KT_BS && !QMET && !BATCH && KT_WAVES_PER_EU < 3;
    constexpr int PIN_COEFS =
        KT_WAVES_PER_EU < 3 && METHOD == KT_DP45 && !QMET && !MIXED && FEAT >= 0 ? ((FEAT & FEAT_SRC) ? 8 : 20) : 0;
    constexpr bool MAY_DISK = FEAT < 0 ? !QMET : (FEAT & FEAT_DISK) != 0;
    constexpr bool MAY_SRC = FEAT < 0 || (FEAT & FEAT_SRC) != 0;
    __shared__ double cold[N_COLD][BLOCK_MAX];
    const int tid = threadIdx.x;
#define COLD(f) cold[f][tid]

    LaneImg li;
    li.st = Spacetime{hp.M, hp.a, hp.a2, hp.two_a2};
    li.feat = hp.feat;
    li.k = 0;
    const uint32_t lane = __lane_id();
    uint32_t n_total;
    // STORE: the first stored ray in the list, and the first that its lane sweeps
    uint32_t adj_first = 0, own_from = NO_RECORD;

    // this wave's queue of ray ids [q_next, q_end).  A persistent wave's
    // first fetch takes 64 ids, one per lane, in one atomic; later fetches
    // take P.batch, or one per idle lane if those are more.  Taken in
    // batch-sized pieces, the start of the launch was a burst of 64 / batch
    // serial round trips per wave on one address, and the wave's first rays
    // came from interleaved places in the dispatch order instead of one run
    // of similar cost.
    uint32_t q_next, q_end;
    bool exhausted;
    bool first_fetch;
    {
        const Params& P = cold_params(hp.cold);
        if constexpr (STORE) {
            const uint32_t* c = P.adj.counters;
            adj_first = uniform(c[ADJ_C_FIRST]);
            own_from = uniform(c[ADJ_C_OVERLAP] != 0u ? c[ADJ_C_SPLIT] : NO_RECORD);
            n_total = hp.sweep_only ? 0u : uniform(c[ADJ_C_END]) - adj_first;
        } else {
            n_total = P.from_list ? *P.fb_count : static_cast<uint32_t>(P.n_rays);
        }
        first_fetch = P.persistent != 0;
    }
    if (first_fetch) {
        q_next = q_end = 0;
        exhausted = false;
    } else {
        const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
        q_next = min(wave * 64u, n_total);
        q_end = min(q_next + 64u, n_total);
        exhausted = true;
    }

    // The constants kept in registers: as many of the Dormand-Prince tableau's 26
    // as there are registers left in the 2-wave build (a wave alone on its SIMD
    // waits for each scalar move that sets one up, ~40 in 626 instructions of an
    // attempt: 96x96 ring 2.71 -> 2.64 ms, 512x512 lensing 3.24 -> 3.06; with three
    // waves per SIMD others fill in); those of the shift from the base point,
    // which every Runge-Kutta stage needs; of sin/cos of theta itself, which each
    // Bulirsch-Stoer substep needs, only for single Kerr images by polynomials in
    // the 2-wave build.  There the loop keeps them although the kernel then has
    // 116 bytes of scratch per lane (20 without them), none of it touched inside
    // the step loop: norm check of 625x625 rays 3.30 ms, 3.42 without, with half
    // of them 3.36; 512x512 ring 3.38 and 3.49, 768x768 7.12 and 7.34.  By rational
    // functions the times are equal (512x512 4.62 and 4.60) and scratch is 28 bytes
    // instead of 124; a batch of 3.6M rays takes 26.4 ms without them, 26.9 with,
    // by rational functions 35.9 and 36.5; with 3 waves 1200x1000 rays 15.1 and 15.9.
    const Elem<PIN_SHIFT, PIN_THETA, PIN_COEFS> el;
    int32_t ray = -1;
    int fl = 0;
    Vec5 ys{}, ks{};  // the state and the field there
    RayConst rc{};
    double h = 0.0;             // the step to try (while locating: the trial step)
    double s0 = 0.0, c0 = 1.0;  // sin, cos of theta at y
    // The swept angle up to y, the largest |2H|, and the |2 Sigma H| and D of
    // the largest |H|_rel.  With 3 waves per SIMD there are no registers left
    // for them, but the other waves hide the LDS reads; a wave alone on its
    // SIMD, the common case of the 2-wave build, would wait for them.
    constexpr bool IN_LDS = KT_WAVES_PER_EU == 3 || MIXED || BATCH;
    double reg_swept, reg_max_h2, reg_rel_k, reg_rel_d;
    double& swept = IN_LDS ? COLD(C_SWEPT) : reg_swept;
    double& max_h2 = IN_LDS ? COLD(C_MAXH2) : reg_max_h2;
    double& rel_k = IN_LDS ? COLD(C_RELK) : reg_rel_k;
    double& rel_d = IN_LDS ? COLD(C_RELD) : reg_rel_d;
    swept = max_h2 = rel_k = 0.0;
    rel_d = 1.0;
    double r_lo = 0.0, r_hi = 0.0;  // MAY_SRC: the window of r without an event
    float fac_max = 5.0f;           // growth limit: 1 after a rejection
    int misses = 0;                 // attempts that were not accepted steps
    uint32_t rec = 0, entry = 0, entry_end = 0;  // STORE: the ray's record, its next entry and their end
    uint32_t own = NO_RECORD, own_last = 0;      // the first and last of the lane's rays that it will sweep itself
    unsigned long long evals_acc = 0, evals32_acc = 0;
    // Attempts are counted for the wave: a lane's are it - it0, its accepted
    // steps those less its misses.  From it_limit on, some lane may have
    // used up its step budget.
    uint32_t it = 0, it0 = 0;
    const uint32_t budget = static_cast<uint32_t>(
        min(hp.max_steps, (hp.max_evals - 1 + EVALS_PER_STEP - 1) / EVALS_PER_STEP));
    uint32_t it_limit = budget;
    // lanes with a ray, and those whose next attempt is part of an event
    // (F_LOCATE or F_RETAKE)
    unsigned long long busy, in_event = 0ull;

    // the q-metric carries (q, q(2+q)) in the spacetime's (a, a^2) slots
    const auto spacetime = [&]() {
        if constexpr (QMET)
            return QSpacetime{li.st.M, li.st.a, li.st.a2};
        else if constexpr (METRIC == METRIC_SCHWARZSCHILD)
            return Schwarzschild{li.st.M};
        else
            return li.st;
    };
    // The window of r inside which no radial event can happen: capture below
    // it, escape above it, and with a source still ahead its sphere, from
    // the side the ray is on.
    const auto set_window = [&](const Radii& rd, double r) {
        if constexpr (MAY_SRC) {
            r_lo = rd.r_cap;
            r_hi = rd.r_esc;
            const int32_t feat = FEAT >= 0 ? FEAT : li.feat;
            if ((feat & FEAT_SRC) && !(fl & F_SRCDONE)) {
                if (r < rd.r_src)
                    r_hi = fmin(r_hi, rd.r_src);
                else
                    r_lo = fmax(r_lo, rd.r_src);
            }
        }
    };
    // STORE: a step of size h from ys goes to the ray's next entry
    const auto put_entry = [&]() {
        double* e = hp.store + static_cast<size_t>(entry) * ADJ_ENTRY;
        e[0] = ys.r;
        e[1] = ys.th;
        e[2] = ys.pr;
        e[3] = ys.pth;
        e[4] = h;
    };
    const auto write_record = [&](int fate, double r_c, double dr_c, double dth_c) {
        const Params& P = cold_params(hp.cold);
        AdjLong& o = P.adj.recs[rec];
        int status = ADJ_OVERFLOW;  // no room, no step, or out of the trace's budget
        if (fate == KT_FATE_DISK) {
            status = P.adj.r_hit && !(r_c == P.adj.r_hit[ray]) ? ADJ_MISMATCH : ADJ_OK;
            put_entry();
            o.n = static_cast<int32_t>(entry - o.base);
            o.zb[0] = r_c;
            o.zb[1] = dr_c;
            o.zb[2] = dth_c;
            o.E = rc.E;
            o.L = rc.L;
        } else if (fate == KT_FATE_CAPTURED || fate == KT_FATE_ESCAPED) {
            status = ADJ_MISMATCH;
        }
        o.status = status;
        if (status == ADJ_OK && rec >= own_from) {
            o.next = NO_RECORD;
            if (own == NO_RECORD)
                own = rec;
            else
                P.adj.recs[own_last].next = rec;
            own_last = rec;
        }
        ray = -1;
    };
    const auto write_outputs = [&](int fate, double r_c, double psi, double defl, double thf, double phf, int nsteps,
                                   int nevals) {
        const Params& P = cold_params(hp.cold);
        const Outputs& o = P.out;
        o.fate[ray] = static_cast<uint8_t>(fate);
        P.rc_buf[ray] = r_c;
        if (o.max_abs_h) o.max_abs_h[ray] = 0.5 * max_h2;
        const double max_rel = rel_k * rcp(QMET ? rel_d : fabs(rel_d));
        if (o.max_rel_h) o.max_rel_h[ray] = max_rel;
        if (o.psi) o.psi[ray] = psi;
        if (o.deflection) o.deflection[ray] = defl;
        if (o.theta_f) o.theta_f[ray] = thf;
        if (o.phi_f) o.phi_f[ray] = phf;
        if (o.n_cross) o.n_cross[ray] = static_cast<uint8_t>((fl >> NCROSS_SHIFT) & 0xff);
        if (o.used_fp64) o.used_fp64[ray] = static_cast<uint8_t>(P.from_list ? 1 : 0);
        if (o.n_steps) o.n_steps[ray] = nsteps;
        if (o.n_evals) o.n_evals[ray] = nevals;
        if constexpr (MIXED) P.need_fb[ray] = ((fl & F_USED32) && !(max_rel <= hp.h_budget)) ? 1 : 0;
        evals_acc += static_cast<unsigned long long>(nevals);
        ray = -1;
    };

    for (;;) {
        // ---- refill idle lanes from the wave queue -------------------------
        // A refill is a chain of memory round trips (ticket, dispatch order),
        // a few microseconds in which the wave's other rays stand still, so
        // it waits until hp.min_idle lanes are idle.  That costs a part of
        // min_idle / 128 of the lanes: 8 for a wave that has its SIMD to
        // itself (512x512 ring 5.98 -> 5.46 ms, disk 3.98 -> 3.62 against a
        // refill per idle lane; 16: 5.52 and 3.75), 4 where other waves fill
        // in (1024x1024 ring 16.35 -> 15.84; 8: 16.09).
        unsigned long long idle = __ballot(ray < 0);
        if (__popcll(idle) < hp.min_idle) idle = 0ull;
        while (idle != 0ull) {
            if (q_next >= q_end) {
                if (exhausted) break;
                const Params& P = cold_params(hp.cold);
                const int leader = __ffsll(idle) - 1;
                uint32_t base = 0;
                const uint32_t take =
                    first_fetch ? hp.first : max(static_cast<uint32_t>(P.batch), static_cast<uint32_t>(__popcll(idle)));
                first_fetch = false;
                if (static_cast<int>(lane) == leader) base = atomicAdd(P.ticket, take);
                base = static_cast<uint32_t>(__shfl(static_cast<int>(base), leader));
                if (base >= n_total) {
                    exhausted = true;
                    break;
                }
                q_next = base;
                q_end = min(base + take, n_total);
            }
            const uint32_t rank = lanes_below(idle);
            const uint32_t avail = q_end - q_next;
            if (ray < 0 && rank < avail) {
                const Params& P = cold_params(hp.cold);
                const uint32_t slot = q_next + rank;
                if constexpr (STORE) {
                    rec = slot;
                    ray = static_cast<int32_t>(P.adj.list[adj_first + slot]);
                } else {
                    ray = static_cast<int32_t>(P.from_list ? P.fb_list[slot] : P.perm ? P.perm[slot] : slot);
                }
                double y[5], E, L;
                bool valid;
                if constexpr (BATCH) {
                    const int k = find_image(P, ray);
                    const Image& im = P.images[k];
                    li = lane_img(im, k);
                    valid = camera_state(im, ray - static_cast<int32_t>(im.first), y, &E, &L);
                } else {
                    valid = camera_state(P.img0, ray, y, &E, &L);
                }
                fl = 0;
                if constexpr (STORE) {
                    // room for the forward render's steps and the partial one
                    const uint32_t room = static_cast<uint32_t>(max(P.adj.n_steps[ray], 0)) + 2u;
                    entry = atomicAdd(P.adj.counters + ADJ_C_STORE, room);
                    entry_end = entry + room;
                    AdjLong& o = P.adj.recs[rec];
                    o.ray = ray;
                    o.base = entry;
                    const bool fits_store = entry_end >= entry && entry_end <= P.adj.entries;
                    if (!valid || !fits_store) {
                        write_record(FATE_NO_ROOM, 0.0, 0.0, 0.0);
                        valid = false;
                    }
                }
                if (!valid) {
                    if constexpr (!STORE) {
                        const double NaN = __builtin_nan("");
                        max_h2 = rel_k = NaN;
                        write_outputs(KT_FATE_INVALID, NaN, NaN, NaN, y[1], y[2], 0, 0);
                    }
                } else {
                    // k1 = f(y0) (FSAL seed) and H at lambda = 0
                    const auto st = spacetime();
                    rc = make_ray_const(st, E, L);
                    Diag dg;
                    double k1[5];
                    rhs<true, S_TIME>(st, rc, y, k1, &dg);
                    ys = Vec5::of(y);
                    ks = Vec5::of(k1);
                    max_h2 = fabs(dg.H2);
                    rel_k = QMET ? dg.Kabs : __builtin_copysign(dg.Kabs, dg.D);
                    rel_d = dg.D;
                    s0 = dg.s;
                    c0 = dg.c;
                    COLD(C_LAM) = 0.0;
                    swept = 0.0;
                    h = ADAPTIVE ? P.h_init : P.h_fixed;
                    fac_max = 5.0f;
                    misses = 0;
                    it0 = it;
                    set_window(event_radii<BATCH>(hp.cold, li.k), y[0]);
                }
            }
            q_next += min(static_cast<uint32_t>(__popcll(idle)), avail);
            idle = __ballot(ray < 0);
        }
        busy = __ballot(ray >= 0);
        if (busy == 0ull) break;

        // ---- the step loop: until some lane needs the long form ------------
        // Idle lanes go along on their last state and change nothing.
        Diag dg;
        Vec5 ye{}, ke{};  // the step's end and the field there
        double msq = 0.0, fac = 1.0;
        bool use32 = false, fits = true, odd;
        for (;;) {
#if KT_WAVES_PER_EU == 3
            // With three waves per SIMD the issue arbiter's preference for
            // the oldest wave runs the three generations of blocks at very
            // different speeds, and the rays a slow wave holds end the
            // launch late.  Each wave steps its priority down from 3 to 0
            // and round again, one level per attempt; the waves' cycles
            // are out of phase, so the highest priority moves from wave to
            // wave and their shares of the issue slots even out.
            switch (it & 3u) {
                case 0: __builtin_amdgcn_s_setprio(3); break;
                case 1: __builtin_amdgcn_s_setprio(2); break;
                case 2: __builtin_amdgcn_s_setprio(1); break;
                default: __builtin_amdgcn_s_setprio(0); break;
            }
#endif
            ++it;
            const auto st = spacetime();
            double y[5], k1[5], yn[5], kn[5], er[5];
            ys.to(y);
            ks.to(k1);
            if constexpr (MIXED) {
                // The FP32 mass part runs wave-uniformly.  A lane locating
                // an event, or retaking the step it lay in, must use the
                // precision of that accepted step (its trial steps are
                // steps of the same stepper, and the retake must reproduce
                // the step bit for bit).  The lowest such lane sets the
                // wave's precision and lanes that cannot use it sit this
                // attempt out; with no such lane the FP32 part runs when
                // every stepping lane is beyond r_switch.
                const bool pinned = (fl & (F_LOCATE | F_RETAKE)) != 0;
                const bool ev32 = (fl & F_EV32) != 0;
                if (in_event != 0ull) {
                    const int lead = __ffsll(in_event) - 1;
                    use32 = ((__ballot(ev32) >> lead) & 1ull) != 0ull;
                } else {
                    use32 = (__ballot(y[0] >= hp.r_switch) & busy) == busy;
                }
                fits = pinned ? (ev32 == use32) : (!use32 || y[0] >= hp.r_switch);
                const Spacetime32 sf{static_cast<float>(st.M), static_cast<float>(st.a), static_cast<float>(st.a2)};
                if (use32) {
                    dp45_step<true>(st, rc, y, k1, s0, c0, h, yn, kn, er, &dg, &sf);
                    if (fits && ray >= 0) {
                        fl |= F_USED32;
                        evals32_acc += EVALS_PER_STEP;
                    }
                } else {
                    dp45_step<false>(st, rc, y, k1, s0, c0, h, yn, kn, er, &dg);
                }
                if (!fits) ++it0;
            } else {
                take_step<METHOD>(st, rc, y, k1, s0, c0, h, yn, kn, er, &dg, el);
            }
            ye = Vec5::of(yn);
            ke = Vec5::of(kn);
            bool accept = true;
            odd = false;
            if constexpr (ADAPTIVE) {
                // mean square of err_i / (atol + rtol max(|y_i|, |yn_i|))
                double sc[5];
#pragma unroll
                for (int i = 0; i < 5; ++i) sc[i] = fma(hp.rtol, max_abs(y[i], yn[i]), hp.atol);
                msq = error_msq<fp64_control<METHOD>()>(er, sc);
                fac = step_scale<METHOD>(msq, fac_max);
                accept = msq <= 1.0;
                // A non-finite r, theta, p_r or p_theta makes kn and with
                // it the error NaN or infinite, an infinite scale makes
                // the norm NaN; phi enters no evaluation and is tested.
                odd = !(msq < 1e20) | !isfinite(yn[2]);
                if constexpr (STORE) odd = odd | (entry + 1u >= entry_end);
            } else {
#pragma unroll
                for (int i = 0; i < 5; ++i) odd = odd | !isfinite(yn[i]);
            }
            // events that an accepted step may hold (each test is at least
            // as wide as the event's own condition in the long form)
            const int32_t feat = FEAT >= 0 ? FEAT : li.feat;
            bool ev = MAY_SRC ? !(yn[0] >= r_lo) | !(yn[0] < r_hi) : !(yn[0] >= hp.r_cap) | !(yn[0] <= hp.r_esc);
            if constexpr (MAY_DISK) {
                const bool cross = (y[1] - HALF_PI) * (yn[1] - HALF_PI) <= 0.0;
                ev = ev | (cross & ((feat & FEAT_DISK) != 0));
            }
            double arc = 0.0;
            if constexpr (MAY_SRC) {
                if (FEAT >= 0 || (feat & FEAT_SRC)) {
                    bool in_range;
                    arc = arc_angle_short(s0, c0, dg.s, dg.c, yn[2] - y[2], &in_range);
                    ev = ev | !in_range;
                }
            }
            odd = odd | (accept & ev) | __builtin_amdgcn_inverse_ballot_w64(in_event) | (it == it_limit);
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(busy) & fits;
            odd = odd & mine;
            if (!odd & mine) {
                if (accept) {
                    // commit
                    if constexpr (STORE) {
                        put_entry();
                        ++entry;
                    } else {
                        keep_max<!QMET>(dg, &max_h2, &rel_k, &rel_d);
                    }
                    unsafeAtomicAdd(&COLD(C_LAM), h);  // one LDS add, no result
                    if constexpr (MAY_SRC) swept += arc;
                    ys = ye;
                    ks = ke;
                    s0 = dg.s;
                    c0 = dg.c;
                    if constexpr (ADAPTIVE) {
                        h *= fac;
                        fac_max = 5.0f;
                    }
                } else {
                    // reject, unless the step underflows
                    const double hn = h * fac;
                    odd = hn < 1e-12 * fmax(1.0, fabs(COLD(C_LAM)));
                    if (!odd) {
                        h = hn;
                        fac_max = 1.0f;
                        ++misses;
                    }
                }
            }
            if (__ballot(odd) != 0ull) break;
        }

        // ---- the long form, for the lanes that need it -----------------
        if (odd) {
            const int32_t feat = FEAT >= 0 ? FEAT : li.feat;
            const Radii rd = event_radii<BATCH>(hp.cold, li.k);
            const double NaN = __builtin_nan("");
            int fate = -1;  // >= 0 once the ray ends
            double thf = ys.th, phf = ys.ph, r_c = NaN, psi = NaN, defl = NaN;
            if (fl & F_LOCATE) {
                // Illinois regula falsi on the event function
                ++misses;
                const bool src = (fl & F_EVSRC) != 0;
                const bool esc = (fl & F_EVESC) != 0;
                const Params& P = cold_params(hp.cold);
                const Image& im = BATCH ? P.images[li.k] : P.img0;
                const double fc = esc ? ye.r - rd.r_esc : src ? ye.r - rd.r_src : ye.th - HALF_PI;
                const double tol = esc ? im.esc_tol : src ? im.src_tol : 1e-14;
                const int n_it = ((fl >> EVIT_SHIFT) & 0xff) + 1;
                fl = (fl & ~(0xff << EVIT_SHIFT)) | (n_it << EVIT_SHIFT);
                if ((fabs(fc) <= tol || n_it >= 64) && esc) {
                    // the ray meets the celestial sphere here
                    fate = KT_FATE_ESCAPED;
                    thf = ye.th;
                    phf = ye.ph;
                } else if (fabs(fc) <= tol || n_it >= 64) {
                    if (!src) {
                        if (ye.r >= rd.r_in && ye.r <= rd.r_out) {
                            fate = KT_FATE_DISK;
                            r_c = ye.r;
                            thf = ye.th;
                            phf = ye.ph;
                        } else {
                            const int nc = min(((fl >> NCROSS_SHIFT) & 0xff) + 1, 255);
                            fl = (fl & ~(0xff << NCROSS_SHIFT)) | (nc << NCROSS_SHIFT) | F_SKIPDISK;
                        }
                    } else {
                        const double sw = swept + arc_angle(s0, c0, dg.s, dg.c, ye.ph - ys.ph);
                        double sp, cp;
                        sincos_fast(ye.ph, &sp, &cp);
                        const double* sn = im.src_n;
                        const double nx = dg.s * cp, ny = dg.s * sp, nz = dg.c;
                        const double cx = ny * sn[2] - nz * sn[1];
                        const double cy = nz * sn[0] - nx * sn[2];
                        const double cz = nx * sn[1] - ny * sn[0];
                        COLD(C_SRCPSI) = atan2_upper(sqrt(fma(cx, cx, fma(cy, cy, cz * cz))),
                                                     fma(nx, sn[0], fma(ny, sn[1], nz * sn[2])));
                        COLD(C_DEFL) = sw;  // parked until the ray ends
                        fl |= F_SRCDONE;
                    }
                    if (fate < 0) {
                        // continue from the end of the accepted step: retake it (bit-identical)
                        fl = (fl & ~F_LOCATE) | F_RETAKE;
                        h = COLD(C_H);
                    }
                } else {
                    double a = COLD(C_EVA), fa = COLD(C_EVFA), b = COLD(C_EVB), fb = COLD(C_EVFB);
                    if (fc * fb < 0.0) {
                        a = b;
                        fa = fb;
                    } else {
                        fa *= 0.5;
                    }
                    b = h;
                    fb = fc;
                    COLD(C_EVA) = a;
                    COLD(C_EVFA) = fa;
                    COLD(C_EVB) = b;
                    COLD(C_EVFB) = fb;
                    h = b - fb * (b - a) / (fb - fa);
                }
            } else {
                const bool finite = isfinite(ye.r) && isfinite(ye.th) && isfinite(ye.ph) && isfinite(ye.pr) &&
                                    isfinite(ye.pth);
                if (!finite || (ADAPTIVE && isnan(msq))) {
                    fate = KT_FATE_STEPFAIL;
                    ++misses;
                } else if (ADAPTIVE && msq > 1.0) {
                    h *= fac;
                    fac_max = 1.0f;
                    ++misses;
                    if (h < 1e-12 * fmax(1.0, fabs(COLD(C_LAM)))) fate = KT_FATE_STEPFAIL;
                } else {
                    if (!(fl & F_RETAKE)) {
                        keep_max<!QMET>(dg, &max_h2, &rel_k, &rel_d);
                    } else {
                        ++misses;
                    }
                    fl &= ~F_RETAKE;
                    // an event inside the step: its function at both ends
                    int locate = 0;  // its F_EV* kind, or F_LOCATE for the disk
                    double fa = 0.0, fb = 0.0;
                    // thin disk: sign change of theta - pi/2 over the step
                    if ((feat & FEAT_DISK) && !(fl & F_SKIPDISK)) {
                        const double ga = ys.th - HALF_PI, gb = ye.th - HALF_PI;
                        if (ga * gb < 0.0) {
                            locate = F_LOCATE;
                            fa = ga;
                            fb = gb;
                        } else if (gb == 0.0) {
                            if (ye.r >= rd.r_in && ye.r <= rd.r_out) {
                                fate = KT_FATE_DISK;
                                r_c = ye.r;
                                thf = ye.th;
                                phf = ye.ph;
                            } else {
                                const int nc = min(((fl >> NCROSS_SHIFT) & 0xff) + 1, 255);
                                fl = (fl & ~(0xff << NCROSS_SHIFT)) | (nc << NCROSS_SHIFT);
                            }
                        }
                    }
                    if (!locate && fate < 0) {
                        if (ye.r < rd.r_cap) {
                            fate = KT_FATE_CAPTURED;
                            thf = ye.th;
                            phf = ye.ph;
                        } else {
                            if ((feat & FEAT_SRC) && !(fl & F_SRCDONE)) {
                                if (ys.r < rd.r_src && ye.r >= rd.r_src) {
                                    locate = F_LOCATE | F_EVSRC;
                                    fa = ys.r - rd.r_src;
                                    fb = ye.r - rd.r_src;
                                } else {
                                    const double dphi = ye.ph - ys.ph;
                                    bool in_range;
                                    double arc = arc_angle_short(s0, c0, dg.s, dg.c, dphi, &in_range);
                                    if (!in_range) arc = arc_angle(s0, c0, dg.s, dg.c, dphi);
                                    swept += arc;
                                }
                            }
                            if (!locate) {
                                if (ye.r > rd.r_esc && (feat & FEAT_SKY)) {
                                    // locate the crossing of the celestial sphere
                                    locate = F_LOCATE | F_EVESC;
                                    fa = ys.r - rd.r_esc;
                                    fb = ye.r - rd.r_esc;
                                } else if (ye.r > rd.r_esc) {
                                    fate = KT_FATE_ESCAPED;
                                    thf = ye.th;
                                    phf = ye.ph;
                                } else {
                                    // commit the step
                                    if constexpr (STORE) {
                                        if (entry + 1u < entry_end) {
                                            put_entry();
                                            ++entry;
                                        } else {
                                            fate = FATE_NO_ROOM;
                                        }
                                    }
                                    ys = ye;
                                    ks = ke;
                                    unsafeAtomicAdd(&COLD(C_LAM), h);  // one LDS add, no result
                                    if constexpr (ADAPTIVE) h *= fac;
                                    fac_max = 5.0f;
                                    fl &= ~F_SKIPDISK;
                                    s0 = dg.s;
                                    c0 = dg.c;
                                }
                            }
                        }
                    }
                    if (locate) {
                        fl = (fl & ~(F_EVSRC | F_EVESC | F_EV32 | (0xff << EVIT_SHIFT))) | locate |
                             (use32 ? F_EV32 : 0);
                        COLD(C_H) = h;
                        COLD(C_EVA) = 0.0;
                        COLD(C_EVFA) = fa;
                        COLD(C_EVB) = h;
                        COLD(C_EVFB) = fb;
                        h = h - fb * h / (fb - fa);
                    }
                }
            }
            const int attempts = static_cast<int>(it - it0);
            const int nevals = 1 + attempts * EVALS_PER_STEP, nsteps = attempts - misses;
            if (fate < 0 && !(fl & (F_LOCATE | F_RETAKE)) && (nsteps >= hp.max_steps || nevals >= hp.max_evals)) {
                fate = KT_FATE_MAXSTEPS;
                thf = ys.th;
                phf = ys.ph;
            }
            if (fate >= 0) {
                if (fl & F_SRCDONE) {
                    defl = COLD(C_DEFL);
                    psi = COLD(C_SRCPSI);
                }
                fl &= ~(F_LOCATE | F_RETAKE);
                if constexpr (STORE)
                    write_record(fate, r_c, ke.r, ke.th);
                else
                    write_outputs(fate, r_c, psi, defl, thf, phf, nsteps, nevals);
            }
            set_window(rd, ys.r);
        }
        in_event = __ballot(ray >= 0 && (fl & (F_LOCATE | F_RETAKE)) != 0);
        if (it == it_limit) {
            // the next attempt at which a lane's budget may end
            const int attempts = static_cast<int>(it - it0);
            const int evals_left = hp.max_evals - (1 + attempts * EVALS_PER_STEP);
            int left = max(1, min(hp.max_steps - (attempts - misses),
                                  (evals_left + EVALS_PER_STEP - 1) / EVALS_PER_STEP));
            int least = static_cast<int>(budget);
            for (unsigned long long m = __ballot(ray >= 0); m != 0ull; m &= m - 1ull)
                least = min(least, __builtin_amdgcn_readlane(left, __ffsll(m) - 1));
            it_limit = it + static_cast<uint32_t>(least);
        }
    }
#undef COLD

    if constexpr (STORE) {
        sweep(hp, own);
        return;
    }
    // one atomic per wave for each evaluation counter
    const unsigned long long evals = wave_sum(evals_acc);
    if (lane == 0 && evals != 0ull) atomicAdd(hp.acc + ACC_EVALS, evals);
    if constexpr (MIXED) {
        const unsigned long long evals32 = wave_sum(evals32_acc);
        if (lane == 0 && evals32 != 0ull) atomicAdd(hp.acc + ACC_EVALS_FP32, evals32);
    }
}

#if !KT_TRACE_ONLY
// Compact the re-run flags into the fallback list (order does not matter:
// every ray is independent) and count them.
__global__ void fallback_list_kernel(const uint8_t* __restrict__ need, int64_t n, uint32_t* __restrict__ list,
                                     uint32_t* count) {
    __shared__ uint32_t block_base;
    __shared__ uint32_t wave_counts[BLOCK_MAX / 64];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t lane = __lane_id();
    for (int64_t base = static_cast<int64_t>(blockIdx.x) * blockDim.x; base < n;
         base += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t k = base + tid;
        const bool want = k < n && need[k];
        const unsigned long long m = __ballot(want);
        const uint32_t rank = static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
        if (lane == 0) wave_counts[wave] = static_cast<uint32_t>(__popcll(m));
        __syncthreads();
        if (tid == 0) {
            uint32_t tot = 0;
            for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) {
                const uint32_t c = wave_counts[w];
                wave_counts[w] = tot;
                tot += c;
            }
            block_base = tot ? atomicAdd(count, tot) : 0u;
        }
        __syncthreads();
        if (want) list[block_base + wave_counts[wave] + rank] = static_cast<uint32_t>(k);
        __syncthreads();
    }
}

// Switch the workspace copy of the parameters to the list-driven FP64 pass.
__global__ void to_fallback_kernel(Params* wp) {
    if (threadIdx.x == 0) {
        *wp->ticket = 0u;
        wp->from_list = 1;
        wp->precision = KT_FP64;
    }
}

// Redshift and observed intensity of every disk pixel from the crossing
// radius the trace kernel parked in rc_buf (eq:redshift read as
// g = 1 / (u^t (E - Omega L)); I_obs = g^3 I_em with I_em = (M/r)^q).
// Omega is Keplerian or from the constant specific angular momentum l0.
__global__ void disk_obs_kernel(const Params* pp) {
    const Params& p = *pp;
    const int64_t n = p.n_rays;
    const double NaN = __builtin_nan("");
    for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < n;
         k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        double r_hit = NaN, g = NaN, inten = 0.0;
        if (p.out.fate[k] == KT_FATE_DISK) {
            const Image& im = p.images[find_image(p, k)];
            double z[5], E, L;
            camera_state(im, static_cast<int32_t>(k - im.first), z, &E, &L);
            const double rc = p.rc_buf[k];
            const double inv_rc = 1.0 / rc;
            const double gtt = -(1.0 - 2.0 * im.M * inv_rc);
            const double gtp = -2.0 * im.M * im.a * inv_rc;
            const double gpp = rc * rc + im.a2 + 2.0 * im.M * im.a2 * inv_rc;
            double Om;
            if (im.rotation == KT_ROT_L0) {
                Om = -(gtp + im.l0 * gtt) / (gpp + im.l0 * gtp);
            } else {
                const double sM = sqrt(im.M);
                Om = sM / fma(rc, sqrt(rc), im.a * sM);
            }
            const double norm = -gtt - 2.0 * Om * gtp - Om * Om * gpp;  // (u^t)^-2
            r_hit = rc;
            if (norm > 0.0) {
                g = sqrt(norm) / (E - Om * L);
                double em;
                if (im.emis_model == KT_EMIS_TAPERED) {
                    const double mr = im.M * inv_rc;
                    em = mr * mr * (1.0 - sqrt(im.r_in * inv_rc));
                    const double sv = (im.r_out - rc) / (2.0 * im.M);
                    if (sv < 1.0) em *= sv * sv * (3.0 - 2.0 * sv);
                } else {
                    em = pow(im.M * inv_rc, im.emis_q);
                }
                inten = g * g * g * em;
            }
        }
        if (p.out.r_hit) p.out.r_hit[k] = r_hit;
        if (p.out.g) p.out.g[k] = g;
        if (p.out.intensity) p.out.intensity[k] = inten;
    }
}

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------

__global__ void ws_init_kernel(const Params p) {
    const int t = threadIdx.x;
    if (t == 0) {
        *p.ticket = 0u;
        *p.fb_count = 0u;
        *p.ws_params = p;
    }
    if (t < 16) p.acc[t] = 0ull;
    if (p.perm)
        for (int b = t; b <= SORT_BINS; b += blockDim.x) p.order_hist[b] = 0u;
}

// ---- dispatch order ------------------------------------------------------
// Rays near the photon ring take the most steps; the persistent waves finish
// soonest when those go out first and the cheap rays fill the tail.  The
// slots are sorted by the bin of the distance from the ring (a counting sort over
// SORT_BINS bins).  Every ray's arithmetic is independent of the lane and
// wave that runs it, so outputs do not change.
//
// Rays go out in groups of consecutive ids (keyed by the group's middle
// ray), so the outputs of neighbouring pixels, which share cache lines, are
// written close together in time and merge in L2 instead of reaching HBM as
// many partial-line writes.  Where there are few rays per lane a group of 32 mixes
// long and short ones: 32 and 16 rays give 2.65/2.57 ms on the 96x96 ring and
// 6.35/5.87 on a 625x600 norm map; with many the writes count, 15.46/15.50 on the
// 1024x1024 ring and 9.83/9.88 on the 1365x683 disk.  The q-metric, whose ring is
// no exact one, keeps groups of 32 (477x361: 6.12 ms, with 16 6.25).
constexpr int64_t ORDER_SMALL = int64_t{1} << 19;
__device__ __forceinline__ int64_t order_group(const Params& P, int64_t ray) {
    const int shift = P.n_rays < ORDER_SMALL && P.images[0].metric == KT_METRIC_KERR ? 4 : 5;
    return min(((ray >> shift) << shift) + (int64_t{1} << (shift - 1)), static_cast<int64_t>(P.n_rays) - 1);
}

// How far a Kerr ray is from one that is caught on a spherical photon orbit, in
// units of M: the difference of sqrt(kappa) = (p_theta^2 + (L / sin theta - a E sin
// theta)^2)^(1/2) / E and its critical value for the ray's L / E.  The spherical
// orbit of radius r has (r - M)(r^2 + a^2 - a L / E) = 2 r Delta, a cubic in r
// (Bardeen 1973), and kappa = 4 r^2 Delta / (r - M)^2; outside the range of L / E
// that has one, the equatorial photon orbit's value continues it.  Single precision
// and the hardware's sine: it only orders the dispatch.  All lengths are divided by
// M first: powers of r reach past the range of single precision where M is 1e13,
// and rays then fall into bins by chance (512x512 ring 6.8 ms instead of 5.3).
// Against the circle of a hole without spin: a 625x600 norm map at a = 0.98 8.25 ->
// 5.87 ms, by Bulirsch-Stoer 3.52 -> 3.30, a 1000x1000 one 8.39 -> 7.58, the 640x640
// mixed disk 8.07 -> 7.86; rings and disks at 60 degrees within 0.5%.
__device__ __forceinline__ float critical_distance(const Image& im, double x, double y) {
    const double iM = rcp(im.M);
    const float a = static_cast<float>(im.a * iM), si = __sinf(static_cast<float>(im.incl));
    const float iE = __frcp_rn(static_cast<float>(im.E0 + x * im.cE)), l = static_cast<float>(x * im.cL * iM) * iE;
    const float pth = static_cast<float>(y * im.cth * iM) * iE, t = __fdividef(l, si) - a * si;
    const float third = acosf(fminf(fabsf(a), 1.0f)) * (2.0f / 3.0f);
    const float r_pro = 2.0f * (1.0f + __cosf(2.0943951f - third)), r_ret = 2.0f * (1.0f + __cosf(third));
    const float b = a * (a + l), c = a * (a - l);
    float r = 0.5f * (3.0f + sqrtf(fmaxf(9.0f - 4.0f * b, 0.0f)));
    for (int k = 0; k < 4; ++k) {
        const float f = ((r - 3.0f) * r + b) * r + c, df = (3.0f * r - 6.0f) * r + b;
        r = fminf(fmaxf(r - __fdividef(f, df), r_pro), r_ret);
    }
    const float q = __fdividef(1.0f, fmaxf(r - 1.0f, 1e-4f));
    const float crit = 2.0f * r * sqrtf(fmaxf(1.0f - (1.0f - a) * (1.0f + a) * q * q, 0.0f));
    return fabsf(sqrtf(pth * pth + t * t) - crit);
}

struct RingKey {
    const Params* p;  // the workspace copy
    __device__ int operator()(int64_t ray) const {
        const Params& P = *p;
        ray = order_group(P, ray);
        const Image* im = P.images;
        int64_t pix = ray;
        if (P.n_images > 1) {
            im = &P.images[find_image(P, ray)];
            pix = ray - im->first;
        }
        const int32_t j = static_cast<int32_t>(pix / im->nx);
        const int32_t i = static_cast<int32_t>(pix - static_cast<int64_t>(j) * im->nx);
        const double x = -im->fov_x + (static_cast<double>(i) + 0.5) * im->dx;
        const double y = -im->fov_y + (static_cast<double>(j) + 0.5) * im->dy;
        double d = fabs(sqrt(fma(x, x, y * y)) - im->rho_ring);
        if (im->metric == KT_METRIC_KERR && im->a != 0.0 && im->rho_ring > 0.0) {
            const double kerr = critical_distance(*im, x, y) * (im->rho_ring / 5.196152422706632);
            if (kerr >= 0.0) d = kerr;  // NaN for an observer on the axis
        }
        d *= im->order_scale;
        return d < static_cast<double>(SORT_BINS - 1) ? static_cast<int>(d) : SORT_BINS - 1;
    }
};

// Copy a chunk of the image table into device memory (the table travels in
// kernel arguments, so nothing on the host has to outlive the call).
constexpr int UPLOAD_CHUNK = 12;
struct ImageChunk {
    Image im[UPLOAD_CHUNK];
    int32_t n, base;
};
static_assert(sizeof(ImageChunk) <= 3900, "image chunk must fit the kernel-argument limit");

__global__ void upload_images_kernel(const ImageChunk c, Image* dev) {
    const int t = threadIdx.x;
    if (t < c.n) dev[c.base + t] = c.im[t];
}

__global__ void reset_ticket_kernel(uint32_t* ticket) {
    if (threadIdx.x == 0) *ticket = 0u;
}

// Odd multiples of pi that are <= v.
__device__ __forceinline__ double odd_pi_count(double v) {
    constexpr double PI = 3.14159265358979323846;
    return floor((v + PI) / (2.0 * PI));
}

// Ring flags, within each image: an odd multiple of pi between a pixel's
// deflection and its +i or +j neighbour's.
__global__ void ring_kernel(const Params* pp) {
    const Params& P = *pp;
    const double* __restrict__ defl = P.out.deflection;
    uint8_t* __restrict__ ring = P.out.ring;
    const int64_t n = P.n_rays;
    for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < n;
         p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const Image& im = P.images[find_image(P, p)];
        const int64_t pix = p - im.first;
        const int32_t nx = im.nx;
        const int32_t j = static_cast<int32_t>(pix / nx);
        const int32_t i = static_cast<int32_t>(pix - static_cast<int64_t>(j) * nx);
        const double d = defl[p];
        uint8_t flag = 0;
        if (isfinite(d)) {
            const double k = odd_pi_count(d);
            if (i + 1 < nx && isfinite(defl[p + 1]) && odd_pi_count(defl[p + 1]) != k) flag = 1;
            if (j + 1 < im.ny && isfinite(defl[p + nx]) && odd_pi_count(defl[p + nx]) != k) flag = 1;
        }
        ring[p] = flag;
    }
}

// Celestial-sphere codes from the located crossings (theta_f, phi_f).
__global__ void sky_kernel(const Params* pp) {
    const Params& P = *pp;
    const int64_t n = P.n_rays;
    for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < n;
         k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        uint8_t code = KT_SKY_NONE;
        if (P.out.fate[k] == KT_FATE_ESCAPED) {
            const Image& im = P.images[find_image(P, k)];
            if (im.sky_on) code = sky_code(P.out.theta_f[k], P.out.phi_f[k], im.grid_deg, im.line_deg);
        }
        P.out.sky[k] = code;
    }
}

// Fate histogram into acc[8..15].
__global__ void fate_hist_kernel(const uint8_t* __restrict__ fate, int64_t n, unsigned long long* acc) {
    // per-lane counts, summed over the wave with shuffles: most fates are
    // equal, so atomics per element would serialise on one LDS word
    __shared__ unsigned int hist[8];
    if (threadIdx.x < 8) hist[threadIdx.x] = 0u;
    __syncthreads();
    unsigned int c[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    for (int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; p < n;
         p += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int f = fate[p] & 7;
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] += f == k ? 1u : 0u;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        unsigned int v = c[k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += static_cast<unsigned int>(__shfl_xor(static_cast<int>(v), off));
        if (__lane_id() == 0 && v) atomicAdd(&hist[k], v);
    }
    __syncthreads();
    if (threadIdx.x < 8 && hist[threadIdx.x]) atomicAdd(acc + 8 + threadIdx.x, static_cast<unsigned long long>(hist[threadIdx.x]));
}

// One reading of the GPU's constant-rate wall clock into acc[slot].  Enqueued
// just before the first trace launch and just after the last one when a
// render asks for statistics, so the trace kernels themselves carry no timing
// code.
__global__ void stamp_kernel(unsigned long long* acc, int slot) {
    if (threadIdx.x == 0) acc[slot] = static_cast<unsigned long long>(wall_clock64());
}

__global__ void stats_kernel(const unsigned long long* acc, const uint32_t* fb_count, int64_t n_rays,
                             double wall_khz, kt_stats* out) {
    if (threadIdx.x == 0) {
        out->rays = static_cast<uint64_t>(n_rays);
        out->evals = acc[ACC_EVALS];
        out->evals_fp32 = acc[ACC_EVALS_FP32];
        out->fallback_rays = *fb_count;
        for (int k = 0; k < 8; ++k) out->fate_count[k] = acc[8 + k];
        const unsigned long long t0 = acc[ACC_T0], t1 = acc[ACC_T1];
        out->trace_ms = (wall_khz > 0.0 && t1 > t0) ? static_cast<double>(t1 - t0) / wall_khz : 0.0;
    }
}

__global__ void init_rays_kernel(const Image im, int64_t n, double* state, uint8_t* invalid) {
    for (int64_t k = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; k < n;
         k += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        double z[5], E, L;
        const bool ok = camera_state(im, static_cast<int32_t>(k), z, &E, &L);
        for (int c = 0; c < 5; ++c) state[c * n + k] = z[c];
        state[5 * n + k] = E;
        state[6 * n + k] = L;
        invalid[k] = ok ? 0 : 1;
    }
}

#endif  // !KT_TRACE_ONLY

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

static int check_launch() { return hipGetLastError() == hipSuccess ? 0 : -1; }

#if !KT_TRACE_ONLY
static int small_grid(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    if (g > 4096) g = 4096;
    return g < 1 ? 1 : static_cast<int>(g);
}

int launch_ws_init(const Params& p, void* stream) {
    hipLaunchKernelGGL(ws_init_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), p);
    return check_launch();
}

int launch_order(const Params& p, void* stream) {
    const SortBufs b{p.n_rays, p.order_hist, p.order_bins, p.perm};
    return launch_sort(b, RingKey{p.ws_params}, static_cast<hipStream_t>(stream));
}

int launch_reset_ticket(const Params& p, void* stream) {
    hipLaunchKernelGGL(reset_ticket_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                       p.ticket);
    return check_launch();
}

int launch_upload_images(const Image* host, int32_t n, Image* dev, void* stream) {
    for (int32_t base = 0; base < n; base += UPLOAD_CHUNK) {
        ImageChunk c;
        c.n = n - base < UPLOAD_CHUNK ? n - base : UPLOAD_CHUNK;
        c.base = base;
        for (int t = 0; t < c.n; ++t) c.im[t] = host[base + t];
        hipLaunchKernelGGL(upload_images_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), c, dev);
        if (check_launch()) return -1;
    }
    return 0;
}

#endif  // !KT_TRACE_ONLY

static Hot make_hot(const Params& p) {
    const Image& im = p.img0;  // batch renders take the per-image values from the table
    Hot hp;
    hp.M = im.M;
    hp.a = im.a;
    hp.a2 = im.a2;
    hp.two_a2 = im.two_a2;
    if (im.metric == KT_METRIC_Q) {
        hp.a = im.q;
        hp.a2 = im.q * (2.0 + im.q);
        hp.two_a2 = 0.0;
    }
    hp.rtol = p.rtol;
    hp.atol = p.atol;
    hp.r_cap = im.r_cap;
    hp.r_esc = im.r_esc;
    hp.h_budget = p.h_budget;
    hp.r_switch = p.r_switch;
    hp.feat = image_features(im);
    hp.max_steps = static_cast<int32_t>(p.max_steps);
    hp.max_evals = static_cast<int32_t>(p.max_evals);
    // one per lane; as a constant in the kernel it costs the q-metric form 1.5%
    // (477x361 rays 5.31 -> 5.40 ms), whose registers the compiler then deals otherwise
    hp.first = 64;
    hp.min_idle = p.min_idle;
    hp.acc = p.acc;
    hp.store = p.adj.store;
    hp.sweep_only = 0;
    hp.cold = p.ws_params;
    return hp;
}

// The single-image Dormand-Prince FP64 kernel with the image's features
// fixed at compile time (every other form reads them at run time), and for a
// hole without spin the right-hand side without its terms: 2048x2048 disk
// 42.8 -> 40.6 ms, 333x333 ring 2.81 -> 2.63.  (RK4 shadows gain nothing: 250x300
// rays 2.72 and 2.71 ms, bound by the chain of dependent operations.)
template <int FEAT>
static void launch_dp45_feat(const Hot& hp, int grid, int block, hipStream_t s) {
    if (hp.a == 0.0)
        hipLaunchKernelGGL((trace_kernel<KT_DP45, KT_FP64, false, METRIC_SCHWARZSCHILD, FEAT>), dim3(grid), dim3(block),
                           0, s, hp);
    else
        hipLaunchKernelGGL((trace_kernel<KT_DP45, KT_FP64, false, METRIC_KERR, FEAT>), dim3(grid), dim3(block), 0, s, hp);
}

template <int METHOD, int PREC>
static void launch_variant(const Params& p, const Hot& hp, int grid, int block, hipStream_t s) {
    if constexpr (PREC == KT_FP64 && METHOD != KT_RK4_S) {
        if (p.img0.metric == KT_METRIC_Q) {
            hipLaunchKernelGGL((trace_kernel<METHOD, PREC, false, METRIC_Q>), dim3(grid), dim3(block), 0, s, hp);
            return;
        }
    }
    if constexpr (METHOD == KT_DP45 && PREC == KT_FP64) {
        if (p.n_images == 1) {
            switch (hp.feat & 7) {
            case 0: launch_dp45_feat<0>(hp, grid, block, s); return;
            case 1: launch_dp45_feat<1>(hp, grid, block, s); return;
            case 2: launch_dp45_feat<2>(hp, grid, block, s); return;
            case 3: launch_dp45_feat<3>(hp, grid, block, s); return;
            case 4: launch_dp45_feat<4>(hp, grid, block, s); return;
            case 5: launch_dp45_feat<5>(hp, grid, block, s); return;
            case 6: launch_dp45_feat<6>(hp, grid, block, s); return;
            default: launch_dp45_feat<7>(hp, grid, block, s); return;
            }
        }
    }
    if (p.n_images > 1)
        hipLaunchKernelGGL((trace_kernel<METHOD, PREC, true>), dim3(grid), dim3(block), 0, s, hp);
    else
        hipLaunchKernelGGL((trace_kernel<METHOD, PREC, false>), dim3(grid), dim3(block), 0, s, hp);
}

int launch_trace(const Params& p, int grid, int block, void* stream) {
    const Hot hp = make_hot(p);
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (p.method) {
    case KT_DP45:
        if (p.precision == KT_MIXED)
            launch_variant<KT_DP45, KT_MIXED>(p, hp, grid, block, s);
        else
            launch_variant<KT_DP45, KT_FP64>(p, hp, grid, block, s);
        break;
    case KT_RKF45: launch_variant<KT_RKF45, KT_FP64>(p, hp, grid, block, s); break;
    case KT_CK45: launch_variant<KT_CK45, KT_FP64>(p, hp, grid, block, s); break;
    case KT_BS: launch_variant<KT_BS, KT_FP64>(p, hp, grid, block, s); break;
    case KT_BS_RAT: launch_variant<KT_BS_RAT, KT_FP64>(p, hp, grid, block, s); break;
    default: launch_variant<KT_RK4_S, KT_FP64>(p, hp, grid, block, s); break;
    }
    return check_launch();
}

#if !KT_TRACE_ONLY
int launch_fallback_list(const Params& p, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(fallback_list_kernel, dim3(small_grid(p.n_rays, 256)), dim3(256), 0, s, p.need_fb,
                       static_cast<int64_t>(p.n_rays), p.fb_list, p.fb_count);
    if (check_launch()) return -1;
    hipLaunchKernelGGL(to_fallback_kernel, dim3(1), dim3(64), 0, s, p.ws_params);
    return check_launch();
}

#endif  // !KT_TRACE_ONLY

int launch_trace_fallback(const Params& p, int grid, int block, void* stream) {
    const Hot hp = make_hot(p);
    launch_variant<KT_DP45, KT_FP64>(p, hp, grid, block, static_cast<hipStream_t>(stream));
    return check_launch();
}

template <int METHOD, int PREC>
static hipError_t occupancy_variant(const Params& p, int* nb, int block) {
    if constexpr (PREC == KT_FP64 && METHOD != KT_RK4_S) {
        if (p.img0.metric == KT_METRIC_Q)
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, trace_kernel<METHOD, PREC, false, METRIC_Q>, block, 0);
    }
    if (p.n_images > 1)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, trace_kernel<METHOD, PREC, true>, block, 0);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(nb, trace_kernel<METHOD, PREC, false>, block, 0);
}

int trace_max_blocks_per_cu(const Params& p, int block) {
    int nb = 0;
    hipError_t e;
    switch (p.method) {
    case KT_DP45:
        e = p.precision == KT_MIXED ? occupancy_variant<KT_DP45, KT_MIXED>(p, &nb, block)
                                    : occupancy_variant<KT_DP45, KT_FP64>(p, &nb, block);
        break;
    case KT_RKF45: e = occupancy_variant<KT_RKF45, KT_FP64>(p, &nb, block); break;
    case KT_CK45: e = occupancy_variant<KT_CK45, KT_FP64>(p, &nb, block); break;
    case KT_BS: e = occupancy_variant<KT_BS, KT_FP64>(p, &nb, block); break;
    case KT_BS_RAT: e = occupancy_variant<KT_BS_RAT, KT_FP64>(p, &nb, block); break;
    default: e = occupancy_variant<KT_RK4_S, KT_FP64>(p, &nb, block); break;
    }
    return (e == hipSuccess && nb > 0) ? nb : 1;
}

#if !KT_TRACE_ONLY
int launch_trace_store(const Params& p, int grid, int sweep_only, void* stream) {
    Hot hp = make_hot(p);
    hp.sweep_only = sweep_only;
    hipLaunchKernelGGL((trace_kernel<KT_DP45, KT_FP64, false, METRIC_KERR, FEAT_DISK, true>), dim3(grid), dim3(BLOCK_MAX), 0,
                       static_cast<hipStream_t>(stream), hp);
    return check_launch();
}

int launch_disk_obs(const Params& p, void* stream) {
    hipLaunchKernelGGL(disk_obs_kernel, dim3(small_grid(p.n_rays, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), p.ws_params);
    return check_launch();
}

int launch_ring(const Params& p, void* stream) {
    hipLaunchKernelGGL(ring_kernel, dim3(small_grid(p.n_rays, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), p.ws_params);
    return check_launch();
}

int launch_sky(const Params& p, void* stream) {
    hipLaunchKernelGGL(sky_kernel, dim3(small_grid(p.n_rays, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), p.ws_params);
    return check_launch();
}

int launch_stats(const Params& p, void* stream) {
    const int64_t n = p.n_rays;
    // few blocks: each ends with one 64-bit atomic per fate on the same
    // eight words, and thousands of those serialise
    const int grid = small_grid(n, 256) < 256 ? small_grid(n, 256) : 256;
    hipLaunchKernelGGL(fate_hist_kernel, dim3(grid), dim3(256), 0,
                       static_cast<hipStream_t>(stream), p.out.fate, n, p.acc);
    if (check_launch()) return -1;
    hipLaunchKernelGGL(stats_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), p.acc,
                       p.fb_count, n, p.wall_khz, p.out.stats);
    return check_launch();
}

int launch_stamp(const Params& p, int slot, void* stream) {
    hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), p.acc, slot);
    return check_launch();
}

int launch_init_rays(const Params& p, double* state, uint8_t* invalid, void* stream) {
    hipLaunchKernelGGL(init_rays_kernel, dim3(small_grid(p.n_rays, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), p.img0, static_cast<int64_t>(p.n_rays), state, invalid);
    return check_launch();
}

#endif  // !KT_TRACE_ONLY

}  // namespace KT_TRACE_NS
