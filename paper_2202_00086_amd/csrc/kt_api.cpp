// kt_api.cpp -- host runtime and C ABI of the Kerr ray tracer: argument
// validation, per-image camera constants, workspace layout and the launch
// sequence on the caller's stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "kerrtrace.h"
#include "kt_dual.h"
#include "kt_internal.h"

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

}  // namespace

namespace kt {
int set_error(int code, const char* msg) {
    std::snprintf(g_err, sizeof g_err, "%s", msg);
    return code;
}
}  // namespace kt

namespace {

bool finite_all(std::initializer_list<double> v) {
    for (double x : v)
        if (!std::isfinite(x)) return false;
    return true;
}

// Compute units of the current device (cached per device id).
int device_cus() {
    static std::mutex mu;
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    std::lock_guard<std::mutex> lk(mu);
    if (cache[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

// The wall clock rate of the current device in kHz (cached per device id;
// 0 when the device reports none).
double device_wall_khz() {
    static std::mutex mu;
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0.0;
    std::lock_guard<std::mutex> lk(mu);
    if (cache[dev] == 0) {
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) khz = -1;
        cache[dev] = khz;
    }
    return cache[dev] > 0 ? static_cast<double>(cache[dev]) : 0.0;
}

// Waves per SIMD of a persistent launch without a shape of its own, and with
// them which build of the trace kernels runs (both give the same outputs bit
// for bit): 3 waves mean the 3-wave form (kt_trace_w3.hip).  More waves keep
// the VALU busier, but each ray then takes longer in wall time, and the
// launch ends with its longest rays, so the choice goes by the rays per lane
// of a one-wave grid (65536 lanes on 256 CUs).  Measured, ms per image at
// 1 / 2 / 3 waves, on ring, disk (a = 0.9) and disk (a = 0) images:
//   448x448 (3.1 rays per lane)  4.04/4.26/5.43  2.80/3.43/4.32  2.82/2.97/3.65
//   512x512 (4)                  5.09/5.40/6.36  3.37/3.59/4.63  3.50/3.56/4.00
//   576x576 (5.1)                6.18/5.98/6.54  4.09/4.19/4.74  4.29/4.30/4.82
//   768x768 (9)                  10.4/9.36/9.69  6.89/6.48/6.79  7.26/6.56/6.81
//   1024x1024 (16)               17.9/15.0/15.4  11.7/10.4/10.7  12.5/10.5/10.7
//   1448x1448 (32)               -/28.9/29.0                     -/20.2/20.0
//   2048x2048 (64)               -/57.0/56.8     -/38.9/38.5     -/39.6/39.0
// The other Runge-Kutta pairs, the mixed form, the q-metric (12.4 rays per lane
// 16.9/17.8 at 2/3 waves, 22 28.8/28.9) and batches (117: 75.2/73.7) cross over
// there too.  The 3-wave build has no registers for the paired midpoint substeps
// of Bulirsch-Stoer, which never takes it; 1 / 2 / 3 waves on the ring and on a
// norm map of a = 0.98 seen edge on, whose longest rays take more of the time:
//   625x625 (6)     4.80/4.38/5.23  3.48/4.41/5.44
//   768x768 (9)     7.08/6.15/7.02  4.99/5.73/6.30
//   1024x1024 (16)  12.3/10.3/11.5  8.47/8.89/10.3
//   1200x1200 (22)  16.8/13.9/15.5  11.5/10.7/12.8
// No one line suits both: up to 9 rays per lane two waves would win 9-13% on rings
// and lose 15-27% on edge-on images of fast spin, which the line is drawn for.
constexpr int64_t ONE_WAVE_MAX_RAYS_PER_LANE = 4, THREE_WAVE_MIN_RAYS_PER_LANE = 32, BS_ONE_WAVE_MAX_RAYS_PER_LANE = 9;

int waves_per_simd(int32_t method, int64_t n_rays) {
    const int64_t lanes = static_cast<int64_t>(device_cus()) * 4 * 64;
    if (method == KT_BS || method == KT_BS_RAT) return n_rays <= BS_ONE_WAVE_MAX_RAYS_PER_LANE * lanes ? 1 : 2;
    if (n_rays <= ONE_WAVE_MAX_RAYS_PER_LANE * lanes) return 1;
    return n_rays >= THREE_WAVE_MIN_RAYS_PER_LANE * lanes ? 3 : 2;
}

constexpr int32_t DEFAULT_BATCH = 4;  // ids per ticket fetch after a wave's first, at least one per idle lane

// The grid of a trace launch of about n_rays / share rays in a render of
// n_rays, the build it runs (a shape of 3 or more waves per SIMD is the 3-wave
// form) and the idle lanes that a refill waits for.
struct Shape {
    bool w3;
    int grid, min_idle;
};

// KT_MIXED's re-run pass is shaped for a sixth of the image's rays, about what it
// takes at budgets of use (13-24% of the 1024x1024 ring at 1e-10, by r_switch, 7% of a
// 2048x2048 disk; only the device knows the number).  At the image's shape, two waves per
// SIMD, the 640x640 disk's pass took 2.7 ms, at one wave 1.7.  A budget that no ray
// meets re-runs every ray that used single precision: the 1024x1024 ring at 0 then
// takes 23.4 ms in all, as at 1e-10 (23.2).
constexpr int MIXED_RERUN_SHARE = 6;

Shape launch_shape(const kt::Params& p, const kt_launch& ln, int64_t n_rays, int share = 1) {
    const int64_t lane_grid = (n_rays + ln.block - 1) / ln.block;
    const int waves =
        ln.blocks_per_cu > 0 ? ln.blocks_per_cu * ln.block / 256 : waves_per_simd(p.method, n_rays / share);
    Shape s;
    s.w3 = ln.persistent && waves >= 3;
    s.min_idle = waves <= 1 ? 8 : 4;
    int64_t grid = lane_grid;
    if (ln.persistent) {
        int per_cu = ln.blocks_per_cu;
        if (per_cu == 0) {
            const int fit =
                s.w3 ? kt_w3::trace_max_blocks_per_cu(p, ln.block) : kt::trace_max_blocks_per_cu(p, ln.block);
            per_cu = std::min(fit, waves * 256 / ln.block);
        }
        grid = std::min<int64_t>(lane_grid, static_cast<int64_t>(device_cus()) * per_cu);
    }
    s.grid = static_cast<int>(std::max<int64_t>(grid, 1));
    return s;
}

double horizon(const kt_spacetime* st) {
    if (st->metric == KT_METRIC_Q) return 2.0 * st->M;
    return st->M + std::sqrt(st->M * st->M - st->a * st->a);
}

int validate_common(const kt_camera* cam, const kt_spacetime* st) {
    if (!cam || !st) return fail(KT_EINVAL, "camera and spacetime must not be NULL");
    if (!finite_all({cam->r_obs, cam->incl, cam->fov_x, cam->fov_y, st->M, st->a}))
        return fail(KT_EINVAL, "non-finite camera or spacetime parameter");
    if (st->metric != KT_METRIC_KERR && st->metric != KT_METRIC_Q)
        return fail(KT_EINVAL, "unknown metric %d", st->metric);
    if (st->metric == KT_METRIC_Q) {
        if (!std::isfinite(st->q) || !(st->q > -1.0)) return fail(KT_EINVAL, "the q-metric needs finite q > -1");
        if (!(st->M > 0.0)) return fail(KT_EINVAL, "the q-metric needs M > 0");
        if (st->a != 0.0) return fail(KT_EINVAL, "the q-metric is static: a must be 0");
    }
    if (!(st->M >= 0.0)) return fail(KT_EINVAL, "M must be >= 0 (got %g)", st->M);
    if (st->a * st->a > st->M * st->M) return fail(KT_EINVAL, "|a| must be <= M (a=%g, M=%g)", st->a, st->M);
    if (!(cam->incl > 0.0 && cam->incl < M_PI))
        return fail(KT_EINVAL, "incl must lie in (0, pi) (got %g)", cam->incl);
    if (!(cam->fov_x > 0.0 && cam->fov_y > 0.0)) return fail(KT_EINVAL, "fov_x and fov_y must be > 0");
    if (cam->nx < 1 || cam->ny < 1) return fail(KT_EINVAL, "nx and ny must be >= 1");
    if (static_cast<int64_t>(cam->nx) * cam->ny >= (int64_t{1} << 31))
        return fail(KT_EINVAL, "nx*ny must be < 2^31");
    return KT_OK;
}

// Per-image camera constants at (r_obs, incl) from the Kerr metric
// (eq:Kerr) and the observer tetrad (eq:matrix, second eq:momentums).
void camera_constants(const kt_camera* cam, const kt_spacetime* st, kt::Image& im) {
    const double M = st->M, a = st->a, r0 = cam->r_obs;
    const double s = std::sin(cam->incl), c = std::cos(cam->incl);
    im.metric = st->metric;
    im.q = st->q;
    if (st->metric == KT_METRIC_Q) {
        // static observer of the q-metric: E0 = sqrt(-g_tt), no frame dragging
        const double f = 1.0 - 2.0 * M / r0, q = st->q, P = q * (2.0 + q);
        const double D = 1.0 + M * M * s * s / (r0 * r0 - 2.0 * M * r0);
        const double fq = std::pow(f, q), DmP = std::pow(D, -P);
        im.E0 = std::sqrt(f * fq);
        im.cE = 0.0;
        im.cL = -std::sqrt(r0 * r0 * s * s / fq) / r0;
        im.cth = std::sqrt(r0 * r0 * DmP / fq) / r0;
        im.g_rr = DmP / (f * fq);
        im.r0 = r0;
        im.incl = cam->incl;
        im.fov_x = cam->fov_x;
        im.fov_y = cam->fov_y;
        im.dx = 2.0 * cam->fov_x / cam->nx;
        im.dy = 2.0 * cam->fov_y / cam->ny;
        im.nx = cam->nx;
        im.ny = cam->ny;
        im.M = M;
        im.a = im.a2 = im.two_a2 = 0.0;
        return;
    }
    const double Sig = r0 * r0 + a * a * c * c;
    const double Del = r0 * r0 - 2.0 * M * r0 + a * a;
    const double g_tph = -2.0 * M * a * r0 * s * s / Sig;
    const double g_phph = s * s * (r0 * r0 + a * a + 2.0 * M * a * a * r0 * s * s / Sig);
    // g_tph^2 - g_tt g_phph = Delta sin^2 for Kerr, so A_t = sqrt(g_phph / (Delta sin^2))
    const double At = std::sqrt(g_phph / (Del * s * s));
    im.E0 = 1.0 / At;
    im.cE = g_tph / (r0 * std::sqrt(g_phph));
    im.cL = -std::sqrt(g_phph) / r0;
    im.cth = std::sqrt(Sig) / r0;
    im.g_rr = Sig / Del;
    im.r0 = r0;
    im.incl = cam->incl;
    im.fov_x = cam->fov_x;
    im.fov_y = cam->fov_y;
    im.dx = 2.0 * cam->fov_x / cam->nx;
    im.dy = 2.0 * cam->fov_y / cam->ny;
    im.nx = cam->nx;
    im.ny = cam->ny;
    im.M = M;
    im.a = a;
    im.a2 = a * a;
    im.two_a2 = 2.0 * a * a;
}

// Image-plane radius of the photon ring seen by a static observer at r_obs:
// the critical impact parameter (sqrt(27) M for Kerr at a = 0; for the
// q-metric M (3+2q) ((3+2q)/(1+2q))^((1+2q)/2), which needs q > -1/2)
// scaled by the observer's redshift factor.  It only orders the dispatch,
// so the spin's distortion of the ring is left out.
double ring_radius(const kt_camera* cam, const kt_spacetime* st) {
    const double M = st->M, r0 = cam->r_obs;
    if (!(M > 0.0)) return 0.0;
    const double f = std::max(0.0, 1.0 - 2.0 * M / r0);
    if (st->metric == KT_METRIC_Q) {
        const double q = st->q, e = 0.5 + q;
        if (!(e > 0.0)) return 0.0;
        return M * (3.0 + 2.0 * q) * std::pow((3.0 + 2.0 * q) / (1.0 + 2.0 * q), e) * std::pow(f, e);
    }
    return std::sqrt(27.0 * f) * M;
}

// Derivatives of the camera constants (E0, cE, cL, cth, g_rr) with respect to
// (a, incl): the formulas of camera_constants carried through dual numbers.
void camera_constant_derivs(const kt_camera* cam, const kt_spacetime* st, double d[5][2]) {
    using D = kt::Dual<2>;
    const D a = D::var(st->a, 0), inc = D::var(cam->incl, 1);
    const double M = st->M, r0 = cam->r_obs;
    D s, c;
    kt::dsincos(inc, &s, &c);
    const D Sig = r0 * r0 + a * a * c * c;
    const D Del = r0 * r0 - 2.0 * M * r0 + a * a;
    const D g_tph = -2.0 * M * a * r0 * s * s / Sig;
    const D g_phph = s * s * (r0 * r0 + a * a + 2.0 * M * a * a * r0 * s * s / Sig);
    const D At = kt::dsqrt(g_phph / (Del * s * s));
    const D v[5] = {1.0 / At, g_tph / (r0 * kt::dsqrt(g_phph)), -kt::dsqrt(g_phph) / r0, kt::dsqrt(Sig) / r0,
                    Sig / Del};
    for (int i = 0; i < 5; ++i)
        for (int k = 0; k < 2; ++k) d[i][k] = v[i].d[k];
}

int validate_integ(const kt_integrator* integ) {
    if (integ->method < KT_RK4_S || integ->method > KT_BS_RAT)
        return fail(KT_EINVAL, "unknown integrator method %d", integ->method);
    if (integ->precision != KT_FP64 && integ->precision != KT_MIXED)
        return fail(KT_EINVAL, "unknown precision %d", integ->precision);
    if (integ->precision == KT_MIXED) {
        if (integ->method != KT_DP45) return fail(KT_EINVAL, "KT_MIXED needs method KT_DP45");
        if (!(integ->h_budget >= 0.0) || !(integ->r_switch > 0.0))
            return fail(KT_EINVAL, "KT_MIXED needs h_budget >= 0 and r_switch > 0");
    }
    if (!finite_all({integ->h_fixed, integ->rtol, integ->atol, integ->h_init, integ->capture_buffer,
                     integ->r_escape, integ->h_budget, integ->r_switch}))
        return fail(KT_EINVAL, "non-finite integrator parameter");
    if (integ->method == KT_RK4_S && !(integ->h_fixed > 0.0))
        return fail(KT_EINVAL, "h_fixed must be > 0");
    if (integ->method != KT_RK4_S && !(integ->rtol > 0.0 && integ->atol > 0.0 && integ->h_init > 0.0))
        return fail(KT_EINVAL, "rtol, atol and h_init must be > 0");
    if (!(integ->capture_buffer >= 0.0)) return fail(KT_EINVAL, "capture_buffer must be >= 0");
    if (integ->max_steps < 1 || integ->max_steps > 100000000)
        return fail(KT_EINVAL, "max_steps must lie in [1, 1e8]");
    if (kt::adj_ck_shift(integ->checkpoint_every) < 0)
        return fail(KT_EINVAL, "checkpoint_every must be 0 or a power of two in [1, 1024] (got %d)",
                    integ->checkpoint_every);
    if (integ->split_above < -1) return fail(KT_EINVAL, "split_above must be -1, 0 or a step count (got %d)",
                                             integ->split_above);
    return KT_OK;
}

// Validate one image and fill its table entry (everything but `first`).
int make_image(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
               const kt_source* source, const kt_integrator* integ, bool want_ring, kt::Image& im) {
    int rc = validate_common(camera, spacetime);
    if (rc) return rc;
    std::memset(&im, 0, sizeof im);
    camera_constants(camera, spacetime, im);
    const double r_plus = horizon(spacetime);
    if (spacetime->metric == KT_METRIC_Q) {
        if (integ->method == KT_RK4_S || integ->precision != KT_FP64)
            return fail(KT_EINVAL, "the q-metric runs with the adaptive FP64 schemes");
        if (disk && disk->enabled) return fail(KT_EINVAL, "the disk's redshift model needs the Kerr metric");
    }
    const double r_cap = r_plus + integ->capture_buffer;
    if (!(camera->r_obs > r_cap)) return fail(KT_EINVAL, "r_obs must exceed r_+ + capture_buffer");
    // e.g. r_obs so large that r_obs^2 overflows, or a q-metric power that
    // under- or overflows
    if (!finite_all({im.E0, im.cE, im.cL, im.cth, im.g_rr, im.dx, im.dy}) || !(im.E0 > 0.0))
        return fail(KT_EINVAL, "camera constants are not finite (r_obs %g, q %g out of range)", camera->r_obs,
                    spacetime->q);
    const double r_esc = integ->r_escape == 0.0 ? 1.1 * camera->r_obs : integ->r_escape;
    if (!(r_esc > camera->r_obs)) return fail(KT_EINVAL, "r_escape must exceed r_obs");
    im.r_cap = r_cap;
    im.r_esc = r_esc;
    im.rho_ring = ring_radius(camera, spacetime);
    {
        const double rho_max = std::sqrt(camera->fov_x * camera->fov_x + camera->fov_y * camera->fov_y);
        const double span = std::max(im.rho_ring, rho_max - im.rho_ring);
        im.order_scale = kt::SORT_BINS / span;
    }

    const bool disk_on = disk && disk->enabled;
    if (disk_on) {
        if (!finite_all({disk->r_in, disk->r_out, disk->emis_index}))
            return fail(KT_EINVAL, "non-finite disk parameter");
        if (!(disk->r_in > r_plus && disk->r_out > disk->r_in))
            return fail(KT_EINVAL, "disk needs r_+ < r_in < r_out");
        if (disk->rotation != KT_ROT_KEPLER && disk->rotation != KT_ROT_L0)
            return fail(KT_EINVAL, "unknown disk rotation %d", disk->rotation);
        if (disk->rotation == KT_ROT_L0 && !std::isfinite(disk->l0))
            return fail(KT_EINVAL, "l0 must be finite");
        if (disk->emissivity != KT_EMIS_POWER && disk->emissivity != KT_EMIS_TAPERED)
            return fail(KT_EINVAL, "unknown disk emissivity %d", disk->emissivity);
        if (disk->emissivity == KT_EMIS_TAPERED && !(spacetime->M > 0.0))
            return fail(KT_EINVAL, "the tapered emissivity needs M > 0");
        im.disk_on = 1;
        im.r_in = disk->r_in;
        im.r_out = disk->r_out;
        im.emis_q = disk->emis_index;
        im.rotation = disk->rotation;
        im.l0 = disk->l0;
        im.emis_model = disk->emissivity;
    }
    const bool src_on = source && source->enabled;
    if (src_on) {
        if (!std::isfinite(source->r_src) || !(source->r_src > r_cap))
            return fail(KT_EINVAL, "r_src must be finite and outside r_+ + capture_buffer");
        im.src_on = 1;
        im.r_src = source->r_src;
        im.src_tol = 1e-12 * source->r_src;
        // the source sits at (theta, phi) = (pi - incl, pi)
        const double ts = M_PI - camera->incl;
        im.src_n[0] = std::sin(ts) * std::cos(M_PI);
        im.src_n[1] = std::sin(ts) * std::sin(M_PI);
        im.src_n[2] = std::cos(ts);
    }
    if (want_ring && !src_on) return fail(KT_EINVAL, "ring needs an enabled source and a deflection output");
    if (source && source->sky) {
        if (!finite_all({source->grid_deg, source->line_deg}) || !(source->grid_deg >= 0.0) ||
            !(source->line_deg >= 0.0))
            return fail(KT_EINVAL, "sky needs finite grid_deg >= 0 and line_deg >= 0");
        im.sky_on = 1;
        im.esc_tol = 1e-12 * r_esc;
        im.grid_deg = source->grid_deg;
        im.line_deg = source->line_deg;
    }
    return KT_OK;
}

bool is_mixed(const kt_integrator* integ) { return integ->precision == KT_MIXED; }

// The launch sequence shared by single and batch renders.  `table` holds the
// validated images with their `first` offsets; for one image it travels in
// Params and the device table is the workspace copy of img0.
int render_images(const kt::Image* table, int32_t n_images, int64_t n_rays, const kt_integrator* integ,
                  const kt_outputs* out, void* workspace, size_t workspace_bytes, void* hip_stream,
                  const kt_launch* launch) {
    kt_launch ln{1, 256, 0, DEFAULT_BATCH, KT_ORDER_RING};
    if (launch) ln = *launch;
    if (ln.block != 64 && ln.block != 128 && ln.block != 256)
        return fail(KT_EINVAL, "launch block must be 64, 128 or 256");
    if (ln.batch < 1 || ln.batch > 4096) return fail(KT_EINVAL, "launch batch must lie in [1, 4096]");
    if (ln.blocks_per_cu < 0 || ln.blocks_per_cu > 64)
        return fail(KT_EINVAL, "launch blocks_per_cu must lie in [0, 64]");
    if (ln.order != KT_ORDER_RING && ln.order != KT_ORDER_ROWS)
        return fail(KT_EINVAL, "launch order must be KT_ORDER_RING or KT_ORDER_ROWS");

    const bool batch = n_images > 1;
    const kt::WsLayout w =
        kt::ws_layout(static_cast<size_t>(n_rays), static_cast<size_t>(n_images), batch, is_mixed(integ));
    if (!workspace) return fail(KT_EINVAL, "workspace must not be NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(KT_EINVAL, "workspace must be 256-byte aligned");
    if (workspace_bytes < w.total)
        return fail(KT_ENOMEM, "workspace too small: %zu < %zu bytes", workspace_bytes, w.total);

    kt::Params p;
    std::memset(&p, 0, sizeof p);
    p.method = integ->method;
    p.precision = integ->precision;
    p.h_fixed = integ->h_fixed;
    p.rtol = integ->rtol;
    p.atol = integ->atol;
    p.h_init = integ->h_init;
    p.max_steps = integ->max_steps;
    p.max_evals = 16 * integ->max_steps;
    p.h_budget = integ->h_budget;
    p.r_switch = integ->r_switch;
    p.n_rays = n_rays;
    p.n_images = n_images;
    p.img0 = table[0];
    p.out.fate = out->fate;
    p.out.r_hit = out->r_hit;
    p.out.g = out->g;
    p.out.intensity = out->intensity;
    p.out.max_abs_h = out->max_abs_h;
    p.out.max_rel_h = out->max_rel_h;
    p.out.psi = out->psi;
    p.out.deflection = out->deflection;
    p.out.theta_f = out->theta_f;
    p.out.phi_f = out->phi_f;
    p.out.n_cross = out->n_cross;
    p.out.used_fp64 = out->used_fp64;
    p.out.ring = out->ring;
    p.out.n_steps = out->n_steps;
    p.out.n_evals = out->n_evals;
    p.out.sky = out->sky;
    p.out.stats = out->stats;
    char* ws = static_cast<char*>(workspace);
    p.ticket = reinterpret_cast<uint32_t*>(ws + kt::WS_TICKET);
    p.acc = reinterpret_cast<unsigned long long*>(ws + kt::WS_ACC);
    p.fb_count = reinterpret_cast<uint32_t*>(ws + kt::WS_FB_COUNT);
    p.ws_params = reinterpret_cast<kt::Params*>(ws + kt::WS_PARAMS);
    p.images = batch ? reinterpret_cast<const kt::Image*>(ws + w.images) : &p.ws_params->img0;
    p.rc_buf = reinterpret_cast<double*>(ws + w.rc);
    p.fb_list = reinterpret_cast<uint32_t*>(ws + w.fb_list);
    p.need_fb = reinterpret_cast<uint8_t*>(ws + w.need);
    // With a ray for every lane of a one-wave grid or fewer all rays start
    // together: an order by length has nothing to give, and its sort takes longer
    // than it saves (72x72 disk 1.60/1.56 ms with and without, 250x250 disk
    // 2.23/2.17, 200x200 shadow 2.83/2.79; 300x300, 1.4 rays per lane, on the
    // q-metric 5.44/6.38).
    const bool all_at_once = ln.persistent && n_rays <= static_cast<int64_t>(device_cus()) * 4 * 64;
    if (ln.order == KT_ORDER_RING && !(all_at_once && ln.blocks_per_cu == 0)) {
        p.perm = reinterpret_cast<uint32_t*>(ws + w.perm);
        p.order_hist = reinterpret_cast<uint32_t*>(ws + w.hist);
        p.order_bins = reinterpret_cast<uint16_t*>(ws + w.bins);
    }
    p.persistent = ln.persistent ? 1 : 0;
    p.from_list = 0;
    p.wall_khz = out->stats ? device_wall_khz() : 0.0;
    p.batch = ln.batch;
    const Shape shape = launch_shape(p, ln, n_rays);
    p.min_idle = shape.min_idle;

    if (batch && kt::launch_upload_images(table, n_images, reinterpret_cast<kt::Image*>(ws + w.images),
                                          hip_stream))
        return fail(KT_EDEVICE, "image table upload failed: %s", hipGetErrorString(hipGetLastError()));
    if (kt::launch_ws_init(p, hip_stream))
        return fail(KT_EDEVICE, "workspace init launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (p.perm && kt::launch_order(p, hip_stream))
        return fail(KT_EDEVICE, "dispatch order launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (out->stats && kt::launch_stamp(p, kt::ACC_T0, hip_stream))
        return fail(KT_EDEVICE, "clock stamp launch failed: %s", hipGetErrorString(hipGetLastError()));
    if ((shape.w3 ? kt_w3::launch_trace : kt::launch_trace)(p, shape.grid, ln.block, hip_stream))
        return fail(KT_EDEVICE, "trace kernel launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (p.precision == KT_MIXED) {
        // re-run every ray over the |H|_rel budget in FP64, from a compacted
        // list whose length stays on the device
        if (kt::launch_fallback_list(p, hip_stream))
            return fail(KT_EDEVICE, "fallback list launch failed: %s", hipGetErrorString(hipGetLastError()));
        const Shape again = launch_shape(p, ln, n_rays, MIXED_RERUN_SHARE);
        p.min_idle = again.min_idle;
        if ((again.w3 ? kt_w3::launch_trace_fallback : kt::launch_trace_fallback)(p, again.grid, ln.block, hip_stream))
            return fail(KT_EDEVICE, "fallback trace launch failed: %s", hipGetErrorString(hipGetLastError()));
    }
    if (out->stats && kt::launch_stamp(p, kt::ACC_T1, hip_stream))
        return fail(KT_EDEVICE, "clock stamp launch failed: %s", hipGetErrorString(hipGetLastError()));
    if ((out->r_hit || out->g || out->intensity) && kt::launch_disk_obs(p, hip_stream))
        return fail(KT_EDEVICE, "disk observables launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (out->ring && kt::launch_ring(p, hip_stream))
        return fail(KT_EDEVICE, "ring kernel launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (out->sky && kt::launch_sky(p, hip_stream))
        return fail(KT_EDEVICE, "sky kernel launch failed: %s", hipGetErrorString(hipGetLastError()));
    if (out->stats && kt::launch_stats(p, hip_stream))
        return fail(KT_EDEVICE, "stats kernel launch failed: %s", hipGetErrorString(hipGetLastError()));
    return KT_OK;
}

int validate_outputs(const kt_outputs* out) {
    if (!out->fate) return fail(KT_EINVAL, "out->fate must not be NULL");
    if (out->ring && !out->deflection)
        return fail(KT_EINVAL, "ring needs an enabled source and a deflection output");
    if (out->sky && !(out->theta_f && out->phi_f))
        return fail(KT_EINVAL, "sky needs the theta_f and phi_f outputs");
    return KT_OK;
}

// Table of a batch with `first` offsets; on error returns the code with the
// image named in the message.
int make_table(int32_t n_images, const kt_image* images, const kt_integrator* integ, bool want_ring,
               std::vector<kt::Image>& table, int64_t* n_rays) {
    if (n_images < 1 || n_images > KT_MAX_IMAGES)
        return fail(KT_EINVAL, "n_images must lie in [1, %d] (got %d)", KT_MAX_IMAGES, n_images);
    if (!images) return fail(KT_EINVAL, "images must not be NULL");
    table.resize(static_cast<size_t>(n_images));
    int64_t first = 0;
    for (int32_t k = 0; k < n_images; ++k) {
        const kt_image& in = images[k];
        if (in.spacetime.metric != KT_METRIC_KERR)
            return fail(KT_EINVAL, "image %d: batches run the Kerr metric", k);
        int rc = make_image(&in.camera, &in.spacetime, &in.disk, &in.source, integ, want_ring, table[k]);
        if (rc) {
            char msg[512];
            std::snprintf(msg, sizeof msg, "image %d: %s", k, g_err);
            std::snprintf(g_err, sizeof g_err, "%s", msg);
            return rc;
        }
        table[k].first = first;
        first += static_cast<int64_t>(in.camera.nx) * in.camera.ny;
        if (first >= (int64_t{1} << 31)) return fail(KT_EINVAL, "total rays of the batch must be < 2^31");
    }
    *n_rays = first;
    return KT_OK;
}

}  // namespace

namespace kt {
int validate_single(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
                    const kt_source* source, const kt_integrator* integ, const kt_outputs* out, Image* im) {
    g_err[0] = 0;
    int rc = validate_common(camera, spacetime);
    if (rc) return rc;
    if (!integ || !out) return fail(KT_EINVAL, "integ and out must not be NULL");
    if ((rc = validate_integ(integ)) || (rc = validate_outputs(out))) return rc;
    if ((rc = make_image(camera, spacetime, disk, source, integ, out->ring != nullptr, *im))) return rc;
    im->first = 0;
    return KT_OK;
}
}  // namespace kt

extern "C" {

const char* kt_last_error(void) { return g_err; }

int kt_version(void) { return KT_VERSION_NUMBER; }

size_t kt_workspace_bytes(const kt_camera* camera, const kt_integrator* integ) {
    if (!camera || !integ || camera->nx < 1 || camera->ny < 1) return 0;
    const size_t n = static_cast<size_t>(camera->nx) * static_cast<size_t>(camera->ny);
    if (n >= (size_t{1} << 31)) return 0;  // ray ids are int32
    return kt::ws_layout(n, 1, false, is_mixed(integ)).total;
}

size_t kt_workspace_bytes_batch(int32_t n_images, const kt_image* images, const kt_integrator* integ) {
    if (!images || !integ || n_images < 1 || n_images > KT_MAX_IMAGES) return 0;
    size_t n = 0;
    for (int32_t k = 0; k < n_images; ++k) {
        if (images[k].camera.nx < 1 || images[k].camera.ny < 1) return 0;
        n += static_cast<size_t>(images[k].camera.nx) * static_cast<size_t>(images[k].camera.ny);
    }
    if (n >= (size_t{1} << 31)) return 0;  // ray ids are int32
    return kt::ws_layout(n, static_cast<size_t>(n_images), n_images > 1, is_mixed(integ)).total;
}

int kt_init_rays(const kt_camera* camera, const kt_spacetime* spacetime, double* state,
                 uint8_t* invalid, void* hip_stream) {
    g_err[0] = 0;
    int rc = validate_common(camera, spacetime);
    if (rc) return rc;
    if (!state || !invalid) return fail(KT_EINVAL, "state and invalid must not be NULL");
    if (!(camera->r_obs > horizon(spacetime)))
        return fail(KT_EINVAL, "r_obs must lie outside the horizon");
    kt::Params p;
    std::memset(&p, 0, sizeof p);
    camera_constants(camera, spacetime, p.img0);
    p.n_rays = static_cast<int64_t>(camera->nx) * camera->ny;
    if (kt::launch_init_rays(p, state, invalid, hip_stream))
        return fail(KT_EDEVICE, "init kernel launch failed: %s", hipGetErrorString(hipGetLastError()));
    return KT_OK;
}

int kt_render_ex(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
                 const kt_source* source, const kt_integrator* integ, const kt_outputs* out,
                 void* workspace, size_t workspace_bytes, void* hip_stream, const kt_launch* launch) {
    g_err[0] = 0;
    kt::Image im;  // one image: no host allocation on this path
    int rc = kt::validate_single(camera, spacetime, disk, source, integ, out, &im);
    if (rc) return rc;
    const int64_t n = static_cast<int64_t>(camera->nx) * camera->ny;
    return render_images(&im, 1, n, integ, out, workspace, workspace_bytes, hip_stream, launch);
}

int kt_render(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
              const kt_source* source, const kt_integrator* integ, const kt_outputs* out,
              void* workspace, size_t workspace_bytes, void* hip_stream) {
    return kt_render_ex(camera, spacetime, disk, source, integ, out, workspace, workspace_bytes,
                        hip_stream, nullptr);
}

int kt_render_batch(int32_t n_images, const kt_image* images, const kt_integrator* integ,
                    const kt_outputs* out, void* workspace, size_t workspace_bytes, void* hip_stream,
                    const kt_launch* launch) {
    g_err[0] = 0;
    if (!integ || !out) return fail(KT_EINVAL, "integ and out must not be NULL");
    int rc;
    if ((rc = validate_integ(integ)) || (rc = validate_outputs(out))) return rc;
    std::vector<kt::Image> table;
    int64_t n = 0;
    if ((rc = make_table(n_images, images, integ, out->ring != nullptr, table, &n))) return rc;
    return render_images(table.data(), n_images, n, integ, out, workspace, workspace_bytes, hip_stream, launch);
}

size_t kt_adjoint_workspace_bytes(const kt_camera* camera, const kt_integrator* integ) {
    if (!camera || !integ || camera->nx < 1 || camera->ny < 1) return 0;
    const size_t n = static_cast<size_t>(camera->nx) * static_cast<size_t>(camera->ny);
    if (n >= (size_t{1} << 31)) return 0;  // ray ids are int32
    const int ck_shift = kt::adj_ck_shift(integ->checkpoint_every);
    if (ck_shift < 0) return 0;
    if (integ->split_above < -1) return 0;
    return kt::adj_layout(n, integ->max_steps, ck_shift, integ->split_above >= 0).total;
}

int kt_adjoint(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
               const kt_integrator* integ, const uint8_t* fate, const double* r_hit, const int32_t* n_steps,
               const double* cot_intensity,
               double* grad_a, double* grad_incl, double* grad_r_in, double* grad_sum, uint64_t* stats,
               void* workspace, size_t workspace_bytes, void* hip_stream) {
    g_err[0] = 0;
    int rc = validate_common(camera, spacetime);
    if (rc) return rc;
    if (!integ || !disk) return fail(KT_EINVAL, "integ and disk must not be NULL");
    if ((rc = validate_integ(integ))) return rc;
    if (integ->method != KT_DP45 || integ->precision != KT_FP64)
        return fail(KT_EINVAL, "the adjoint follows the KT_DP45 / KT_FP64 integration");
    if (!disk->enabled) return fail(KT_EINVAL, "the adjoint differentiates a disk image: enable the disk");
    if (!(spacetime->M > 0.0)) return fail(KT_EINVAL, "the adjoint needs M > 0");
    if (spacetime->metric != KT_METRIC_KERR) return fail(KT_EINVAL, "the adjoint differentiates Kerr images");
    if (!fate || !cot_intensity) return fail(KT_EINVAL, "fate and cot_intensity must not be NULL");
    const int ck_shift = kt::adj_ck_shift(integ->checkpoint_every);
    if (ck_shift < 0)
        return fail(KT_EINVAL, "checkpoint_every must be 0 or a power of two in [1, 1024] (got %d)",
                    integ->checkpoint_every);
    kt::Image im;
    if ((rc = make_image(camera, spacetime, disk, nullptr, integ, false, im))) return rc;
    im.first = 0;
    const size_t n = static_cast<size_t>(camera->nx) * static_cast<size_t>(camera->ny);
    const kt::AdjLayout w = kt::adj_layout(n, integ->max_steps, ck_shift, integ->split_above >= 0);
    if (!workspace) return fail(KT_EINVAL, "workspace must not be NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return fail(KT_EINVAL, "workspace must be 256-byte aligned");
    if (workspace_bytes < w.total)
        return fail(KT_ENOMEM, "workspace too small: %zu < %zu bytes", workspace_bytes, w.total);

    kt::AdjParams p;
    std::memset(&p, 0, sizeof p);
    p.im = im;
    camera_constant_derivs(camera, spacetime, p.dcam);
    p.dm = kt::adj::DiskModel{spacetime->M, disk->r_out, disk->emis_index, disk->l0, disk->rotation,
                              disk->emissivity};
    p.rtol = integ->rtol;
    p.atol = integ->atol;
    p.h_init = integ->h_init;
    p.max_attempts = 16 * integ->max_steps;
    p.n_rays = static_cast<int64_t>(n);
    p.fate = fate;
    p.r_hit = r_hit;
    p.cot = cot_intensity;
    char* ws = static_cast<char*>(workspace);
    // per-pixel gradients go to the caller's arrays, else to the workspace
    // (the image sums read them)
    double* wg = reinterpret_cast<double*>(ws + w.grad);
    p.grad_a = grad_a ? grad_a : wg;
    p.grad_incl = grad_incl ? grad_incl : wg + n;
    p.grad_rin = grad_r_in ? grad_r_in : wg + 2 * n;
    p.grad_sum = grad_sum;
    p.partials = reinterpret_cast<double*>(ws + w.partials);
    p.ck_shift = ck_shift;
    p.ticket = reinterpret_cast<uint32_t*>(ws + kt::ADJ_WS_TICKET);
    p.stats = stats ? reinterpret_cast<unsigned long long*>(stats)
                    : reinterpret_cast<unsigned long long*>(ws + w.stats);
    p.ckpt = reinterpret_cast<double*>(ws + w.ckpt);
    p.seg = reinterpret_cast<double*>(ws + w.seg);
    p.n_steps = n_steps;
    p.hist = reinterpret_cast<uint32_t*>(ws + w.hist);
    p.keys = reinterpret_cast<uint16_t*>(ws + w.keys);
    p.list = reinterpret_cast<uint32_t*>(ws + w.list);
    p.n_lanes = w.n_lanes;
    p.max_ckpt = w.max_ckpt;
    // stored forward passes need the forward step counts
    p.split_above = integ->split_above;
    p.max_long = n_steps && integ->split_above >= 0 ? w.max_long : 0;
    p.long_cap = integ->split_above >= 0 ? kt::adj_store_cap(w, workspace_bytes) : 0u;
    p.item_cap = w.item_cap;
    p.counters = reinterpret_cast<uint32_t*>(ws + kt::ADJ_WS_COUNTERS);
    p.long_store = reinterpret_cast<double*>(ws + w.ckpt);
    p.longs = reinterpret_cast<kt::AdjLong*>(ws + w.longs);
    p.owner = reinterpret_cast<uint32_t*>(ws + w.owner);
    p.items = reinterpret_cast<double*>(ws + w.items);
    p.params = reinterpret_cast<kt::Params*>(ws + w.params);
    // One wave per SIMD for the stored passes: their end is a chain of steps of the
    // longest rays, which a second wave slows, and a lane that has twice the rays
    // leaves fewer sweeps to split (four step VJPs for one).  ms of the adjoint at 1
    // and 2 waves, disks at 20, 45 and 70 degrees:
    //   512x512    3.84/5.05  3.03/4.35  2.99/4.01    700x700    7.04/7.40  6.63/6.15  3.19/4.58
    //   850x850    10.6/10.8  7.97/8.70  4.60/5.73    1024x1024  16.8/16.9  11.0/11.7  6.63/7.27
    //   1400x1400  32.5/33.4  23.2/25.7  11.3/11.8    2048x2048  76.8/76.7  52.9/54.8  28.2/32.7
    p.trace_blocks = device_cus();
    p.grid_lanes = device_cus() * 256;
    if (kt::launch_adjoint(p, hip_stream))
        return fail(KT_EDEVICE, "adjoint launch failed: %s", hipGetErrorString(hipGetLastError()));
    return KT_OK;
}

int kt_autotune_batch(int32_t n_images, const kt_image* images, const kt_integrator* integ,
                      const kt_outputs* out, void* workspace, size_t workspace_bytes, void* hip_stream,
                      const kt_launch* candidates, int32_t n_candidates, int32_t repeats, kt_launch* best,
                      float* times_ms) {
    g_err[0] = 0;
    if (!integ || !out || !best) return fail(KT_EINVAL, "integ, out and best must not be NULL");
    if (repeats < 1 || repeats > 100) return fail(KT_EINVAL, "repeats must lie in [1, 100]");
    if ((candidates == nullptr) != (n_candidates == 0) || n_candidates < 0 || n_candidates > 4096)
        return fail(KT_EINVAL, "give candidates with 1..4096 entries, or NULL with n_candidates = 0");
    int rc;
    if ((rc = validate_integ(integ)) || (rc = validate_outputs(out))) return rc;
    std::vector<kt::Image> table;
    int64_t n = 0;
    if ((rc = make_table(n_images, images, integ, out->ring != nullptr, table, &n))) return rc;

    std::vector<kt_launch> cand;
    if (candidates) {
        cand.assign(candidates, candidates + n_candidates);
    } else {
        for (int block : {128, 256})
            for (int waves : {1, 2, 3})
                for (int batch : {4, 8, 16, 32, 64})
                    cand.push_back(kt_launch{1, block, waves * 256 / block, batch, KT_ORDER_RING});
    }
    // the untimed first render also validates every shape before any timing
    for (const kt_launch& ln : cand)
        if ((ln.block != 64 && ln.block != 128 && ln.block != 256) || ln.batch < 1 || ln.batch > 4096 ||
            ln.blocks_per_cu < 0 || ln.blocks_per_cu > 64 ||
            (ln.order != KT_ORDER_RING && ln.order != KT_ORDER_ROWS))
            return fail(KT_EINVAL, "candidate launch shape out of range (block %d, blocks_per_cu %d, batch %d, order %d)",
                        ln.block, ln.blocks_per_cu, ln.batch, ln.order);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(KT_EDEVICE, "hipEventCreate failed");
    }
    int best_i = -1;
    float best_ms = 0.0f;
    rc = render_images(table.data(), n_images, n, integ, out, workspace, workspace_bytes, hip_stream, &cand[0]);
    for (size_t i = 0; rc == KT_OK && i < cand.size(); ++i) {
        if (hipEventRecord(e0, s) != hipSuccess) { rc = fail(KT_EDEVICE, "hipEventRecord failed"); break; }
        for (int r = 0; r < repeats && rc == KT_OK; ++r)
            rc = render_images(table.data(), n_images, n, integ, out, workspace, workspace_bytes, hip_stream,
                               &cand[i]);
        if (rc) break;
        float ms = 0.0f;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            rc = fail(KT_EDEVICE, "event timing failed: %s", hipGetErrorString(hipGetLastError()));
            break;
        }
        ms /= static_cast<float>(repeats);
        if (times_ms) times_ms[i] = ms;
        if (best_i < 0 || ms < best_ms) {
            best_i = static_cast<int>(i);
            best_ms = ms;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    *best = cand[static_cast<size_t>(best_i)];
    return KT_OK;
}

}  // extern "C"
