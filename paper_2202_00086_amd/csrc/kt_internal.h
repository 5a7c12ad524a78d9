// kt_internal.h -- parameter blocks shared by the host runtime and the kernels.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "kerrtrace.h"
#include "kt_adjoint_math.h"

namespace kt {

constexpr int ACC_EVALS = 0, ACC_EVALS_FP32 = 1;  // acc[8..15]: fate histogram
constexpr int ACC_T0 = 2, ACC_T1 = 3;  // wall clock ticks just before and just after the trace launches

struct Outputs {
    uint8_t* fate;
    double *r_hit, *g, *intensity, *max_abs_h, *max_rel_h, *psi, *deflection, *theta_f, *phi_f;
    uint8_t *n_cross, *used_fp64, *ring;
    int32_t *n_steps, *n_evals;
    uint8_t* sky;
    kt_stats* stats;
};

// Everything that belongs to one image: spacetime, camera constants, disk,
// source, and where its rays sit in the batch.
struct Image {
    // spacetime (eq:Kerr; or the q-metric, metric = KT_METRIC_Q) and the end radii
    double M, a, a2, two_a2;
    int32_t metric;
    double q;
    double r_cap, r_esc;
    // camera and per-image camera constants (Sect. 2.3)
    double r0, incl, fov_x, fov_y, dx, dy;
    double E0;      // 1 / A_t
    double cE;      // g_tphi / (r0 sqrt(g_phph)):  E = E0 + x cE
    double cL;      // -sqrt(g_phph) / r0:          L = x cL
    double cth;     // sqrt(g_thth) / r0:           p_theta = y cth
    double g_rr;    // g_rr at the camera:          p_r = -sqrt(g_rr (1 - (y/r0)^2 - (x/r0)^2))
    int32_t nx, ny;
    int64_t first;  // ray id of pixel 0 (outputs of this image start here)
    // disk (Sect. 5)
    int32_t disk_on, rotation, emis_model;
    double r_in, r_out, emis_q, l0;
    // source for the deflection diagnostics
    int32_t src_on;
    double r_src, src_tol;
    double src_n[3];  // unit vector towards the source
    // celestial sphere at r_esc (Sect. 4.1)
    int32_t sky_on;
    double esc_tol, grid_deg, line_deg;
    // dispatch order: pixels go out by the bin of |rho - rho_ring|, rho the
    // image-plane radius, bin = that distance times order_scale
    double rho_ring, order_scale;
};

// Where the adjoint's forward pass leaves the accepted steps of the rays it
// stores: entries of ADJ_ENTRY doubles (r, theta, p_r, p_theta at a step's
// start and its size), a ray's in order from its record's base.
struct AdjLong;
struct AdjStore {
    const uint32_t* list;     // the work list; the stored rays are [FIRST, END) of it
    const int32_t* n_steps;   // the forward render's step counts
    const double* r_hit;      // its hit radii, or NULL
    const double* cot;        // cotangents of the intensity
    uint32_t* counters;       // ADJ_C_*
    AdjLong* recs;            // record of list entry t at t - FIRST
    double* store;
    const uint32_t* owner;    // record of each segment item
    double* items;            // [item_cap][8]
    uint32_t entries, item_cap;
    adj::DiskModel dm;
};

// Everything a render needs, copied into the workspace by ws_init.
struct Params {
    // integrator (shared by all images)
    int32_t method, precision;
    double h_fixed, rtol, atol, h_init;
    int64_t max_steps, max_evals;
    double h_budget, r_switch;
    // images: a single render uses a one-entry table (img0)
    int64_t n_rays;
    int32_t n_images;
    const Image* images;  // device table
    Image img0;
    // outputs and workspace
    Outputs out;
    uint32_t* ticket;
    unsigned long long* acc;
    uint32_t* fb_list;
    uint32_t* fb_count;
    double* rc_buf;
    uint8_t* need_fb;   // KT_MIXED: 1 where the ray must be re-run in FP64
    Params* ws_params;  // where ws_init leaves the device copy of this struct
    uint32_t* perm;     // dispatch order: ray id of each slot, or NULL for slot = ray id
    uint32_t* order_hist;  // uint32[SORT_BINS + 1] counts, then offsets and the total
    uint16_t* order_bins;  // uint16[n_rays] bin of each ray
    // launch
    int32_t persistent, batch, min_idle;
    int32_t from_list;  // take ray ids from fb_list[0 .. *fb_count)
    double wall_khz;    // the device's wall clock rate, kHz (0: unknown)
    AdjStore adj;       // the adjoint's forward pass only
};

// Bins of the device counting sorts (dispatch order, adjoint work list), and
// the key of an id the sort leaves out.
constexpr int SORT_BINS = 1024;
constexpr uint16_t SORT_SKIP = 0xffff;

// Workspace layout (byte offsets from the start of the caller's buffer).
constexpr size_t WS_TICKET = 0;       // uint32 ray ticket
constexpr size_t WS_ACC = 64;         // uint64[16]
constexpr size_t WS_FB_COUNT = 192;   // uint32 fallback list length
constexpr size_t WS_PARAMS = 256;     // device copy of Params
constexpr size_t WS_PARAMS_MAX = 1792;
static_assert(sizeof(Params) <= WS_PARAMS_MAX, "Params must fit its workspace slot");

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct WsLayout {
    size_t images;   // Image[n_images] (batch renders)
    size_t rc;       // double[n_rays] disk crossing radius per ray
    size_t fb_list;  // uint32[n_rays] (KT_MIXED)
    size_t need;     // uint8[n_rays] (KT_MIXED)
    size_t perm;     // uint32[n_rays] dispatch order
    size_t hist;     // uint32[SORT_BINS + 1]
    size_t bins;     // uint16[n_rays]
    size_t total;
};

inline WsLayout ws_layout(size_t n_rays, size_t n_images, bool batch, bool mixed) {
    WsLayout w;
    w.images = WS_PARAMS + WS_PARAMS_MAX;
    w.rc = align256(w.images + (batch ? n_images * sizeof(Image) : 0));
    w.fb_list = align256(w.rc + 8 * n_rays);
    w.need = align256(w.fb_list + (mixed ? 4 * n_rays : 0));
    w.perm = align256(w.need + (mixed ? n_rays : 0));
    w.hist = align256(w.perm + 4 * n_rays);
    w.bins = align256(w.hist + 4 * (SORT_BINS + 1));
    w.total = align256(w.bins + 2 * n_rays);
    return w;
}

enum : int32_t { FEAT_DISK = 1, FEAT_SRC = 2, FEAT_SKY = 4 };

constexpr int32_t image_features(const Image& im) {
    return (im.disk_on ? FEAT_DISK : 0) | (im.src_on ? FEAT_SRC : 0) | (im.sky_on ? FEAT_SKY : 0);
}

// The values the trace kernel's inner loop reads every step, passed by value
// so they sit in scalar registers; everything else is read through `cold`.
// For batch renders the per-image ones become per-lane values.
struct Hot {
    double M, a, a2, two_a2;
    double rtol, atol, r_cap, r_esc;
    double h_budget, r_switch;  // KT_MIXED
    int32_t feat;               // FEAT_* bits of the image's disk, source and sky
    int32_t max_steps, max_evals;
    uint32_t first;             // ray ids of a persistent wave's first fetch: 64 (see make_hot)
    int32_t min_idle;           // idle lanes a refill waits for
    unsigned long long* acc;    // the evaluation counters
    double* store;              // the adjoint's step store
    int32_t sweep_only;         // STORE: the second launch, which has only sweeps to do
    const Params* cold;         // the workspace copy of Params
};

// A ray whose forward pass is stored (kt_adjoint with step counts).  Its
// entries start at `base`: entry j < n the j-th accepted step before the
// crossing, entry n the located partial step.  The seed kernel turns the
// crossing into the cotangents at it; the sweep leaves those at the camera
// (status ADJ_OK), or for a split ray, the first n_split of the stored ones,
// the maps of its segments as items item_base + 4 s + b (segment s covers the
// entries [ADJ_SEG s, ADJ_SEG (s + 1)), b runs over the basis cotangents).
enum : int { ADJ_OK = 0, ADJ_FAIL = 1, ADJ_OVERFLOW = 2, ADJ_MISMATCH = 3 };
struct AdjLong {
    int32_t ray, status, n, n_seg;
    uint32_t base, item_base;
    uint32_t next;  // the record that the same lane finished after this one
    uint32_t left;  // slot of the list of the records whose sweep is left to the second launch
    double zb[4];     // cotangents of (r, theta, p_r, p_theta); first (r, r', theta') at the crossing
    double pb[3];     // of (E, L, a)
    double gr, E, L;  // the r_in gradient (from the seed alone) and the ray constants
};

// Everything the adjoint kernel needs (passed by value).
struct AdjParams {
    Image im;
    double dcam[5][2];  // d(E0, cE, cL, cth, g_rr) / d(a, incl)
    adj::DiskModel dm;
    double rtol, atol, h_init;
    int64_t max_attempts;
    int64_t n_rays;
    const uint8_t* fate;
    const double* r_hit;
    const double* cot;
    double *grad_a, *grad_incl, *grad_rin;  // per pixel: the caller's arrays or the workspace's
    double* grad_sum;           // the three sums (caller's device memory), or NULL
    double* partials;           // [3][ADJ_RED_BLOCKS] block sums of the reduction
    uint32_t* ticket;
    unsigned long long* stats;  // [ok, failed, overflow, mismatch]
    double* ckpt;               // [max_ckpt][6][n_lanes]
    double* seg;                // [1 << ck_shift][6][n_lanes]
    int32_t n_lanes, max_ckpt;
    int32_t ck_shift;           // checkpoints every 1 << ck_shift accepted steps
    // work list: the differentiated rays, longest forward integration first
    const int32_t* n_steps;     // the forward render's step counts (may be NULL)
    uint32_t* hist;             // [SORT_BINS + 1] bin counts, then offsets; [SORT_BINS] = list length
    uint16_t* keys;             // [n_rays] bin of each ray, SORT_SKIP if not differentiated
    uint32_t* list;             // [n_rays] ray ids
    // stored forward passes (only with n_steps; max_long 0 switches them off)
    int32_t split_above;        // 0: threshold from the work list; > 0: this many steps
    int32_t max_long;           // records in `longs`
    uint32_t long_cap, item_cap;  // long_cap: the store's size in 6 doubles
    uint32_t* counters;         // ADJ_C_*
    double* long_store;         // the stored entries (shares the checkpoints' memory)
    AdjLong* longs;             // [max_long]
    uint32_t* owner;            // [item_cap] record of each segment item
    double* items;              // [item_cap][8] one segment's sweep of one basis cotangent
    Params* params;             // the forward pass's parameters (device copy)
    int32_t trace_blocks, grid_lanes;  // grid of the forward pass, lanes of the sweep's
};

// AdjParams.counters
enum : int {
    ADJ_C_SPLIT = 0,     // split rays
    ADJ_C_STORE = 1,     // entries taken
    ADJ_C_ITEMS = 2,     // segment items taken
    ADJ_C_FIRST = 3,     // the stored rays' range of the work list
    ADJ_C_END = 4,
    ADJ_C_TRACE = 5,     // ticket of the forward pass
    ADJ_C_SWEEP = 6,     // ticket of the sweep
    ADJ_C_REDO = 7,      // stored rays left to the one-lane path
    ADJ_C_DONE = 8,      // waves of the forward pass that have no forward ray left
    ADJ_C_LEFT = 9,      // sweeps left to the second launch
    ADJ_C_OVERLAP = 10,  // 1: the forward pass's waves sweep their own rays
    ADJ_C_COUNT = 11
};

#ifndef KT_ADJ_MAX_LANES
#define KT_ADJ_MAX_LANES 65536
#endif
constexpr int ADJ_MAX_LANES = KT_ADJ_MAX_LANES;
constexpr int ADJ_MAX_CKPT = 256;            // checkpoint slots per lane, at least
constexpr int ADJ_MIN_STEPS_COVERED = 2048;  // and at least this many accepted steps covered
constexpr int ADJ_CK_SHIFT_DEFAULT = 6;      // checkpoints every 64 accepted steps
// 0 stores every accepted step (start state and accepted size): the reverse
// sweep then reads each step instead of recomputing it
constexpr int ADJ_CK_SHIFT_MIN = 0, ADJ_CK_SHIFT_MAX = 10;
constexpr int ADJ_RED_BLOCKS = 256;      // fixed grid of the gradient reduction (deterministic)
// Stored forward passes: ADJ_ENTRY doubles per accepted step (a 512x512 disk image
// of 117k hits takes 136 steps per pixel, 1.4 GB), at most ADJ_STORE_MAX_BYTES
// unless the one-lane path's part of the workspace is larger and ADJ_MAX_RECORDS
// rays, sweeps split into segments of ADJ_SEG entries.
constexpr int ADJ_SEG = 64, ADJ_ENTRY = 5;
constexpr size_t ADJ_STORE_MAX_BYTES = KT_ADJOINT_ROOM_MAX;
constexpr size_t ADJ_MAX_RECORDS = 524288;
// Room for the records and the segment items, part of the size that callers'
// buffers have: ADJ_SPLIT_LANE_BYTES per lane and ADJ_SPLIT_RAY_BYTES per ray, of
// ADJ_SPLIT_RAYS at most.  The records come first, 112 bytes per ray; what they
// leave holds items of ADJ_ITEM_BYTES, four per segment: 1.2M at 512x512, where the
// automatic threshold uses 85 thousand.  A caller's threshold that asks for more
// than there are splits the longest rays only (adjoint_split_kernel).
constexpr size_t ADJ_SPLIT_LANE_BYTES = 1672, ADJ_SPLIT_RAY_BYTES = 384, ADJ_SPLIT_RAYS = 8192;
constexpr size_t ADJ_ITEM_BYTES = 8 * sizeof(double) + sizeof(uint32_t);
static_assert(ADJ_MAX_RECORDS * sizeof(AdjLong) <= ADJ_SPLIT_LANE_BYTES * static_cast<size_t>(ADJ_MAX_LANES) &&
                  sizeof(AdjLong) <= ADJ_SPLIT_LANE_BYTES,
              "the records must leave room for items");

// log2 of kt_integrator.checkpoint_every (0 selects 64); -1 unless a power
// of two in [1, 1024].
inline int adj_ck_shift(int32_t every) {
    if (every == 0) return ADJ_CK_SHIFT_DEFAULT;
    for (int s = ADJ_CK_SHIFT_MIN; s <= ADJ_CK_SHIFT_MAX; ++s)
        if (every == (1 << s)) return s;
    return -1;
}

struct AdjLayout {
    size_t stats, hist, partials, params, keys, list, grad, longs, owner, items, ckpt, seg, total;
    int32_t n_lanes, max_ckpt, max_long;
    uint32_t item_cap;
};

// Byte offsets in the first 256 bytes of the adjoint's workspace.
constexpr size_t ADJ_WS_TICKET = 0, ADJ_WS_COUNTERS = 16;

// split: room for split backward sweeps (kt_integrator.split_above >= 0).  `total`
// is the least workspace.  The checkpoints and segment slots of the one-lane path
// come last; the stored forward passes, done with before that path starts, share
// their memory and take what a larger workspace has behind it (adj_store_cap).
inline AdjLayout adj_layout(size_t n_rays, int64_t max_steps, int ck_shift, bool split) {
    AdjLayout w;
    size_t lanes = (n_rays + 255) / 256 * 256;
    if (lanes > static_cast<size_t>(ADJ_MAX_LANES)) lanes = ADJ_MAX_LANES;
    if (lanes < 256) lanes = 256;
    int64_t ck = (max_steps >> ck_shift) + 2;
    const int64_t cap = ADJ_MAX_CKPT > (ADJ_MIN_STEPS_COVERED >> ck_shift) ? ADJ_MAX_CKPT
                                                                         : (ADJ_MIN_STEPS_COVERED >> ck_shift);
    if (ck > cap) ck = cap;
    w.n_lanes = static_cast<int32_t>(lanes);
    w.max_ckpt = static_cast<int32_t>(ck);
    w.stats = 64;
    w.hist = 256;
    w.partials = align256(w.hist + 4u * (SORT_BINS + 1));
    w.params = align256(w.partials + 3u * ADJ_RED_BLOCKS * sizeof(double));
    w.keys = align256(w.params + WS_PARAMS_MAX);
    w.list = align256(w.keys + 2u * n_rays);
    w.grad = align256(w.list + 4u * n_rays);
    w.longs = align256(w.grad + 3u * sizeof(double) * n_rays);
    w.max_long = split ? static_cast<int32_t>(n_rays < ADJ_MAX_RECORDS ? n_rays : ADJ_MAX_RECORDS) : 0;
    const size_t recs = static_cast<size_t>(w.max_long) * sizeof(AdjLong);
    const size_t few = n_rays < ADJ_SPLIT_RAYS ? n_rays : ADJ_SPLIT_RAYS;
    const size_t room = lanes * ADJ_SPLIT_LANE_BYTES + few * ADJ_SPLIT_RAY_BYTES;
    const size_t seg_items = 4u * ADJ_ITEM_BYTES;  // those of one segment, rounded up
    w.item_cap = split ? static_cast<uint32_t>((room - recs + seg_items - 1u) / seg_items * 4u) : 0u;
    w.owner = align256(w.longs + recs);
    w.items = align256(w.owner + sizeof(uint32_t) * w.item_cap);
    w.ckpt = align256(w.items + 8u * sizeof(double) * w.item_cap);
    w.seg = align256(w.ckpt + static_cast<size_t>(ck) * 6u * lanes * sizeof(double));
    w.total = align256(w.seg + (size_t{1} << ck_shift) * 6u * lanes * sizeof(double));
    return w;
}

// The store's size in a workspace of so many bytes, in 6 doubles.
inline uint32_t adj_store_cap(const AdjLayout& w, size_t workspace_bytes) {
    const size_t least = w.total - w.ckpt, most = least > ADJ_STORE_MAX_BYTES ? least : ADJ_STORE_MAX_BYTES;
    const size_t room = workspace_bytes - w.ckpt;
    return static_cast<uint32_t>((room < most ? room : most) / (6u * sizeof(double)));
}

// Leave msg for kt_last_error() on this host thread and return code (kt_api.cpp).
int set_error(int code, const char* msg);

// The argument checks of a single-image render; fills the image's table
// entry.  Returns KT_OK or the error code (message left as for a render).
int validate_single(const kt_camera* camera, const kt_spacetime* spacetime, const kt_disk* disk,
                    const kt_source* source, const kt_integrator* integ, const kt_outputs* out, Image* im);

// Host-side launchers (kt_trace.hip, kt_adjoint.hip).
int launch_adjoint(const AdjParams& p, void* stream);
// The adjoint's forward pass and sweeps, then (sweep_only) what is left of the sweeps.
int launch_trace_store(const Params& p, int grid, int sweep_only, void* stream);
int launch_ws_init(const Params& p, void* stream);  // also copies p into the workspace
int launch_upload_images(const Image* host, int32_t n, Image* dev, void* stream);
int launch_order(const Params& p, void* stream);  // fills p.perm (ring-first dispatch)
int launch_trace(const Params& p, int grid, int block, void* stream);  // pass of p.precision
int launch_fallback_list(const Params& p, void* stream);  // compact need_fb, switch the copy to from_list
int launch_trace_fallback(const Params& p, int grid, int block, void* stream);  // FP64 re-run from the list
int launch_reset_ticket(const Params& p, void* stream);
int launch_ring(const Params& p, void* stream);
int launch_sky(const Params& p, void* stream);  // needs theta_f and phi_f outputs
int launch_disk_obs(const Params& p, void* stream);
int launch_stats(const Params& p, void* stream);
int launch_stamp(const Params& p, int slot, void* stream);  // acc[slot] = the wall clock now
int launch_init_rays(const Params& p, double* state, uint8_t* invalid, void* stream);
int trace_max_blocks_per_cu(const Params& p, int block);

}  // namespace kt

// The same trace kernels built for 3 waves per SIMD (kt_trace_w3.hip): the
// default for renders of many rays per lane, and for launch shapes of 3 or
// more waves per SIMD.  Their outputs equal the 2-wave kernels' bit for bit.
namespace kt_w3 {
int launch_trace(const kt::Params& p, int grid, int block, void* stream);
int launch_trace_fallback(const kt::Params& p, int grid, int block, void* stream);
int trace_max_blocks_per_cu(const kt::Params& p, int block);
}  // namespace kt_w3
