// kt_adjoint.hip -- discrete adjoint of the disk image (observed intensity
// per pixel) with respect to the spin a, the inclination and the disk's
// inner radius.
//
// Per ray:
//   1. re-integrate from the camera with the trace kernel's own stepper and
//      controller (bit-identical steps) up to the located disk crossing;
//   2. seed the cotangent of the crossing state from the intensity's
//      derivatives, with the crossing-time correction that keeps theta on
//      the equatorial plane;
//   3. run the vector-Jacobian products of the Dormand-Prince steps backward
//      with the accepted step sizes frozen, the located partial step first;
//   4. chain the cotangents of the initial state and of (E, L) through the
//      camera's dependence on (a, inclination).
// With the forward step counts step 1 is the trace kernel itself (its STORE
// form) with every accepted step written to a store, and step 3 reads the steps
// back, one item per lane, partly by waves of the forward pass that have no ray
// left (see sweep in kt_trace.hip).  A long ray's sweep is split: each 64-step
// segment is swept backward from four basis cotangents (its transposed Jacobian,
// a linear map since the steps are frozen), one lane each, and the last kernel
// applies the segments' maps to the ray's seeded cotangent in order.  A sweep is
// otherwise one lane's sequential work, and the longest would set the run time.
// Rays beyond the store, those that end there without a crossing, and all of them
// without step counts or with split sweeps off, take the one-lane path (adjoint_kernel): checkpoints every
// 2^ck_shift accepted steps and each segment between them recomputed.
// The results are the per-pixel products cot_I * dI/d(a, incl, r_in) and,
// on request, their three sums over the image (a fixed-order block-then-grid
// reduction, so the sums do not depend on which lane ran which ray).
#include <hip/hip_runtime.h>

#include <cstring>

#include "kt_adjoint_math.h"
#include "kt_device.h"
#include "kt_internal.h"
#include "kt_ray.h"
#include "kt_sort.h"

namespace kt {

// Where the forward pass keeps states: entry idx at p + idx * istride, its
// field f (0..4 the state, 5 a step size) at + f * fstride, at most cap
// entries.  With shift > 0 entry c is the state after c * 2^shift accepted
// steps and the trial size of the next step (entry 0 the start); with shift
// 0 entry j is the start state of accepted step j and its accepted size.
// A lane's checkpoints and segment slots sit in [index][field][lane] arrays.
struct StepStore {
    double* p;
    size_t istride, fstride;
    int32_t cap, shift;
    __device__ double* at(int idx) const { return p + static_cast<size_t>(idx) * istride; }
};
__device__ __forceinline__ void put6(double* p, size_t fstride, const double y[5], double h) {
#pragma unroll
    for (int f = 0; f < 5; ++f) p[f * fstride] = y[f];
    p[5 * fstride] = h;
}
__device__ __forceinline__ void get6(const double* p, size_t fstride, double y[5], double* h) {
#pragma unroll
    for (int f = 0; f < 5; ++f) y[f] = p[f * fstride];
    *h = p[5 * fstride];
}

// One attempt of the adaptive step as the trace kernel takes it.  Returns 1
// for an accepted step (yn, kn, dg, h_next set), 0 for a rejection (h
// shrunk), -1 for a failure.
__device__ __forceinline__ int try_step(const Spacetime& st, const RayConst& rc, const AdjParams& P,
                                        const double y[5], const double k1[5], double s0, double c0, double* h,
                                        bool* rejected, double yn[5], double kn[5], Diag* dg, double* h_next) {
    double er[5];
    dp45_step(st, rc, y, k1, s0, c0, *h, yn, kn, er, dg);
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 5; ++i) finite = finite && isfinite(yn[i]);
    if (!finite) return -1;
    double sc[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) sc[i] = fma(P.rtol, fmax(fabs(y[i]), fabs(yn[i])), P.atol);
    const double msq = error_msq(er, sc);
    if (isnan(msq)) return -1;
    if (msq > 1.0) {
        *h *= reject_factor<KT_DP45>(msq);
        *rejected = true;
        return 0;
    }
    double fac = accept_factor<KT_DP45>(msq);
    if (*rejected) fac = fmin(fac, 1.0);
    *h_next = *h * fac;
    return 1;
}

constexpr int ADJ_BLOCK = 256;

// What the forward pass leaves for the backward one.
struct Fwd {
    double y[5];  // start of the located partial step
    double E, L;
    double zs[5], ks[5], hstar;  // crossing state, the field there, the partial step's size
    int n;                       // accepted steps before the crossing
};

// 1. Forward from the camera to the disk crossing, storing states in `sto`.
__device__ __forceinline__ int forward_to_hit(const AdjParams& P, const Spacetime& st, int32_t ray,
                                              const StepStore& sto, Fwd* f) {
    const Image& im = P.im;
    double* y = f->y;
    camera_state(im, ray, y, &f->E, &f->L);
    const RayConst rc = make_ray_const(st, f->E, f->L);
    const int ck_mask = (1 << sto.shift) - 1;
    double k1[5];
    Diag dg;
    rhs<true, false>(st, rc, y, k1, &dg);
    double s0 = dg.s, c0 = dg.c, h = P.h_init;
    bool rej = false;
    int n = 0;  // accepted steps
    if (sto.shift > 0) put6(sto.at(0), sto.fstride, y, h);
    bool hit = false;
    for (int64_t guard = 0; guard < P.max_attempts && !hit; ++guard) {
        double yn[5], kn[5], hn = 0.0;
        Diag dn;
        const int ok = try_step(st, rc, P, y, k1, s0, c0, &h, &rej, yn, kn, &dn, &hn);
        if (ok < 0) return ADJ_FAIL;
        if (ok == 0) continue;
        const double fa0 = y[1] - HALF_PI, fb0 = yn[1] - HALF_PI;
        if (fa0 * fb0 < 0.0) {
            // Illinois regula falsi on theta - pi/2, trial steps from y
            double A = 0.0, FA = fa0, B = h, FB = fb0, C = h - fb0 * h / (fb0 - fa0);
            double zc[5], kc[5];
            for (int it = 1;; ++it) {
                double ec[5];
                Diag dc;
                dp45_step(st, rc, y, k1, s0, c0, C, zc, kc, ec, &dc);
                const double fc = zc[1] - HALF_PI;
                if (fabs(fc) <= 1e-14 || it >= 64) break;
                if (fc * FB < 0.0) {
                    A = B;
                    FA = FB;
                } else {
                    FA *= 0.5;
                }
                B = C;
                FB = fc;
                C = B - FB * (B - A) / (FB - FA);
            }
            if (zc[0] >= im.r_in && zc[0] <= im.r_out) {
                hit = true;
                f->hstar = C;
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    f->zs[i] = zc[i];
                    f->ks[i] = kc[i];
                }
                break;
            }
        } else if (fb0 == 0.0 && yn[0] >= im.r_in && yn[0] <= im.r_out) {
            hit = true;
            f->hstar = h;
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                f->zs[i] = yn[i];
                f->ks[i] = kn[i];
            }
            break;
        }
        if (yn[0] < im.r_cap || yn[0] > im.r_esc) return ADJ_MISMATCH;
        if (sto.shift == 0) {
            // every accepted step: its start state and its accepted size
            if (n >= sto.cap) return ADJ_OVERFLOW;
            put6(sto.at(n), sto.fstride, y, h);
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            y[i] = yn[i];
            k1[i] = kn[i];
        }
        s0 = dn.s;
        c0 = dn.c;
        h = hn;
        rej = false;
        ++n;
        if (sto.shift > 0 && (n & ck_mask) == 0) {
            if ((n >> sto.shift) >= sto.cap) return ADJ_OVERFLOW;
            put6(sto.at(n >> sto.shift), sto.fstride, y, h);
        }
    }
    if (!hit) return ADJ_FAIL;
    if (P.r_hit && !(f->zs[0] == P.r_hit[ray])) return ADJ_MISMATCH;
    f->n = n;
    return ADJ_OK;
}

// 3. The rest of the reverse sweep with frozen steps, from the lane's own
// checkpoints: stored steps are read back; otherwise each segment between
// checkpoints is recomputed forward from its checkpoint into the lane's
// segment slots first.
__device__ __forceinline__ int sweep_lane(const AdjParams& P, const Spacetime& st, int lane, const Fwd& f,
                                          double zb[5], adj::ParBar* pb) {
    const Image& im = P.im;
    const size_t fs = static_cast<size_t>(P.n_lanes), is = 6u * fs;
    int n = f.n;
    if (P.ck_shift == 0) {
        // every step was stored: no recomputation
        for (int j = n - 1; j >= 0; --j) {
            double yj[5], hj;
            get6(P.ckpt + j * is + lane, fs, yj, &hj);
            adj::dp_step_vjp<false>(im.M, im.a, f.E, f.L, yj, hj, zb, pb);
        }
        return ADJ_OK;
    }
    const RayConst rc = make_ray_const(st, f.E, f.L);
    const int ck_mask = (1 << P.ck_shift) - 1;
    for (int s = (n - 1) >> P.ck_shift; n > 0 && s >= 0; --s) {
        const int first = s << P.ck_shift, last = min(n, first + ck_mask + 1);
        double ys[5], hs;
        get6(P.ckpt + s * is + lane, fs, ys, &hs);
        double kk[5];
        Diag dr;
        rhs<true, false>(st, rc, ys, kk, &dr);
        double ss = dr.s, cc = dr.c;
        bool rj = false;
        int attempts = 0;
        for (int j = first; j < last;) {
            // the recomputation repeats the forward's attempts exactly; the
            // bound only guarantees that the loop ends
            if (++attempts > 64 * (ck_mask + 1)) return ADJ_FAIL;
            double yn[5], kn[5], hn = 0.0;
            Diag dn;
            const int ok = try_step(st, rc, P, ys, kk, ss, cc, &hs, &rj, yn, kn, &dn, &hn);
            if (ok < 0) return ADJ_FAIL;
            if (ok == 0) continue;
            put6(P.seg + (j - first) * is + lane, fs, ys, hs);
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                ys[i] = yn[i];
                kk[i] = kn[i];
            }
            ss = dn.s;
            cc = dn.c;
            hs = hn;
            rj = false;
            ++j;
        }
        for (int j = last - 1; j >= first; --j) {
            double yj[5], hj;
            get6(P.seg + (j - first) * is + lane, fs, yj, &hj);
            adj::dp_step_vjp<false>(im.M, im.a, f.E, f.L, yj, hj, zb, pb);
        }
    }
    return ADJ_OK;
}

// 4. The camera: z0 = (r0, incl, 0, p_r, p_th), E, L of (a, incl).
__device__ __forceinline__ void camera_chain(const AdjParams& P, int32_t ray, const double zb[5],
                                             const adj::ParBar& pb, double* ga, double* gi) {
    const Image& im = P.im;
    const int32_t jj = ray / im.nx, ii = ray - jj * im.nx;
    const double x = -im.fov_x + (static_cast<double>(ii) + 0.5) * im.dx;
    const double yy = -im.fov_y + (static_cast<double>(jj) + 0.5) * im.dy;
    const double rad = 1.0 - (yy / im.r0) * (yy / im.r0) - (x / im.r0) * (x / im.r0);
    const double pr0 = -sqrt(im.g_rr * rad);
    double g2[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double dE = P.dcam[0][k] + x * P.dcam[1][k];
        const double dL = x * P.dcam[2][k];
        const double dpth = yy * P.dcam[3][k];
        const double dpr = 0.5 * pr0 * P.dcam[4][k] / im.g_rr;
        g2[k] = pb.E * dE + pb.L * dL + zb[3] * dpr + zb[4] * dpth;
    }
    *ga = pb.a + g2[0];
    *gi = zb[1] + g2[1];
}

__device__ __forceinline__ void put_grads(const AdjParams& P, int32_t ray, int status, double ga, double gi,
                                          double gr) {
    if (status != ADJ_OK) ga = gi = gr = 0.0;
    atomicAdd(P.stats + status, 1ull);
    if (P.grad_a) P.grad_a[ray] = ga;
    if (P.grad_incl) P.grad_incl[ray] = gi;
    if (P.grad_rin) P.grad_rin[ray] = gr;
}

// One entry t of the work list, the whole adjoint of its ray on this lane.
__device__ __forceinline__ void adjoint_entry(const AdjParams& P, const Spacetime& st, int lane, uint32_t t) {
    const Image& im = P.im;
    const int32_t ray = static_cast<int32_t>(P.list[t]);
    const size_t fs = static_cast<size_t>(P.n_lanes);
    const StepStore sto{P.ckpt + lane, 6u * fs, fs, P.max_ckpt, P.ck_shift};
    Fwd f;
    double zb[5], ga = 0.0, gi = 0.0, gr = 0.0;
    adj::ParBar pb;
    int status = forward_to_hit(P, st, ray, sto, &f);
    if (status == ADJ_OK) {
        adj::seed(P.dm, im.a, im.r_in, f.zs[0], f.ks[0], f.ks[1], f.E, f.L, P.cot[ray], zb, &pb, &gr);
        adj::dp_step_vjp<false>(im.M, im.a, f.E, f.L, f.y, f.hstar, zb, &pb);
        status = sweep_lane(P, st, lane, f, zb, &pb);
    }
    if (status == ADJ_OK) camera_chain(P, ray, zb, pb, &ga, &gi);
    put_grads(P, ray, status, ga, gi, gr);
}

// Lanes take the entries of the work list that are not stored from an atomic
// ticket.  One wave per SIMD: the forward pass, its recomputation and the
// step VJP in one kernel want more than a two-wave budget.
__global__ void __launch_bounds__(ADJ_BLOCK) __attribute__((amdgpu_waves_per_eu(1)))
adjoint_kernel(const AdjParams P) {
    const int lane = blockIdx.x * blockDim.x + threadIdx.x;
    if (lane >= P.n_lanes) return;
    const Spacetime st{P.im.M, P.im.a, P.im.a2, P.im.two_a2};
    const bool stored = P.max_long > 0;
    const uint32_t first = stored ? P.counters[ADJ_C_FIRST] : 0u, end = stored ? P.counters[ADJ_C_END] : 0u;
    const uint32_t n = P.hist[SORT_BINS] - (end - first);
    // then the stored rays that took more steps than the caller's count said
    const uint32_t total = n + (stored && P.counters[ADJ_C_REDO] != 0u ? end - first : 0u);
    for (;;) {
        uint32_t t = atomicAdd(P.ticket, 1u);
        if (t >= total) break;
        if (t >= n) {
            t = t - n + first;
            if (P.longs[t - first].status != ADJ_OVERFLOW) continue;
        } else if (t >= first) {
            t += end - first;
        }
        adjoint_entry(P, st, lane, t);
    }
}

// Inclusive sums over the block's threads (Hillis-Steele).
__device__ __forceinline__ unsigned long long block_scan(unsigned long long v, unsigned long long* part) {
    const int t = threadIdx.x;
    __syncthreads();
    part[t] = v;
    __syncthreads();
    for (int off = 1; off < SORT_BLOCK; off <<= 1) {
        const unsigned long long add = t >= off ? part[t - off] : 0ull;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    return part[t];
}

// Which rays are stored and which of them split, from the sorted work list's
// bins (one block, after the sort: hist[k] is then the end of bin k, and bin
// k holds the rays of 4 v to 4 v + 3 forward steps, v = SORT_BINS - 1 - k, bin
// 0 also every longer ray).  Both are whole bins, longest first, so that the
// sets, and with them the gradients, do not depend on which lanes take the
// rays: stored are the bins from `skip` + 1 on as long as the store and the
// records hold them for certain (a ray of bin v takes at most 4 v + 5
// entries).  Bin 0, which has no such bound, and bins of more steps than the
// one-lane path's checkpoints cover are left to that path, which counts such
// rays as it does without step counts.  A store that holds less than one in
// ADJ_STORE_SHARE of those bins' steps is left empty: the one-lane path then has most
// of the work to do after it, and with so many lanes' work gains nothing from having
// the longest rays done.  ms of the adjoint with and without stored passes, by the
// share that the store held: 1400x1400 at 45 degrees (0.70) 23.9 and 28.0, 600x600
// (0.51) 6.4 and 10.9, 700x700 (0.37) 9.0 and 13.0, 2048x2048 (0.36) 53.5 and 57.9,
// 850x850 (0.25) 12.0 and 11.5, 1400x1400 (0.09) 29.9 and 28.1, 2048x2048 (0.04) 60.8
// and 58.0; at 20 degrees 600x600 (0.37) 8.3 and 8.1, 850x850 (0.19) 14.9 and 14.8.
// A split sweep takes four step VJPs per step instead of one, in pieces of
// ADJ_SEG steps instead of the ray's length.  The longest bins are split until
// the longest sweep left is no longer than the sweep kernel's work per lane,
// (all steps + 3 times the split ones) / lanes: splitting fewer would leave
// that sweep running alone at the end, splitting more only adds work.  With a
// threshold of the caller's, the rays above it are split.
// The forward pass's waves sweep their own rays where that pass is bound by its
// longest ray, that is where a lane's share of all steps is at most half of that
// ray's: ms of a fit's step without and with it, by that share, 512x512 at 45
// degrees (0.32) 8.4 and 7.0, 560x560 at 60 degrees 9.3 and 8.2; where lanes
// have more to do the sweeps are better dealt out once, in order of length:
// 480x480 at 30 degrees 6.3 and 7.6, 640x640 at 30 degrees 11.7 and 12.9.
constexpr unsigned long long ADJ_STORE_SHARE = 3;
__global__ void __launch_bounds__(SORT_BLOCK) adjoint_split_kernel(const AdjParams P) {
    constexpr int PER = SORT_BINS / SORT_BLOCK;  // consecutive bins per thread
    static_assert(SORT_BINS % SORT_BLOCK == 0, "bins must split evenly over the block");
    __shared__ unsigned long long part[SORT_BLOCK];
    __shared__ unsigned long long all_steps;
    __shared__ int stop_store, stop_split, longest_bin;
    const int t = threadIdx.x;
    const int covered = (P.max_ckpt << P.ck_shift) / 4 - 2;  // v of the longest bin within the checkpoints
    const int skip = SORT_BINS - 2 < covered ? 0 : SORT_BINS - 2 - covered;
    const uint32_t first = P.hist[skip];
    if (t == 0) stop_store = stop_split = longest_bin = SORT_BINS;
    uint32_t cnt[PER];
    unsigned long long need = 0;
    for (int i = 0; i < PER; ++i) {
        const int k = t * PER + i;
        cnt[i] = k > skip ? P.hist[k] - P.hist[k - 1] : 0u;
        need += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * (SORT_BINS - 1 - k) + 5);
    }
    unsigned long long run = block_scan(need, part) - need;
    const unsigned long long entries = static_cast<unsigned long long>(P.long_cap) * 6ull / ADJ_ENTRY;
    for (int i = 0; i < PER; ++i) {
        const int k = t * PER + i;
        run += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * (SORT_BINS - 1 - k) + 5);
        if (cnt[i] != 0u && (run > entries || P.hist[k] - first > static_cast<uint32_t>(P.max_long))) {
            atomicMin(&stop_store, k);
            break;
        }
    }
    __syncthreads();
    unsigned long long listed = 0;  // steps of the bins that could be stored, where not all are
    if (stop_store < SORT_BINS) {
        for (int i = 0; i < PER; ++i)
            listed += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * (SORT_BINS - 1 - (t * PER + i)) + 2);
        listed = block_scan(listed, part);
    }
    // steps and segment items of the stored bins, and the bins to split
    unsigned long long steps = 0, items = 0;
    for (int i = 0; i < PER; ++i) {
        const int k = t * PER + i, v = SORT_BINS - 1 - k;
        if (k >= stop_store) cnt[i] = 0u;
        steps += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * v + 2);
        items += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * ((4 * v + 4) / ADJ_SEG + 1));
        if (cnt[i] != 0u) atomicMin(&longest_bin, k);
    }
    unsigned long long run_steps = block_scan(steps, part);
    if (t == SORT_BLOCK - 1) {
        all_steps = run_steps;
        if (ADJ_STORE_SHARE * run_steps < listed) stop_store = skip + 1;
    }
    run_steps -= steps;
    unsigned long long run_items = block_scan(items, part) - items;
    for (int i = 0; i < PER; ++i) {
        const int k = t * PER + i, v = SORT_BINS - 1 - k;
        // run_steps: the steps of the bins before this one
        const unsigned long long load = (all_steps + 3ull * run_steps) / static_cast<unsigned long long>(P.grid_lanes);
        const unsigned long long longest = static_cast<unsigned long long>(4 * v + 3);
        const bool enough = P.split_above > 0 ? 4 * v <= P.split_above
                                              : longest <= (load > ADJ_SEG ? load : ADJ_SEG);
        run_steps += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * v + 2);
        run_items += static_cast<unsigned long long>(cnt[i]) * static_cast<unsigned long long>(4 * ((4 * v + 4) / ADJ_SEG + 1));
        if (k > skip && (enough || k >= stop_store || run_items > P.item_cap)) {
            atomicMin(&stop_split, k);
            break;
        }
    }
    __syncthreads();
    if (t == 0) {
        P.counters[ADJ_C_FIRST] = first;
        P.counters[ADJ_C_END] = P.hist[stop_store - 1];
        P.counters[ADJ_C_SPLIT] = P.hist[stop_split - 1] - first;
        P.counters[ADJ_C_OVERLAP] = 2ull * all_steps <= static_cast<unsigned long long>(4 * (SORT_BINS - longest_bin)) * P.grid_lanes ? 1u : 0u;
    }
}

// The seeds of the rays that no wave of the forward pass has swept, from the
// crossing left in each record, and the items of the split ones.
__global__ void __launch_bounds__(ADJ_BLOCK) adjoint_seed_kernel(const AdjParams P) {
    const uint32_t n_split = P.counters[ADJ_C_SPLIT];
    const uint32_t n = P.counters[ADJ_C_OVERLAP] != 0u ? n_split : P.counters[ADJ_C_END] - P.counters[ADJ_C_FIRST];
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        AdjLong& rec = P.longs[k];
        if (rec.status != ADJ_OK) continue;
        double zb[5], gr;
        adj::ParBar pb;
        adj::seed(P.dm, P.im.a, P.im.r_in, rec.zb[0], rec.zb[1], rec.zb[2], rec.E, rec.L, P.cot[rec.ray], zb, &pb, &gr);
        rec.zb[0] = zb[0];
        rec.zb[1] = zb[1];
        rec.zb[2] = rec.zb[3] = 0.0;
        rec.pb[0] = pb.E;
        rec.pb[1] = pb.L;
        rec.pb[2] = pb.a;
        rec.gr = gr;
        if (k >= n_split) continue;
        const uint32_t n_seg = static_cast<uint32_t>(rec.n) / ADJ_SEG + 1u;  // of n + 1 entries
        const uint32_t ib = atomicAdd(P.counters + ADJ_C_ITEMS, 4u * n_seg);
        rec.n_seg = static_cast<int32_t>(n_seg);
        rec.item_base = ib;
        // the split kernel left room for every split ray's items
        if (ib + 4u * n_seg > P.item_cap) rec.status = ADJ_OVERFLOW;
        for (uint32_t i = 0; i < 4u * n_seg && ib + i < P.item_cap; ++i) P.owner[ib + i] = k;
    }
}

// The stored rays' ends: a split ray's seeded cotangent through the segments'
// maps, last segment first (cotangent' = sum_b cotangent_b * column_b,
// parameter cotangents += sum_b cotangent_b * their column_b), then the camera.
__global__ void __launch_bounds__(ADJ_BLOCK) adjoint_combine_kernel(const AdjParams P) {
    const uint32_t n = P.counters[ADJ_C_END] - P.counters[ADJ_C_FIRST], n_split = P.counters[ADJ_C_SPLIT];
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const AdjLong& rec = P.longs[k];
        if (rec.status == ADJ_OVERFLOW) {
            atomicAdd(P.counters + ADJ_C_REDO, 1u);  // left to the one-lane path
            continue;
        }
        if (rec.status != ADJ_OK) {
            put_grads(P, rec.ray, rec.status, 0.0, 0.0, 0.0);
            continue;
        }
        double v[4] = {rec.zb[0], rec.zb[1], rec.zb[2], rec.zb[3]};
        adj::ParBar pb{rec.pb[0], rec.pb[1], rec.pb[2]};
        for (int s = k < n_split ? rec.n_seg - 1 : -1; s >= 0; --s) {
            const double* o = P.items + (static_cast<size_t>(rec.item_base) + 4u * static_cast<size_t>(s)) * 8u;
            double nv[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const double* c = o + 8 * b;
#pragma unroll
                for (int i = 0; i < 4; ++i) nv[i] = fma(v[b], c[i], nv[i]);
                pb.E = fma(v[b], c[4], pb.E);
                pb.L = fma(v[b], c[5], pb.L);
                pb.a = fma(v[b], c[6], pb.a);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = nv[i];
        }
        const double zb[5] = {v[0], v[1], 0.0, v[2], v[3]};
        double ga, gi;
        camera_chain(P, rec.ray, zb, pb, &ga, &gi);
        put_grads(P, rec.ray, ADJ_OK, ga, gi, rec.gr);
    }
}

// Clears the ticket, the statistics, the counters and the sort's histogram,
// and leaves the forward pass its parameters.
__global__ void adjoint_init_kernel(const AdjParams P, const Params fwd) {
    const int t = threadIdx.x;
    if (t == 0) *P.ticket = 0u;
    if (t < 4) P.stats[t] = 0ull;
    if (P.max_long > 0) {
        if (t < ADJ_C_COUNT) P.counters[t] = 0u;
        if (t == 0) *P.params = fwd;
    }
    for (int b = t; b <= SORT_BINS; b += blockDim.x) P.hist[b] = 0u;
}

// ---- work list ------------------------------------------------------------
// The lanes of a wave run their rays' loops in step, so a wave costs as much
// as its longest ray.  The differentiated rays (disk hits with a nonzero
// cotangent) are compacted into a list sorted by the forward render's step
// count, longest first (a counting sort over SORT_BINS bins of 4 steps):
// neighbouring lanes then take rays of nearly equal length.  Pixels outside
// the list get zero gradients from the key function.
struct StepKey {
    const uint8_t* fate;
    const double* cot;
    const int32_t* n_steps;  // may be NULL: every listed ray gets the same key
    double *ga, *gi, *gr;
    __device__ int operator()(int64_t ray) const {
        if (fate[ray] == KT_FATE_DISK && cot[ray] != 0.0) {
            int steps = n_steps ? n_steps[ray] >> 2 : 0;
            steps = steps < 0 ? 0 : steps > SORT_BINS - 1 ? SORT_BINS - 1 : steps;
            return SORT_BINS - 1 - steps;
        }
        if (ga) ga[ray] = 0.0;
        if (gi) gi[ray] = 0.0;
        if (gr) gr[ray] = 0.0;
        return SORT_SKIP;
    }
};

// ---- the image sums of the three gradient maps ---------------------------
// A fixed grid of ADJ_RED_BLOCKS blocks: thread t of block b adds pixels
// t + 256 b, t + 256 (b + ADJ_RED_BLOCKS), ... in that order, the block adds
// its 256 partial sums by a fixed tree in LDS, and one block then adds the
// ADJ_RED_BLOCKS block sums by the same tree.  Every sum is taken in one
// order whatever the device or the lanes that ran the rays.
constexpr int RED_THREADS = 256;

__device__ __forceinline__ void tree_sum3(double (*v)[RED_THREADS], int t) {
#pragma unroll
    for (int w = RED_THREADS / 2; w > 0; w >>= 1) {
        __syncthreads();
        if (t < w) {
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c][t] += v[c][t + w];
        }
    }
    __syncthreads();
}

__global__ void __launch_bounds__(RED_THREADS) grad_block_sum_kernel(const double* __restrict__ ga,
                                                                     const double* __restrict__ gi,
                                                                     const double* __restrict__ gr, int64_t n,
                                                                     double* __restrict__ partials) {
    __shared__ double v[3][RED_THREADS];
    const int t = threadIdx.x;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * RED_THREADS + t; k < n;
         k += static_cast<int64_t>(ADJ_RED_BLOCKS) * RED_THREADS) {
        s0 += ga[k];
        s1 += gi[k];
        s2 += gr[k];
    }
    v[0][t] = s0;
    v[1][t] = s1;
    v[2][t] = s2;
    tree_sum3(v, t);
    if (t < 3) partials[t * ADJ_RED_BLOCKS + blockIdx.x] = v[t][0];
}

__global__ void __launch_bounds__(RED_THREADS) grad_final_sum_kernel(const double* __restrict__ partials,
                                                                     double* __restrict__ out) {
    static_assert(ADJ_RED_BLOCKS == RED_THREADS, "one partial per thread");
    __shared__ double v[3][RED_THREADS];
    const int t = threadIdx.x;
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c][t] = partials[c * ADJ_RED_BLOCKS + t];
    tree_sum3(v, t);
    if (t < 3) out[t] = v[t][0];
}

// The parameters of the stored forward pass.
static Params forward_params(const AdjParams& p) {
    Params f;
    std::memset(&f, 0, sizeof f);
    f.method = KT_DP45;
    f.precision = KT_FP64;
    f.rtol = p.rtol;
    f.atol = p.atol;
    f.h_init = p.h_init;
    f.max_steps = p.max_attempts / 16;
    f.max_evals = p.max_attempts;
    f.n_rays = p.n_rays;
    f.n_images = 1;
    f.img0 = p.im;
    f.ticket = p.counters + ADJ_C_TRACE;
    f.ws_params = p.params;
    f.persistent = 1;
    f.batch = 4;
    f.min_idle = 8;
    f.adj.list = p.list;
    f.adj.n_steps = p.n_steps;
    f.adj.r_hit = p.r_hit;
    f.adj.cot = p.cot;
    f.adj.counters = p.counters;
    f.adj.recs = p.longs;
    f.adj.store = p.long_store;
    f.adj.owner = p.owner;
    f.adj.items = p.items;
    f.adj.entries = static_cast<uint32_t>(static_cast<uint64_t>(p.long_cap) * 6u / ADJ_ENTRY);
    f.adj.item_cap = p.item_cap;
    f.adj.dm = p.dm;
    return f;
}

int launch_adjoint(const AdjParams& p, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool stored = p.max_long > 0;
    const Params fwd = forward_params(p);
    hipLaunchKernelGGL(adjoint_init_kernel, dim3(1), dim3(256), 0, s, p, fwd);
    if (hipGetLastError() != hipSuccess) return -1;
    const SortBufs b{p.n_rays, p.hist, p.keys, p.list};
    if (launch_sort(b, StepKey{p.fate, p.cot, p.n_steps, p.grad_a, p.grad_incl, p.grad_rin}, s)) return -1;
    if (stored) {
        hipLaunchKernelGGL(adjoint_split_kernel, dim3(1), dim3(SORT_BLOCK), 0, s, p);
        if (hipGetLastError() != hipSuccess) return -1;
        const int64_t need = (p.n_rays + ADJ_BLOCK - 1) / ADJ_BLOCK;
        if (launch_trace_store(fwd, static_cast<int>(need < p.trace_blocks ? need : p.trace_blocks), 0, s)) return -1;
        hipLaunchKernelGGL(adjoint_seed_kernel, dim3(static_cast<int>(need < 1024 ? need : 1024)), dim3(ADJ_BLOCK), 0, s, p);
        if (hipGetLastError() != hipSuccess) return -1;
        if (launch_trace_store(fwd, p.trace_blocks, 1, s)) return -1;
        hipLaunchKernelGGL(adjoint_combine_kernel, dim3(static_cast<int>(need < 1024 ? need : 1024)), dim3(ADJ_BLOCK), 0, s, p);
        if (hipGetLastError() != hipSuccess) return -1;
    }
    const int grid = (p.n_lanes + ADJ_BLOCK - 1) / ADJ_BLOCK;
    hipLaunchKernelGGL(adjoint_kernel, dim3(grid), dim3(ADJ_BLOCK), 0, s, p);
    if (hipGetLastError() != hipSuccess) return -1;
    if (p.grad_sum) {
        hipLaunchKernelGGL(grad_block_sum_kernel, dim3(ADJ_RED_BLOCKS), dim3(RED_THREADS), 0, s, p.grad_a,
                           p.grad_incl, p.grad_rin, static_cast<int64_t>(p.n_rays), p.partials);
        if (hipGetLastError() != hipSuccess) return -1;
        hipLaunchKernelGGL(grad_final_sum_kernel, dim3(1), dim3(RED_THREADS), 0, s, p.partials, p.grad_sum);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace kt
