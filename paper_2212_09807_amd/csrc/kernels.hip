// kernels.hip -- gfx950 kernels of the pixelated-LArTPC charge path (arXiv 2212.09807, Sec. 3).
//
// Stage map (one event, or a batch of events whose pixel spaces are concatenated):
//   k_quench_drift   Sec. 3.1-3.2: recombination, lifetime, diffusion widths per segment; charge box in
//                    (tick, sub-pixel bin) space; pixel rectangle the box reaches; per-pixel pair counts (a
//                    difference array over the pixel grid, k_prefix_rows / k_prefix_cols).
//   scans            pair / cell offsets (exclusive scans), active-pixel compaction (slots).
//   k_fill_pairs     pixel-major (pixel, segment) pair lists; k_sort_pairs orders each list by segment id.
//   k_cells          Sec. 3.3.2 eq. (rho), expectation over the Gaussian perturbations: charge per
//                    (tick, x-bin, y-bin) cell of each segment, as a sum over sample points of separable
//                    truncated-Gaussian bin masses.
//   k_induce_*       Sec. 3.3.2 eq. (current): per (segment, pixel) pair and tick, the cells in the pixel's table
//                    reach convolved in time with the field-response column of their mirror-folded bin; summed
//                    over the pixel's segments (Sec. 3.4) either in a fixed order with Kahan compensation
//                    (sorted variant) or with FP32 atomics (atomic variant).  k_induce_z*: as matrix products over
//                    groups of a pixel's segments (default); k_induce_sorted / k_induce_atomic: on the vector units.
//   k_sum_*          the same sum by linearity as sum-then-convolve: segments' charges summed per sub-pixel
//                    column (column lists, sort, intervals, summed charges), per-pixel records by folded table
//                    column, the mirror merge, then k_induce_summed_mma (default) / k_induce_summed over the records.
//   k_electronics    Sec. 3.4: integrate, threshold (with discriminator noise), hold, digitise, reset, with
//                    Philox4x32-10 noise; also the FP64 per-event sum of the currents.
//   k_settle         the currents of pixels with a decision on the edge once more, in the vector kernels' order, and
//                    k_electronics over them (after matrix-core sums only).
//   k_compact        packets of all pixels into the caller's arrays.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.hpp"
#include "launch.hpp"

namespace ltsim {

constexpr uint64_t kMask40 = (1ull << 40) - 1;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ float lane_value(float v, int32_t l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, v), l));
}

// FP64 per-event report accumulation, aggregated over the wavefront when all valid lanes share the event.
// Must be reached by all 64 lanes of the wavefront.
__device__ __forceinline__ void add_report(double *rep, int e, int k, double v, bool valid) {
    unsigned long long m = __ballot(valid);
    if (m == 0) return;
    int lead = __ffsll((long long)m) - 1;
    int el = __shfl(e, lead);
    bool same = __all(!valid || e == el);
    if (same) {
        double x = valid ? v : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
        if (lane_id() == lead && x != 0.0) atomicAdd(&rep[(int64_t)el * 5 + k], x);
    } else if (valid && v != 0.0) {
        atomicAdd(&rep[(int64_t)e * 5 + k], v);
    }
}

__device__ __forceinline__ int find_event(const int64_t *off, int n_ev, int64_t s) {
    int lo = 0, hi = n_ev - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= s) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ================================================================================================= scans
// Exclusive scans of one or two 64-bit arrays of the same length or not (blockIdx.y); an array's last element is taken as 0,
// so that it receives the total, which also goes to `total` (and its upper part to `total_hi`, for the pixel counts).  With
// `mark` every count > 0 gets a one in the bits above 40, so one scan yields pair offsets and slot indices.  Short arrays
// take one workgroup and one launch each, or together (a launch costs more than their scan); longer ones a reduction per
// tile, a scan of the tiles' sums and a scan per tile.
constexpr int kScanPT = 8;
constexpr int kScanTile = kWG * kScanPT;
constexpr int kScanOneWG = 1024;
constexpr int64_t kScanOne = 16384;                     // elements of an array that one workgroup takes: two passes

struct ScanJob {
    uint64_t *data;
    int64_t n;
    int64_t *total, *total_hi;
    bool mark;
    __device__ __forceinline__ uint64_t at(int64_t i) const {
        const uint64_t v = i < n - 1 ? data[i] : 0;
        return mark && v ? v | (1ull << 40) : v;
    }
    __device__ __forceinline__ void put(int64_t i, uint64_t v) const {
        data[i] = v;
        if (i == n - 1 && total) {
            *total = (int64_t)(total_hi ? v & kMask40 : v);
            if (total_hi) *total_hi = (int64_t)(v >> 40);
        }
    }
};
struct ScanJobs {
    ScanJob job[2];
};

template <int WG>
__device__ __forceinline__ uint64_t block_exclusive(uint64_t v, uint64_t *lds, uint64_t &total) {
    // wavefront inclusive scan
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wv] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t run = 0;
        for (int i = 0; i < WG / 64; ++i) { const uint64_t t = lds[i]; lds[i] = run; run += t; }
        lds[WG / 64] = run;
    }
    __syncthreads();
    const uint64_t res = x - v + lds[wv];
    total = lds[WG / 64];
    __syncthreads();
    return res;
}

__global__ __launch_bounds__(kScanOneWG) void k_scan_one(ScanJobs jobs) {
    __shared__ uint64_t lds[kScanOneWG / 64 + 1];
    const ScanJob j = jobs.job[blockIdx.y];
    uint64_t carry = 0;
    for (int64_t b0 = 0; b0 < j.n; b0 += kScanOneWG * kScanPT) {
        const int64_t base = b0 + (int64_t)threadIdx.x * kScanPT;
        uint64_t v[kScanPT], s = 0, tot;
#pragma unroll
        for (int i = 0; i < kScanPT; ++i) {
            v[i] = j.at(base + i);
            s += v[i];
        }
        uint64_t run = block_exclusive<kScanOneWG>(s, lds, tot) + carry;
        carry += tot;
#pragma unroll
        for (int i = 0; i < kScanPT; ++i)
            if (base + i < j.n) { j.put(base + i, run); run += v[i]; }
    }
}

__global__ __launch_bounds__(kWG) void k_scan_reduce(ScanJobs jobs, uint64_t *part, int64_t stride) {
    __shared__ uint64_t lds[kWG / 64 + 1];
    const ScanJob j = jobs.job[blockIdx.y];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPT;
    uint64_t s = 0, tot;
#pragma unroll
    for (int i = 0; i < kScanPT; ++i) s += j.at(base + i);
    block_exclusive<kWG>(s, lds, tot);
    if (threadIdx.x == 0) part[blockIdx.y * stride + blockIdx.x] = tot;
}

__global__ __launch_bounds__(kWG) void k_scan_partials(uint64_t *part, int64_t stride, int64_t nb) {
    __shared__ uint64_t lds[kWG / 64 + 1];
    part += blockIdx.y * stride;
    uint64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kWG) {
        const int64_t i = b0 + threadIdx.x;
        const uint64_t v = i < nb ? part[i] : 0;
        uint64_t tot;
        const uint64_t ex = block_exclusive<kWG>(v, lds, tot);
        if (i < nb) part[i] = ex + carry;
        carry += tot;
    }
}

__global__ __launch_bounds__(kWG) void k_scan_apply(ScanJobs jobs, const uint64_t *part, int64_t stride) {
    __shared__ uint64_t lds[kWG / 64 + 1];
    const ScanJob j = jobs.job[blockIdx.y];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPT;
    uint64_t v[kScanPT], s = 0, tot;
#pragma unroll
    for (int i = 0; i < kScanPT; ++i) {
        v[i] = j.at(base + i);
        s += v[i];
    }
    uint64_t run = block_exclusive<kWG>(s, lds, tot) + part[blockIdx.y * stride + blockIdx.x];
#pragma unroll
    for (int i = 0; i < kScanPT; ++i)
        if (base + i < j.n) { j.put(base + i, run); run += v[i]; }
}

int64_t scan_tmp_needed(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

static void scan_jobs(const ScanJobs &jobs, int n_job, void *tmp, hipStream_t st) {
    int64_t n = 0;
    for (int i = 0; i < n_job; ++i) n = std::max(n, jobs.job[i].n);
    if (n <= 0) return;
    if (n <= kScanOne) {
        k_scan_one<<<dim3(1, (unsigned)n_job), kScanOneWG, 0, st>>>(jobs);
        return;
    }
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    uint64_t *part = (uint64_t *)tmp;
    k_scan_reduce<<<dim3((unsigned)nb, (unsigned)n_job), kWG, 0, st>>>(jobs, part, nb);
    k_scan_partials<<<dim3(1, (unsigned)n_job), kWG, 0, st>>>(part, nb, nb);
    k_scan_apply<<<dim3((unsigned)nb, (unsigned)n_job), kWG, 0, st>>>(jobs, part, nb);
}

void scan_exclusive(int64_t *data, int64_t n, int64_t *total, void *tmp, hipStream_t st) {
    scan_jobs(ScanJobs{{{(uint64_t *)data, n, total, nullptr, false}, {}}}, 1, tmp, st);
}
void scan_exclusive2(int64_t *a, int64_t *b, int64_t n, int64_t *total_a, int64_t *total_b, void *tmp, hipStream_t st) {
    scan_jobs(ScanJobs{{{(uint64_t *)a, n, total_a, nullptr, false}, {(uint64_t *)b, n, total_b, nullptr, false}}}, 2, tmp,
              st);
}

// ================================================================================================= quench / drift
struct QDOut {
    float q_r, q_a, t_drift, sigma_t, sigma_time, dedx;
    int32_t n_points, flags;
};

// Recombination (Sec. 3.1) and drift (Sec. 3.2) of segment s, plus its local reference frame.
__device__ __forceinline__ void segment_setup(const DevParams &P, const SegArrays &S, int64_t s, SegInfo &g, QDOut &o) {
    const float x0 = S.x0[s], y0 = S.y0[s], z0 = S.z0[s], t0 = S.t0[s];
    const float x1 = S.x1[s], y1 = S.y1[s], z1 = S.z1[s], t1 = S.t1[s];
    const float E = S.energy[s];
    int32_t flags = 0;
    const float dx = __fsub_rn(x1, x0), dy = __fsub_rn(y1, y0), dz = __fsub_rn(z1, z0), dt = __fsub_rn(t1, t0);
    // number of sample points (integer decided in IEEE single precision, no contraction)
    const float L2 = __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
    const float L = __fsqrt_rn(L2);
    const float cN = ceilf(__fdiv_rn(L, P.step));
    const int32_t N = cN >= 1.0f ? (int32_t)fminf(cN, 1.0e8f) : 1;
    float dedx;
    if (L > 0.0f) dedx = __fdiv_rn(E, L);                         // constant within the segment (Sec. 2)
    else if (S.dedx && isfinite(S.dedx[s])) dedx = S.dedx[s];
    else { dedx = 0.0f; flags |= SEG_INVALID; }
    // finite, and small enough that bin / tick indices stay far from int32 limits (|coordinate| <= 1e6)
    const float cmax = fmaxf(fmaxf(fmaxf(fabsf(x0), fabsf(y0)), fmaxf(fabsf(z0), fabsf(t0))),
                             fmaxf(fmaxf(fabsf(x1), fabsf(y1)), fmaxf(fabsf(z1), fabsf(t1))));
    const bool fin = isfinite(x0) && isfinite(y0) && isfinite(z0) && isfinite(t0) && isfinite(x1) && isfinite(y1) &&
                     isfinite(z1) && isfinite(t1) && isfinite(E);       // (fmaxf would drop NaNs)
    if (!(fin && cmax <= 1.0e6f && E >= 0.0f)) flags |= SEG_INVALID;
    if (N > 65536) flags |= SEG_TOO_LONG;
    float R;
    if (P.recomb_model == 0) {
        R = P.birks_ab / (1.0f + P.birks_kb_eps * dedx);           // eq. (birks)
    } else {
        const float xi = P.box_beta_eps * dedx;                    // eq. (box)
        R = xi > 0.0f ? logf(P.box_alpha + xi) / xi : -1.0f;
        if (!(R >= 0.0f)) { R = 0.0f; flags |= SEG_BOX_CLAMP; }
    }
    const float qr = R * (E * P.inv_w_ion);
    const float zm = 0.5f * (z0 + z1);
    const float td = fabsf(zm - P.za_hi) * P.inv_vd_hi;            // eq. (drift) at the midpoint
    const float qa = qr * expf(-td * P.inv_lifetime);              // eq. (lifetime)
    const float sT = sqrtf(P.two_dt * td);                         // sigma = sqrt(2 D t)
    const float sL = sqrtf(P.two_dl * td) * P.inv_vd_hi;           // longitudinal, as time

    g.q_r = qr; g.q_a = qa; g.q_pt = qa / (float)N; g.t_drift = td;
    g.sigma_t = sT; g.sigma_time = sL; g.dedx = dedx;
    g.n_points = N;
    float qa_seg = qa;
    // local frame: reference bin / tick of the start point and exact offsets
    ref_offset(x0, 0.0f, P.x0_hi, P.x0_lo, P.b_hi, P.b_lo, g.u_ref, g.ox);
    ref_offset(y0, 0.0f, P.y0_hi, P.y0_lo, P.b_hi, P.b_lo, g.v_ref, g.oy);
    float zh, zl;
    two_sum(z0, -P.za_hi, zh, zl);
    zl = __fsub_rn(zl, P.za_lo);
    const float dh = fabsf(zh), dl = zh >= 0.0f ? zl : -zl;       // |z0 - z_anode| as hi + lo
    const float q = __fmul_rn(dh, P.inv_vd_hi);
    const float qe = __fadd_rn(fmaf(dh, P.inv_vd_hi, -q), __fadd_rn(__fmul_rn(dh, P.inv_vd_lo), __fmul_rn(dl, P.inv_vd_hi)));
    float vh, ve;
    two_sum(t0, q, vh, ve);
    ref_offset(vh, __fadd_rn(ve, qe), P.tb_hi, P.tb_lo, P.tick_hi, P.tick_lo, g.a_ref, g.ot);
    const float zz0 = __fsub_rn(z0, P.za_hi), zz1 = __fsub_rn(z1, P.za_hi);
    const bool straddle = (zz0 < 0.0f && zz1 > 0.0f) || (zz0 > 0.0f && zz1 < 0.0f);
    const float sg = (zz0 > 0.0f || (zz0 == 0.0f && zz1 >= 0.0f)) ? 1.0f : -1.0f;
    g.dx = dx; g.dy = dy; g.dz = dz; g.dt = dt; g.zz0 = zz0;
    g.dta = fmaf(sg * dz, P.inv_vd_hi, dt);
    if (straddle) flags |= SEG_STRADDLE;
    g.flags = flags;
    if (P.per_point && !(flags & (SEG_INVALID | SEG_TOO_LONG))) {
        // collected charge = sum of the points' charges; the box uses the widths of the point farthest from the
        // anode (the widest cloud), a superset of the points' own supports
        float sum = 0.0f, cmp = 0.0f;
        for (int32_t mu = 0; mu < N; ++mu) {
            float q, a, b;
            point_drift(g, P, mu, q, a, b);
            const float y = q - cmp, t = sum + y;
            cmp = (t - sum) - y;
            sum = t;
        }
        qa_seg = sum;
        g.q_a = sum;
        g.q_pt = sum / (float)N;
        const float tdm = fmaxf(fabsf(zz0), fabsf(zz1)) * P.inv_vd_hi;
        g.sigma_t = sqrtf(P.two_dt * tdm);
        g.sigma_time = sqrtf(P.two_dl * tdm) * P.inv_vd_hi;
    }
    o.q_r = qr; o.q_a = qa_seg; o.t_drift = td; o.sigma_t = sT; o.sigma_time = sL; o.dedx = dedx;
    o.n_points = N; o.flags = flags;
}

// Charge box (tick x bin x bin) that the truncated clouds of the sample points can reach, and the pixel
// rectangle whose table reach meets it.
__device__ __forceinline__ void segment_box(const DevParams &P, SegInfo &g) {
    float lx0, ly0, lt0, lx1, ly1, lt1;
    point_local(g, P, 0, lx0, ly0, lt0);
    point_local(g, P, g.n_points - 1, lx1, ly1, lt1);
    float tmin = fminf(lt0, lt1), tmax = fmaxf(lt0, lt1);
    if ((g.flags & SEG_STRADDLE) && !(g.flags & (SEG_TOO_LONG | SEG_INVALID))) {
        for (int32_t mu = 1; mu < g.n_points - 1; ++mu) {
            float a, b, t;
            point_local(g, P, mu, a, b, t);
            tmin = fminf(tmin, t);
            tmax = fmaxf(tmax, t);
        }
    }
    const float ext = P.nsig * g.sigma_t, ext_t = P.nsig * g.sigma_time;
    const int32_t ulo = (int32_t)floorf(__fdiv_rn(fminf(lx0, lx1) - ext, P.b_hi));
    const int32_t uhi = (int32_t)floorf(__fdiv_rn(fmaxf(lx0, lx1) + ext, P.b_hi));
    const int32_t vlo = (int32_t)floorf(__fdiv_rn(fminf(ly0, ly1) - ext, P.b_hi));
    const int32_t vhi = (int32_t)floorf(__fdiv_rn(fmaxf(ly0, ly1) + ext, P.b_hi));
    const int32_t alo = (int32_t)floorf(__fdiv_rn(tmin - ext_t, P.tick_hi));
    const int32_t ahi = (int32_t)floorf(__fdiv_rn(tmax + ext_t, P.tick_hi));
    g.u0 = g.u_ref + ulo; g.nu = uhi - ulo + 1;
    g.v0 = g.v_ref + vlo; g.nv = vhi - vlo + 1;
    g.a0 = g.a_ref + alo; g.na = ahi - alo + 1;
    g.na_pad = (g.na + P.cell_pad - 1) / P.cell_pad * P.cell_pad;
    if (!(g.nu >= 1 && g.nu <= kBoxMax && g.nv >= 1 && g.nv <= kBoxMax && g.na >= 1 && g.na <= kNaMax))
        g.flags |= SEG_TOO_LONG;
    // pixel ix reaches sub-pixel bins u in [ix*nsub + nsub/2 - bx, ix*nsub + nsub/2 + bx - 1]
    const int32_t h = P.nsub / 2;
    g.ix0 = max(ceil_div(g.u0 - h - P.bx + 1, P.nsub), 0);
    g.ix1 = min(floor_div(g.u0 + g.nu - 1 - h + P.bx, P.nsub), P.nx - 1);
    g.iy0 = max(ceil_div(g.v0 - h - P.by + 1, P.nsub), 0);
    g.iy1 = min(floor_div(g.v0 + g.nv - 1 - h + P.by, P.nsub), P.ny - 1);
    if (g.flags & (SEG_INVALID | SEG_TOO_LONG)) { g.ix1 = g.ix0 - 1; }
    g.n_pairs = (g.ix1 >= g.ix0 && g.iy1 >= g.iy0) ? (g.ix1 - g.ix0 + 1) * (g.iy1 - g.iy0 + 1) : 0;
}

__global__ __launch_bounds__(kWG) void k_quench_drift(DevParams P, SegArrays S, int64_t n_seg, const int64_t *ev_off,
                                                      int32_t n_ev, SegInfo *si, int64_t *cell_cnt, uint64_t *pix_cnt,
                                                      DevHeader *H, double *report) {
    const int64_t s = (int64_t)blockIdx.x * kWG + threadIdx.x;
    const bool valid = s < n_seg;
    SegInfo g = {};
    QDOut o;
    int e = 0;
    if (valid) {
        e = find_event(ev_off, n_ev, s);
        segment_setup(P, S, s, g, o);
        segment_box(P, g);
        g.event = e;
        si[s] = g;
        const bool skip = g.flags & (SEG_INVALID | SEG_TOO_LONG);
        cell_cnt[s] = skip ? 0 : (int64_t)g.nu * g.nv * g.na_pad;
        if (!skip) atomicAdd((unsigned long long *)&H->n_colseg, (unsigned long long)g.nu * g.nv);
        if (g.flags & SEG_INVALID) atomicOr(&H->status, ST_INVALID);
        if (g.flags & SEG_TOO_LONG) atomicOr(&H->status, ST_TOO_LONG);
        // pairs per pixel: the reach is a rectangle of the event's pixel grid, counted by a difference array (+1 at
        // its first corner, -1 / -1 / +1 one past it; prefix sums along the rows and down the columns follow)
        if (g.ix1 >= g.ix0 && g.iy1 >= g.iy0) {
            unsigned long long *pc = (unsigned long long *)pix_cnt + (int64_t)e * P.npx;
            const int32_t xb = g.ix1 + 1, yb = g.iy1 + 1;
            atomicAdd(&pc[g.iy0 * P.nx + g.ix0], 1ull);
            if (xb < P.nx) atomicAdd(&pc[g.iy0 * P.nx + xb], ~0ull);
            if (yb < P.ny) {
                atomicAdd(&pc[yb * P.nx + g.ix0], ~0ull);
                if (xb < P.nx) atomicAdd(&pc[yb * P.nx + xb], 1ull);
            }
        }
    }
    add_report(report, e, 0, valid ? (double)g.q_r : 0.0, valid);
    add_report(report, e, 1, valid ? (double)g.q_a : 0.0, valid);
}

// inclusive prefix sums along each row of a set of grids (one wavefront per row of len values)
__global__ __launch_bounds__(kWG) void k_prefix_rows(int64_t *a, int64_t n_rows, int32_t len) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (row >= n_rows) return;
    int64_t *r = a + row * len, carry = 0;
    for (int32_t c0 = 0; c0 < len; c0 += 64) {
        int64_t x = c0 + lane < len ? r[c0 + lane] : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        x += carry;
        if (c0 + lane < len) r[c0 + lane] = x;
        carry = __shfl(x, 63);
    }
}

// inclusive prefix sums down each column of n_ev grids of CU rows x CV values.  A workgroup takes 16 columns, every 16
// lanes a sixteenth of their rows, which they add up first.  (A thread down a whole column is one long chain of loads: 88 us
// for 1490 x 1490 columns, 21 so; 64 columns by 16 parts took 42, and workgroups of 1024 threads wait for a free CU beside
// the charge cells on the other stream.)
constexpr int kColsWG = 256, kColsWide = 16, kColsParts = kColsWG / kColsWide;
__global__ __launch_bounds__(kColsWG) void k_prefix_cols(int64_t *a, int32_t n_ev, int32_t CU, int32_t CV) {
    __shared__ int64_t lds[kColsParts][kColsWide];
    const int32_t n_blk = (CV + kColsWide - 1) / kColsWide, ev = blockIdx.x / n_blk;
    const int32_t col = threadIdx.x % kColsWide, part = threadIdx.x / kColsWide;
    const int32_t v = (blockIdx.x - ev * n_blk) * kColsWide + col;
    const int32_t per = (CU + kColsParts - 1) / kColsParts, u0 = min(part * per, CU), u1 = v < CV ? min(u0 + per, CU) : u0;
    int64_t *p = a + (int64_t)ev * CU * CV + v;
    int64_t sum = 0;
    for (int32_t u = u0; u < u1; u += 8) {
        int64_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = u + i < u1 ? p[(int64_t)(u + i) * CV] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += x[i];
    }
    lds[part][col] = sum;
    __syncthreads();
    int64_t run = 0;
    for (int32_t i = 0; i < part; ++i) run += lds[i][col];
    for (int32_t u = u0; u < u1; u += 8) {
        int64_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = u + i < u1 ? p[(int64_t)(u + i) * CV] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            run += x[i];
            if (u + i < u1) p[(int64_t)(u + i) * CV] = run;
        }
    }
}
static void launch_prefix_cols(int64_t *a, int32_t n_ev, int32_t CU, int32_t CV, hipStream_t st) {
    k_prefix_cols<<<(unsigned)(n_ev * ((CV + kColsWide - 1) / kColsWide)), kColsWG, 0, st>>>(a, n_ev, CU, CV);
}

void launch_quench_drift(const DevParams &P, const SegArrays &S, const Work &w, hipStream_t st) {
    const int64_t n_gp = (int64_t)w.n_ev * P.npx;
    if (w.n_seg > 0)
        k_quench_drift<<<(unsigned)((w.n_seg + kWG - 1) / kWG), kWG, 0, st>>>(P, S, w.n_seg, w.seg_ev_off, w.n_ev, w.si,
                                                                            w.cell_off, w.pix_cnt, w.hdr, w.report);
    if (n_gp > 0) {
        const int64_t rows = (int64_t)w.n_ev * P.ny;
        k_prefix_rows<<<(unsigned)((rows + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>((int64_t *)w.pix_cnt, rows, P.nx);
        launch_prefix_cols((int64_t *)w.pix_cnt, w.n_ev, P.ny, P.nx, st);
    }
    scan_jobs(ScanJobs{{{w.pix_cnt, n_gp + 1, &w.hdr->n_pairs, &w.hdr->n_slots, true},
                        {(uint64_t *)w.cell_off, w.n_seg + 1, &w.hdr->n_cells, nullptr, false}}}, 2, w.scan_tmp, st);
}

__global__ void k_stage_qd(DevParams P, SegArrays S, int64_t n, float *out_f, int32_t *out_i) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    SegInfo g = {};
    QDOut o;
    segment_setup(P, S, s, g, o);
    float *f = out_f + 6 * s;
    f[0] = o.q_r; f[1] = o.q_a; f[2] = o.t_drift; f[3] = o.sigma_t; f[4] = o.sigma_time; f[5] = o.dedx;
    out_i[2 * s] = o.n_points;
    out_i[2 * s + 1] = o.flags & (SEG_BOX_CLAMP | SEG_INVALID);
}

void launch_stage_quench_drift(const DevParams &P, const SegArrays &S, int64_t n, float *out_f, int32_t *out_i,
                               hipStream_t st) {
    if (n > 0) k_stage_qd<<<(unsigned)((n + kWG - 1) / kWG), kWG, 0, st>>>(P, S, n, out_f, out_i);
}

// ================================================================================================= slots / pairs
// Also the events' first slots, and zeros in the packet counts (n_zero words).
__global__ void k_slots(DevParams P, int64_t n_gp, const uint64_t *pix_off, int32_t *pix_slot, int32_t *slot_gp,
                        int64_t *slot_off, int32_t *pixel_id_out, int64_t *ev_pix_off, const DevHeader *H, uint32_t *zero,
                        int64_t n_zero) {
    int64_t gp = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = gp; i < n_zero; i += (int64_t)gridDim.x * blockDim.x) zero[i] = 0u;
    if (gp > n_gp) return;
    uint64_t v = pix_off[gp];
    if (ev_pix_off && gp % P.npx == 0) ev_pix_off[gp / P.npx] = (int64_t)(v >> 40);
    if (gp == n_gp) {
        slot_off[H->n_slots] = H->n_pairs;
        return;
    }
    uint64_t vn = pix_off[gp + 1];
    bool active = (vn >> 40) > (v >> 40);
    int64_t slot = (int64_t)(v >> 40);
    pix_slot[gp] = active ? (int32_t)slot : -1;
    if (active) {
        slot_gp[slot] = (int32_t)gp;
        slot_off[slot] = (int64_t)(v & kMask40);
        if (pixel_id_out) pixel_id_out[slot] = (int32_t)(gp % P.npx);
    }
}

void launch_slots(const DevParams &P, const Work &w, int32_t *pixel_id_out, int64_t *ev_pix_off, void *zero,
                  int64_t zero_bytes, hipStream_t st) {
    const int64_t n_gp = (int64_t)w.n_ev * P.npx;
    k_slots<<<(unsigned)((n_gp + 1 + kWG - 1) / kWG), kWG, 0, st>>>(P, n_gp, w.pix_cnt, w.pix_slot, w.slot_gp, w.slot_off,
                                                                   pixel_id_out, ev_pix_off, w.hdr, (uint32_t *)zero,
                                                                   zero_bytes / 4);
}

// Also stores each segment's scanned charge-cell offset in its record (the scan runs after k_quench_drift); with
// pairs = null only that.
__global__ __launch_bounds__(kWG) void k_fill_pairs(DevParams P, SegInfo *si, int64_t n_seg, const int64_t *cell_off,
                                                    const uint64_t *pix_off, int32_t *cursor, int32_t *pairs) {
    int64_t s = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (s >= n_seg) return;
    si[s].cell_off = cell_off[s];
    if (!pairs) return;                                  // the summed induction needs no pair lists
    const SegInfo &g = si[s];
    const int64_t base = (int64_t)g.event * P.npx;
    for (int32_t iy = g.iy0; iy <= g.iy1; ++iy)
        for (int32_t ix = g.ix0; ix <= g.ix1; ++ix) {
            int64_t gp = base + iy * P.nx + ix;
            int64_t pos = (int64_t)(pix_off[gp] & kMask40) + atomicAdd(&cursor[gp], 1);
            pairs[pos] = (int32_t)s;
        }
}

// Zero fill by a kernel (a memset node recorded into a captured graph is avoided: the pipeline's launch sequence
// may be captured).
__global__ void k_zero_words(uint32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// Several buffers at once, and the events' offsets and ids of a call with few of them (their copies would be a launch each).
__global__ void k_start(ZeroRanges z, EventList ev, int64_t *ev_off, uint64_t *ev_ids) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
#pragma unroll
    for (int r = 0; r < kZeroRanges; ++r)
        for (int64_t i = t; i < z.words[r]; i += (int64_t)gridDim.x * blockDim.x) z.p[r][i] = 0u;
    if (t <= ev.n && ev_off) ev_off[t] = ev.off[t];
    if (t < ev.n && ev_off) ev_ids[t] = ev.id[t];
}
void launch_start(const ZeroRanges &z, const EventList &ev, int64_t *ev_off, uint64_t *ev_ids, hipStream_t st) {
    int64_t most = kWG;
    for (int r = 0; r < kZeroRanges; ++r) most = std::max(most, z.words[r]);
    k_start<<<(unsigned)std::min<int64_t>((most + kWG - 1) / kWG, 4096), kWG, 0, st>>>(z, ev, ev_off, ev_ids);
}

__global__ void k_store_u64(uint64_t *p, uint64_t v) { *p = v; }

void launch_store_u64(uint64_t *p, uint64_t v, hipStream_t st) { k_store_u64<<<1, 1, 0, st>>>(p, v); }

void launch_zero(void *p, int64_t bytes, hipStream_t st) {
    const int64_t n = bytes / 4;
    if (n <= 0) return;
    const int64_t g = std::min<int64_t>((n + kWG - 1) / kWG, 4096);
    k_zero_words<<<(unsigned)g, kWG, 0, st>>>((uint32_t *)p, n);
}

void launch_fill_pairs(const DevParams &P, const Work &w, hipStream_t st) {
    if (w.n_seg > 0)
        k_fill_pairs<<<(unsigned)((w.n_seg + kWG - 1) / kWG), kWG, 0, st>>>(P, w.si, w.n_seg, w.cell_off, w.pix_cnt,
                                                                          w.cursor, w.pairs_unsorted);
}

// Each pixel's segment list in ascending segment id (ids are unique within a list): rank = number of smaller ids.
constexpr int kSortLds = 4096;
__global__ __launch_bounds__(kWG) void k_sort_pairs(const int64_t *slot_off, const DevHeader *H, const int32_t *in,
                                                    int32_t *out) {
    __shared__ int32_t lds[kSortLds];
    const int64_t n_slots = H->n_slots;
    for (int64_t slot = blockIdx.x; slot < n_slots; slot += gridDim.x) {
        const int64_t off = slot_off[slot];
        const int32_t cnt = (int32_t)(slot_off[slot + 1] - off);
        const int32_t *src = in + off;
        if (cnt <= kSortLds) {
            for (int i = threadIdx.x; i < cnt; i += kWG) lds[i] = src[i];
            __syncthreads();
            for (int i = threadIdx.x; i < cnt; i += kWG) {
                int32_t v = lds[i], r = 0;
                for (int j = 0; j < cnt; ++j) r += lds[j] < v;
                out[off + r] = v;
            }
            __syncthreads();
        } else {
            for (int i = threadIdx.x; i < cnt; i += kWG) {
                int32_t v = src[i], r = 0;
                for (int j = 0; j < cnt; ++j) r += src[j] < v;
                out[off + r] = v;
            }
        }
    }
}

void launch_sort_pairs(const Work &w, int64_t n_slots_host, hipStream_t st) {
    int64_t g = n_slots_host < 1 ? 1 : (n_slots_host > 8192 ? 8192 : n_slots_host);
    k_sort_pairs<<<(unsigned)g, kWG, 0, st>>>(w.slot_off, w.hdr, w.pairs_unsorted, w.pairs);
}

// ================================================================================================= charge cells
constexpr int kCellLds = 6144;    // floats (24 KB: several workgroups per CU; long segments take several passes)
constexpr int kCellRows = 4 * kBoxMax + 2 * kNaMax + 9;   // rows of a pass at most (bins, edges, 6): one more float each

// Monte Carlo cells of one segment (the paper's estimator of eq. (rho) with M = P.mc_draws perturbations per point):
// every moved copy of a sample point adds one hit to the cell that contains it (integer counts, in LDS when the box
// fits, two to a word where none can pass 16 bits, else in the cell buffer itself), then cell = hits * q / M.  Counts make
// the result independent of the order in which the workgroup's threads land their hits.  The cell buffer's atomics need
// device fences, which cost more than the draws: 200 segments of 139 draws in boxes of 5600 cells, a third of them beyond
// 6144, took 56 us by 256 threads with one count a word, 15 so.
template <int WG>
__device__ void mc_cells(const DevParams &P, const SegInfo &g, uint32_t seg, uint64_t event, float *out,
                         uint32_t *lds, int64_t ncell) {
    const int tid = threadIdx.x;
    const uint32_t M = (uint32_t)P.mc_draws;
    const int64_t nd = (int64_t)g.n_points * M;
    const int two = nd < 65536;
    const bool in_lds = ncell <= (int64_t)(kCellLds + kCellRows) << two;
    uint32_t *hist = in_lds ? lds : (uint32_t *)out;
    const int sh = in_lds ? two : 0;
    for (int64_t c = tid; c < (ncell + sh) >> sh; c += WG) hist[c] = 0u;
    if (!in_lds) __threadfence();                       // (a device fence per wavefront costs more than the draws)
    __syncthreads();
    for (int64_t d = tid; d < nd; d += WG) {
        float lx, ly, lt, gx, gy, gt;
        point_local(g, P, (int32_t)(d / M), lx, ly, lt);
        mc_normals(P, seg, (uint32_t)d, event, gx, gy, gt);
        // the truncated cloud lies inside the box; the clamps only guard the memory
        const int32_t u = min(max(g.u_ref + local_bin(fmaf(g.sigma_t, gx, lx), P.b_hi, P.b_lo) - g.u0, 0), g.nu - 1);
        const int32_t v = min(max(g.v_ref + local_bin(fmaf(g.sigma_t, gy, ly), P.b_hi, P.b_lo) - g.v0, 0), g.nv - 1);
        const int32_t a =
            min(max(g.a_ref + local_bin(fmaf(g.sigma_time, gt, lt), P.tick_hi, P.tick_lo) - g.a0, 0), g.na - 1);
        const int64_t c = ((int64_t)u * g.nv + v) * g.na_pad + a;
        atomicAdd(&hist[c >> sh], sh && (c & 1) ? 0x10000u : 1u);
    }
    if (!in_lds) __threadfence();
    __syncthreads();
    const float w = __fdiv_rn(g.q_pt, (float)M);
    for (int64_t c = tid; c < ncell; c += WG) {
        const uint32_t h = sh ? hist[c >> 1] >> (16 * (c & 1)) & 0xffffu
                           : in_lds ? hist[c]
                                    : __hip_atomic_load(&hist[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        out[c] = (float)h * w;
    }
    __syncthreads();
}

// The charge box of one pass over np sample points as a matrix product on the FP32 matrix cores: with the point index
// m as the contraction, cells[(u, v)][a] = sum_m (fx[u][m] fy[v][m]) ft[a][m], times q (the point charge when every
// point carries the same charge, else 1: ft then already holds it).  16x16x4 MFMA tiles: rows are 16 (u, v) columns
// of the box, columns 16 ticks, each instruction takes 4 points (lane l gives A[l % 16][l / 16] = fx fy of its row's
// column at point l / 16 and B[l / 16][l % 16] = ft of that point at its tick).  Each wavefront of the workgroup takes
// 2 x 2 blocks of tiles in turn, so every A value serves two tiles and every B value two.  Out-of-box rows and ticks
// repeat one of the box and are not written; points past the last one meet ft = 0.  `first` writes the pass's sums,
// otherwise they are added.
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
template <int WG>
__device__ __forceinline__ void cells_mfma(const float *fx, const float *fy, const float *ft, int32_t nu, int32_t nv,
                                           int32_t nap, int32_t np, int32_t pitch, float q, bool first, float *out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int32_t ncol = nu * nv, tm = (ncol + 15) / 16, tn = (nap + 15) / 16;
    const int32_t bm = (tm + 1) / 2, bn = (tn + 1) / 2;
    const int32_t il = lane & 15, kl = lane >> 4;
    for (int32_t blk = wv; blk < bm * bn; blk += WG / 64) {
        const int32_t mi0 = (blk / bn) * 2, nj0 = (blk % bn) * 2;
        const float *px[2], *py[2], *pt[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int32_t c = min((mi0 + t) * 16 + il, ncol - 1), u = c / nv;
            px[t] = fx + u * pitch + kl;
            py[t] = fy + (c - u * nv) * pitch + kl;
            pt[t] = ft + min((nj0 + t) * 16 + il, nap - 1) * pitch + kl;
        }
        floatx4 D[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) D[i][j] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
        auto step = [&](int32_t m, bool all) {
            float A[2], B[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int32_t at = all || m + kl < np ? m : np - 1 - kl;
                A[t] = px[t][at] * py[t][at];
                B[t] = all || m + kl < np ? pt[t][at] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) D[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[i], B[j], D[i][j], 0, 0, 0);
        };
        int32_t m0 = 0;
        for (; m0 + 4 <= np; m0 += 4) step(m0, true);
        if (m0 < np) step(m0, false);
        // lane l holds rows 4 (l / 16) + r of each tile (a box column) at column l % 16 (a tick)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t c = (mi0 + i) * 16 + 4 * kl + r, a = (nj0 + j) * 16 + il;
                    if (c < ncol && a < nap) {
                        const float v = D[i][j][r] * q;
                        float *o = out + (int64_t)c * nap + a;
                        if (first) *o = v; else *o += v;
                    }
                }
    }
}

template <int WG>
__global__ __launch_bounds__(WG, WG == kWG ? 5 : 4) void k_cells(DevParams P, const SegInfo *si, int64_t n_seg, float *cells,
                                               const int64_t *seg_ev_off, const uint64_t *event_ids, double *report) {
    __shared__ float sm[kCellLds + kCellRows];
    __shared__ double red[WG / 64];
    const int tid = threadIdx.x;
    const float end_tail = tail(P.nsig);
    for (int64_t s = blockIdx.x; s < n_seg; s += gridDim.x) {
        const SegInfo g = si[s];
        if (g.flags & (SEG_INVALID | SEG_TOO_LONG)) continue;
        const int32_t nu = g.nu, nv = g.nv, na = g.na, nap = g.na_pad, N = g.n_points;
        const int32_t row = nu + nv + nap, ne = nu + nv + na + 3;      // bins and bin edges of a point's three axes
        const int32_t pc = min(256, kCellLds / (row + ne + 6));
        const int64_t ncell = (int64_t)nu * nv * nap;
        float *out = cells + g.cell_off;
        if (P.mc_draws > 0)
            mc_cells<WG>(P, g, (uint32_t)(s - seg_ev_off[g.event]), event_ids[g.event], out, (uint32_t *)sm, ncell);
        for (int32_t mu0 = 0; mu0 < (P.mc_draws > 0 ? 0 : N); mu0 += pc) {
            const int32_t np = min(pc, N - mu0), pitch = np | 1;
            // rows of points (odd pitch: neighbouring rows in different banks)
            float *fx = sm, *fy = fx + pitch * nu, *ft = fy + pitch * nv;
            float *tl = ft + pitch * nap;               // [edge][point]: the edge's tail, negated below the mean
            float *pl = tl + pitch * ne;                // [6][point]: local x, y, t, widths, charge
            const uint32_t inv_np = 0xffffffffu / (uint32_t)np + 1u;   // r / np = hi(r inv_np) for r np < 2^32 (np > 1)
            // Per point and axis, the masses of consecutive bins (edges (k0 + j) * width from the reference edge)
            // of the point's Gaussian of width sigma, truncated at +-n sigma and renormalised, each taken as a
            // difference of tails on the side away from the mean.  Spread over the workgroup: each point's frame,
            // then every edge's tail, then every bin's mass from its two edges; neighbouring lanes take neighbouring
            // points of one edge, so most edges beyond the truncation (one tail for all) are skipped together.
            for (int m = tid; m < np; m += WG) {
                float q = 1.0f, sT = g.sigma_t, sL = g.sigma_time;
                point_local(g, P, mu0 + m, pl[m], pl[pitch + m], pl[2 * pitch + m]);
                if (P.per_point) point_drift(g, P, mu0 + m, q, sT, sL);
                pl[3 * pitch + m] = sT;
                pl[4 * pitch + m] = sL;
                pl[5 * pitch + m] = q;
            }
            __syncthreads();
            for (int r = tid; r < np * ne; r += WG) {
                const int32_t k = np > 1 ? (int32_t)__umulhi((uint32_t)r, inv_np) : r, m = r - k * np;
                const int ax = k <= nu ? 0 : k <= nu + nv + 1 ? 1 : 2;
                const int32_t j = ax == 0 ? k : ax == 1 ? k - nu - 1 : k - nu - nv - 2;
                const float l = pl[ax * pitch + m], sg = pl[(ax == 2 ? 4 : 3) * pitch + m];
                const int32_t k0 = ax == 0 ? g.u0 - g.u_ref : ax == 1 ? g.v0 - g.v_ref : g.a0 - g.a_ref;
                const float wh = ax == 2 ? P.tick_hi : P.b_hi, wl = ax == 2 ? P.tick_lo : P.b_lo;
                float t = 0.0f;
                if (sg > 0.0f) {
                    const float kf = (float)(k0 + j);
                    const float e = __fadd_rn(fmaf(kf, wh, -l), __fmul_rn(kf, wl));
                    const float z = fminf(fmaxf(e * (1.0f / sg), -P.nsig), P.nsig);
                    t = end_tail;
                    if (fabsf(z) < P.nsig) t = tail(z);
                    if (!(z >= 0.0f)) t = -t;               // the sign bit keeps the side of the mean
                }
                tl[k * pitch + m] = t;
            }
            __syncthreads();
            for (int r = tid; r < np * row; r += WG) {
                const int32_t k = np > 1 ? (int32_t)__umulhi((uint32_t)r, inv_np) : r, m = r - k * np;
                const int ax = k < nu ? 0 : k < nu + nv ? 1 : 2;
                const int32_t j = ax == 0 ? k : ax == 1 ? k - nu : k - nu - nv;
                float mass = 0.0f;
                if (ax < 2 || j < na) {
                    const float sg = pl[(ax == 2 ? 4 : 3) * pitch + m];
                    if (sg > 0.0f) {
                        // tmass only asks on which side of the mean each edge lies; an edge at z = 0 counted as
                        // above it gives the same value, (1 - 1/2) - ta = 1/2 - ta
                        const float *e = tl + (k + ax) * pitch + m;      // one edge more than bins per axis
                        const float a = e[0], b = e[pitch];
                        mass = tmass(__builtin_signbit(a) ? -1.0f : 1.0f, fabsf(a), __builtin_signbit(b) ? -1.0f : 1.0f,
                                     fabsf(b), P.inv_norm);
                    } else {                            // no spread: all of the point in the bin that holds it
                        const float l = pl[ax * pitch + m];
                        const float wh = ax == 2 ? P.tick_hi : P.b_hi;
                        const int32_t k0 = ax == 0 ? g.u0 - g.u_ref : ax == 1 ? g.v0 - g.v_ref : g.a0 - g.a_ref;
                        mass = j == (int32_t)floorf(__fdiv_rn(l, wh)) - k0 ? 1.0f : 0.0f;
                    }
                    if (ax == 2 && P.per_point) mass *= pl[5 * pitch + m];   // per point: its charge rides on the time masses
                }
                fx[k * pitch + m] = mass;               // (the rows of fy and ft follow those of fx)
            }
            __syncthreads();
            cells_mfma<WG>(fx, fy, ft, nu, nv, nap, np, pitch, P.per_point ? 1.0f : g.q_pt, mu0 == 0, out);
            __syncthreads();
        }
        // charge whose cells lie outside the pixel grid
        const int32_t ug = P.nx * P.nsub, vg = P.ny * P.nsub;
        if (g.u0 < 0 || g.u0 + nu > ug || g.v0 < 0 || g.v0 + nv > vg) {
            double loc = 0.0;
            for (int64_t c = tid; c < ncell; c += WG) {
                const int32_t uv = (int32_t)(c / nap);
                const int32_t v = g.v0 + uv % nv, u = g.u0 + uv / nv;
                if (u < 0 || u >= ug || v < 0 || v >= vg) loc += (double)out[c];
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) loc += __shfl_xor(loc, o);
            if (lane_id() == 0) red[tid >> 6] = loc;
            __syncthreads();
            if (tid == 0) {
                double t = 0.0;
                for (int i = 0; i < WG / 64; ++i) t += red[i];
                if (t != 0.0) atomicAdd(&report[(int64_t)g.event * 5 + 4], t);
            }
            __syncthreads();
        }
    }
}

// Up to one segment a CU, a workgroup of 1024 threads per segment, beyond that 256: with 200 segments of 139 points 40
// instead of 66 us, of 41 points 12.5 instead of 15; with 300 of 41 points 18 instead of 15.5, with 1000 of 139 128
// instead of 110.
constexpr int64_t kCellWide = 256;
void launch_cells(const DevParams &P, const Work &w, hipStream_t st) {
    if (w.n_seg <= 0) return;
    auto *k = w.n_seg <= kCellWide ? k_cells<1024> : k_cells<kWG>;
    k<<<(unsigned)std::min<int64_t>(w.n_seg, 8192), w.n_seg <= kCellWide ? 1024 : kWG, 0, st>>>(
        P, w.si, w.n_seg, w.cells, w.seg_ev_off, w.event_ids, w.report);
}

// ================================================================================================= induction
// A global-memory pointer whose value is taken from the first active lane (wave-uniform by construction).  The
// global address space is kept explicit so loads through it stay global loads (a generic pointer would become a
// flat load, whose completion order forces a full wait on every outstanding load).
typedef const float __attribute__((address_space(1))) *gfloat_ptr;
__device__ __forceinline__ gfloat_ptr uniform_ptr(const float *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (gfloat_ptr)(((uint64_t)hi << 32) | lo);
}
// The same for data that no kernel of the launch writes (charge cells during induction): loads through the
// constant address space become scalar loads into SGPRs, read by the whole wavefront at once.
typedef const float __attribute__((address_space(4))) *cfloat_ptr;
__device__ __forceinline__ cfloat_ptr uniform_cptr(const float *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (cfloat_ptr)(((uint64_t)hi << 32) | lo);
}

// Current of one (segment, pixel) pair on RT consecutive ticks nb .. nb+RT-1 (eq. (current)):
//   I[n] = sum over cells (a, u, v) in the pixel's reach of c[a,u,v] * R[n - a + T_R - 1, fold(u - uc), fold(v - vc)].
// The table column is zero-padded by kPad on both sides, so no bounds test is needed in the inner loop; the cell
// column is padded with zeros to a multiple of kAC ticks.
template <int RT>
__device__ __forceinline__ void pair_block(const DevParams &P, const float *__restrict__ cc0, int32_t nv, int32_t nap,
                                           int32_t u0, int32_t v0, int32_t a0, const float *__restrict__ Rpad,
                                           int32_t ulo, int32_t uhi, int32_t vlo, int32_t vhi, int32_t uc, int32_t vc,
                                           int32_t nb, float (&acc)[RT]) {
    const int32_t K0 = nb - a0 + P.t_r - 1 + kPad;
    for (int32_t u = ulo; u <= uhi; ++u) {
        const int32_t i = fold(u - uc);
        const float *ccu = cc0 + (int64_t)(u - u0) * nv * nap;
        for (int32_t v = vlo; v <= vhi; ++v) {
            const int32_t j = fold(v - vc);
            const float *col = Rpad + (int64_t)(i * P.by + j) * P.col_len + K0 - (kAC - 1);
            const float *cc = ccu + (int64_t)(v - v0) * nap;
            for (int32_t ac = 0; ac < nap; ac += kAC) {
                float w[RT + kAC - 1];
#pragma unroll
                for (int m = 0; m < RT + kAC - 1; ++m) w[m] = col[m - ac];
                float cv[kAC];
#pragma unroll
                for (int q = 0; q < kAC; ++q) cv[q] = cc[ac + q];
#pragma unroll
                for (int q = 0; q < kAC; ++q)
#pragma unroll
                    for (int r = 0; r < RT; ++r) acc[r] = fmaf(cv[q], w[r - q + kAC - 1], acc[r]);
            }
        }
    }
}

// Value of lane - 1 of the wavefront (DPP wave_shr:1); lane 0 has no source lane and keeps `lane0`.
__device__ __forceinline__ float shift_up_or(float v, float lane0) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, lane0),
                                                                  __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, false));
}


// The same product for RT = 8, streaming each table column through a ring of four 8-value register blocks.  Lane t
// covers ticks nb .. nb+7; for cell-tick block j (ticks a0 + 8j .. +7) its window is R[K0-8j-7 .. K0-8j+7], i.e.
// its block b_j = R[K0-8j .. +7] and seven values of b_{j+1} = R[K0-8j-8 .. -1], so every block serves two
// consecutive cell-tick blocks and is fetched once.  Block b_{j+3} is fetched into the slot of the dead block
// b_{j-1}, three blocks ahead; the next column's first three blocks are fetched while the current column runs.
//   Two ways to fetch b_{j+1}:
//   * SHIFT = false: every lane loads its own 8 values (two 16-byte loads when ALIGNED, i.e. K0 % 8 == 0);
//   * SHIFT = true: b_{j+1} is b_j of the lane below (DPP wave_shr:1); only lane 0 loads (its values come from
//     below the wavefront's span).  All 64 lanes must then execute the loop (inactive lanes get a safe in-bounds
//     base; their results are discarded, and lanes above an inactive lane are inactive too).
template <int S, bool SHIFT>
__device__ __forceinline__ void ring_block(float (&B)[4][8], const float (&cv)[kAC], float (&acc)[8]) {
    constexpr int N = (S + 1) & 3;
    if constexpr (SHIFT) {
#pragma unroll
        for (int k = 0; k < 8; ++k) B[N][k] = shift_up_or(B[S][k], B[N][k]);
    }
    // w[m] = R[K0 - 8j - 7 + m]: m < 7 from b_{j+1}[m + 1], m >= 7 from b_j[m - 7]
#pragma unroll
    for (int q = 0; q < kAC; ++q)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int m = r - q + kAC - 1;
            acc[r] = fmaf(cv[q], m < 7 ? B[N][m + 1] : B[S][m - 7], acc[r]);
        }
}

template <bool ALIGNED>
__device__ __forceinline__ void load8(const float *p, float (&d)[8]) {
    if constexpr (ALIGNED) {
        const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
        d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w; d[4] = b.x; d[5] = b.y; d[6] = b.z; d[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) d[k] = p[k];
    }
}

// Streams a sequence of (table column, cell column) pairs through the ring.  `col` is this lane's pointer to
// R[K0 .. K0+7] of the first table column, `cc` the first cell column (nblk blocks of kAC ticks).  adv(col, cc, nblk)
// moves to the next column (false at the end); it is called while the current column runs, so the next column's
// first blocks are in flight before they are needed.  done() runs after each column's last block.  Loads reach at
// most 8 * nblk + 16 values below K0 (every caller keeps them inside the column's zero padding); the cell values of
// the block after a column's last lie in the next column or in the buffer's kCellSlack tail.
template <bool SHIFT, bool ALIGNED, class Adv, class Done>
__device__ __forceinline__ void column_stream(const float *col, const float *cc, int32_t nblk, Adv adv, Done done,
                                              float (&acc)[8]) {
    const bool lane0 = lane_id() == 0;
    gfloat_ptr col0 = uniform_ptr(col);
    float F[8], P1[8] = {}, P2[8] = {};
    load8<ALIGNED>(col, F);
    if (!SHIFT) {
        load8<ALIGNED>(col - 8, P1);
        load8<ALIGNED>(col - 16, P2);
    } else if (lane0) {                                 // lane 0 alone loads what is shifted in at the bottom
#pragma unroll
        for (int k = 0; k < 8; ++k) { P1[k] = col0[k - 8]; P2[k] = col0[k - 16]; }
    }
    const float *cl = col;
    for (;;) {
        float B[4][8];
#pragma unroll
        for (int k = 0; k < 8; ++k) { B[0][k] = F[k]; B[1][k] = P1[k]; B[2][k] = P2[k]; B[3][k] = 0.0f; }
        gfloat_ptr c0 = col0;
        const float *cur = cl;
        cfloat_ptr ccu = uniform_cptr(cc);
        const int32_t nb_cur = nblk;
        const bool more = adv(cl, cc, nblk);
        if (more) {                                     // next column, one column ahead
            col0 = uniform_ptr(cl);
            load8<ALIGNED>(cl, F);
            if (!SHIFT) {
                load8<ALIGNED>(cl - 8, P1);
                load8<ALIGNED>(cl - 16, P2);
            } else if (lane0) {
#pragma unroll
                for (int k = 0; k < 8; ++k) { P1[k] = col0[k - 8]; P2[k] = col0[k - 16]; }
            }
        }
        float cvb[2][kAC];                              // cell values of the current and the next block
#pragma unroll
        for (int q = 0; q < kAC; ++q) cvb[0][q] = ccu[q];
        for (int32_t j = 0; j < nb_cur; j += 4) {
#define LTS_RING_STEP(S)                                                                        \
    {                                                                                           \
        _Pragma("unroll") for (int q = 0; q < kAC; ++q) cvb[(S + 1) & 1][q] = ccu[kAC * (j + S + 1) + q]; \
        if constexpr (!SHIFT) {                                                                 \
            load8<ALIGNED>(cur - 8 * (j + S + 3), B[(S + 3) & 3]);                              \
        } else if (lane0) {                                                                     \
            _Pragma("unroll") for (int k = 0; k < 8; ++k) B[(S + 3) & 3][k] = c0[k - 8 * (j + S + 3)]; \
        }                                                                                       \
        __builtin_amdgcn_sched_barrier(0);          /* keep the prefetches ahead of this block's math */ \
        ring_block<S, SHIFT>(B, cvb[S & 1], acc);                                               \
    }
            LTS_RING_STEP(0)
            if (j + 1 >= nb_cur) break;
            LTS_RING_STEP(1)
            if (j + 2 >= nb_cur) break;
            LTS_RING_STEP(2)
            if (j + 3 >= nb_cur) break;
            LTS_RING_STEP(3)
#undef LTS_RING_STEP
        }
        done();
        if (!more) break;
    }
}

// Products of one table column with one cell column for RT = 8, two 8-value blocks in ping-pong: block j of cell
// ticks needs b_j = R[K0-8j .. +7] and b_{j+1} = R[K0-8j-8 .. -1]; the buffer holding b_j is refilled with b_{j+2}
// after block j, so each block loads only its 8 new values (no copies, no cross-lane traffic).
template <bool ALIGNED>
__device__ __forceinline__ void column_pingpong(const float *col, cfloat_ptr cc, int32_t nblk, float (&acc)[8]) {
    float X[8], Y[8], cv[kAC];
    load8<ALIGNED>(col, X);
    for (int32_t j = 0; j < nblk; j += 2) {
        load8<ALIGNED>(col - 8 * (j + 1), Y);
#pragma unroll
        for (int q = 0; q < kAC; ++q) cv[q] = cc[kAC * j + q];
#pragma unroll
        for (int q = 0; q < kAC; ++q)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int m = r - q + kAC - 1;
                acc[r] = fmaf(cv[q], m < 7 ? Y[m + 1] : X[m - 7], acc[r]);
            }
        if (j + 1 >= nblk) break;
        load8<ALIGNED>(col - 8 * (j + 2), X);
#pragma unroll
        for (int q = 0; q < kAC; ++q) cv[q] = cc[kAC * (j + 1) + q];
#pragma unroll
        for (int q = 0; q < kAC; ++q)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int m = r - q + kAC - 1;
                acc[r] = fmaf(cv[q], m < 7 ? X[m + 1] : Y[m - 7], acc[r]);
            }
    }
}


// One (segment, pixel) pair through the lane-exchange ring: the columns (u, v) of its charge box inside the pixel's
// reach, in row order.
__device__ __forceinline__ void pair_block_ring(const DevParams &P, const float *__restrict__ cc0, int32_t nv, int32_t nap,
                                                int32_t u0, int32_t v0, int32_t a0, const float *__restrict__ Rpad,
                                                int32_t ulo, int32_t uhi, int32_t vlo, int32_t vhi, int32_t uc,
                                                int32_t vc, int32_t nb, bool active, float (&acc)[8]) {
    const int32_t K0 = active ? nb - a0 + P.t_r - 1 + kPad : kPad;
    int32_t u = ulo, v = vlo;
    auto colp = [&](int32_t uu, int32_t vv) {
        return Rpad + (int64_t)(fold(uu - uc) * P.by + fold(vv - vc)) * P.col_len + K0;
    };
    auto cellp = [&](int32_t uu, int32_t vv) { return cc0 + ((int64_t)(uu - u0) * nv + (vv - v0)) * nap; };
    auto adv = [&](const float *&col, const float *&cc, int32_t &nblk) {
        if (++v > vhi) { v = vlo; ++u; }
        if (u > uhi) return false;
        col = colp(u, v);
        cc = cellp(u, v);
        return true;
    };
    column_stream<true, false>(colp(u, v), cellp(u, v), nap / kAC, adv, [] {}, acc);
}

// Signed induction of a pair's cells that falls outside the tick window [0, n_ticks), from FP64 prefix sums of
// the table columns.  Threads of the workgroup split the cells; returns this thread's part.
__device__ double pair_clipped(const DevParams &P, const float *cc0, int32_t nv, int32_t nap, int32_t na, int32_t u0,
                               int32_t v0, int32_t a0, const double *prefix, int32_t ulo, int32_t uhi, int32_t vlo,
                               int32_t vhi, int32_t uc, int32_t vc) {
    double acc = 0.0;
    const int32_t nuu = uhi - ulo + 1, nvv = vhi - vlo + 1;
    const int64_t tot = (int64_t)nuu * nvv * na;
    const int32_t T = P.t_r;
    for (int64_t c = threadIdx.x; c < tot; c += kWG) {
        const int32_t a = (int32_t)(c % na);
        const int32_t uv = (int32_t)(c / na);
        const int32_t v = vlo + uv % nvv, u = ulo + uv / nvv;
        const float cval = cc0[((int64_t)(u - u0) * nv + (v - v0)) * nap + a];
        if (cval == 0.0f) continue;
        const int32_t aa = a0 + a;
        const double *pf = prefix + (int64_t)(fold(u - uc) * P.by + fold(v - vc)) * (T + 1);
        const int32_t klo = min(max(T - 1 - aa, 0), T);                 // first kept table tick
        const int32_t khi = min(max(P.nticks + T - 1 - aa, 0), T);       // one past the last kept tick
        const double dropped = klo >= khi ? pf[T] : pf[klo] + (pf[T] - pf[khi]);
        acc += (double)cval * dropped;
    }
    return acc;
}

__device__ __forceinline__ double block_sum_double(double v, double *red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if (lane_id() == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < kWG / 64; ++i) t += red[i];
    return t;
}

// Sorted variant: one workgroup per active pixel (dynamic work queue); the pixel's segments in ascending id
// order; per-pair FP32 sums in registers added into a Kahan-compensated FP32 accumulator in LDS.
template <int RT, bool SHIFT>
__global__ __launch_bounds__(kWG) void k_induce_sorted(DevParams P, const SegInfo *__restrict__ si,
                                                       const float *__restrict__ cells, const float *__restrict__ Rpad,
                                                       const double *__restrict__ prefix,
                                                       const int64_t *__restrict__ slot_off,
                                                       const int32_t *__restrict__ pairs,
                                                       const int32_t *__restrict__ slot_gp,
                                                       const int32_t *__restrict__ order, float *__restrict__ wave,
                                                       DevHeader *H, double *report) {
    extern __shared__ float sm[];
    __shared__ int32_t s_slot;
    __shared__ double red[kWG / 64];
    const int NT = P.nticks;
    float *s_sum = sm, *s_cmp = sm + NT;
    const int tid = threadIdx.x;
    const int64_t n_slots = H->n_slots;
    for (;;) {
        if (tid == 0) s_slot = (int32_t)atomicAdd(&H->work[0], 1u);
        __syncthreads();
        if (s_slot >= n_slots) break;
        const int64_t slot = order ? order[s_slot] : s_slot;           // largest-first when an order is given
        for (int n = tid; n < NT; n += kWG) { s_sum[n] = 0.0f; s_cmp[n] = 0.0f; }
        const int32_t gp = slot_gp[slot];
        const int32_t e = gp / P.npx, p = gp - e * P.npx;
        const int32_t ix = p % P.nx, iy = p / P.nx;
        const int32_t uc = ix * P.nsub + P.nsub / 2, vc = iy * P.nsub + P.nsub / 2;
        const int64_t pb = slot_off[slot], pe = slot_off[slot + 1];
        double clip = 0.0;
        __syncthreads();
        for (int64_t q = pb; q < pe; ++q) {
            const int32_t s = __builtin_amdgcn_readfirstlane(pairs[q]);
            const SegInfo &g = si[s];
            const int32_t u0 = g.u0, v0 = g.v0, a0 = g.a0, nv = g.nv, nap = g.na_pad, na = g.na;
            const int32_t ulo = max(u0, uc - P.bx), uhi = min(u0 + g.nu - 1, uc + P.bx - 1);
            const int32_t vlo = max(v0, vc - P.by), vhi = min(v0 + nv - 1, vc + P.by - 1);
            if (ulo > uhi || vlo > vhi) continue;
            const float *cc0 = cells + g.cell_off;
            const int32_t wlo = a0 - (P.t_r - 1), whi = a0 + na - 1;
            if (wlo < 0 || whi >= NT)
                clip += pair_clipped(P, cc0, nv, nap, na, u0, v0, a0, prefix, ulo, uhi, vlo, vhi, uc, vc);
            const int32_t lo = max(wlo, 0), hi = min(whi, NT - 1);
            for (int32_t nb0 = lo; nb0 <= hi; nb0 += kWG * RT) {
                const int32_t nb = nb0 + tid * RT;
                float acc[RT];
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[r] = 0.0f;
                if constexpr (RT == 8 && SHIFT)
                    pair_block_ring(P, cc0, nv, nap, u0, v0, a0, Rpad, ulo, uhi, vlo, vhi, uc, vc, nb, nb <= hi, acc);
                else if (nb <= hi)
                    pair_block<RT>(P, cc0, nv, nap, u0, v0, a0, Rpad, ulo, uhi, vlo, vhi, uc, vc, nb, acc);
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const int32_t n = nb + r;
                    if (n <= hi) {                                       // Kahan: s_cmp holds the lost low part
                        const float y = acc[r] - s_cmp[n];
                        const float t = s_sum[n] + y;
                        s_cmp[n] = (t - s_sum[n]) - y;
                        s_sum[n] = t;
                    }
                }
            }
            __syncthreads();
        }
        float *wrow = wave + slot * NT;
        for (int n = tid; n < NT; n += kWG) wrow[n] = s_sum[n] - s_cmp[n];
        const double c = block_sum_double(clip, red);
        if (tid == 0 && c != 0.0) atomicAdd(&report[(int64_t)e * 5 + 3], c);
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------ matrix-core form
// By eq. (current), a pair's current is I[n] = sum_a sum_col c[col][a] R[col][n - c0 - a] with c0 = a0 - (T_R - 1):
// a column's cell ticks a against its table column, shifted by a.  Summing over the columns first gives the matrix
// product Z[a][tau] = sum_col c[col][a] R[col][tau] (cell ticks x table ticks, contracted over the pair's columns),
// and then I[n] = sum_a Z[a][n - c0 - a], a sum along the anti-diagonals of Z.  The product runs on 32x32x2 FP32
// MFMA instructions (lane l gives A[l % 32][l / 32] = c[col k0 + l / 32][a] and B[l / 32][l % 32] =
// R[col k0 + l / 32][tau]): both operands are rows of 32 consecutive floats, and there is no padding beyond
// rounding the cell ticks to 32 and the columns to 2.  Each 32 x 64 block of Z goes through LDS for the
// anti-diagonal sums, which each lane adds to its wavefront's output ticks in a fixed order.
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int32_t kBufferWord3 = 0x00020000;    // raw 32-bit buffer descriptor word 3 (gfx9 family)
constexpr int32_t kZT = 64;                     // table ticks per block of Z
constexpr int32_t kZA = 32;                     // cell ticks per block of Z
constexpr int32_t kZS = kZT + 1;                // LDS row stride of a Z block
constexpr int32_t kZOut = 512;                  // output ticks per wavefront and pass
constexpr int32_t kZLds = kZA * kZS + kZOut;    // floats of LDS per wavefront

// One pair's contribution to ticks n_w .. n_w + 511, added to Ow (this wavefront's 512 output sums in LDS).
__device__ __forceinline__ void pair_zgemm(const DevParams &P, const float *__restrict__ cc0, int32_t nu, int32_t nv,
                                           int32_t nap, int32_t na, int32_t u0, int32_t v0, int32_t a0,
                                           __amdgpu_buffer_rsrc_t rt, int32_t ulo, int32_t uhi, int32_t vlo,
                                           int32_t vhi, int32_t uc, int32_t vc, int32_t n_w, float *Zb, float *Ow) {
    const int l = lane_id();
    const int32_t c0 = a0 - (P.t_r - 1);
    const int32_t nvv = vhi - vlo + 1, ncol = (uhi - ulo + 1) * nvv;
    // the descriptors must be wavefront-uniform (scalar registers)
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)uniform_ptr(cc0), (short)0, __builtin_amdgcn_readfirstlane(nu * nv * nap * 4), kBufferWord3);
    for (int32_t ab = 0; ab < na; ab += kZA) {
        // table ticks that reach this wavefront's outputs from cell ticks ab .. ab + 31
        const int32_t t_first = max(n_w - c0 - ab - (kZA - 1), 0);
        const int32_t t_last = min(n_w + kZOut - 1 - c0 - ab, P.t_r - 1);
        for (int32_t t0 = t_first; t0 <= t_last; t0 += kZT) {
            floatx16 D[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) D[nt][r] = 0.0f;
            // 32x32x2: lane l gives A[l % 32][l / 32] (cell tick ab + l % 32 of column k0 + l / 32) and
            // B[l / 32][l % 32] (table tick t0 + 32 nt + l % 32 of that column)
            const int32_t i32 = l & 31, h = l >> 5;
            // this lane's columns: k = h, h + 2, ... in row-major (u, v) order; a step of 2 moves du rows and dv
            // columns, plus at most one wrap; colc (the column's cell offset) follows incrementally
            int32_t k = h, uu = ulo + h / nvv, vv = vlo + h % nvv;
            const int32_t du = 2 / nvv, dv = 2 - du * nvv;
            int32_t colc = ((uu - u0) * nv + (vv - v0)) * nap;
            const int32_t step_c = (du * nv + dv) * nap, wrap_c = (nv - nvv) * nap;
            auto fetch = [&](float &A, float (&B)[2]) {
                const bool valid = k < ncol;
                const int32_t fu = uu - uc, fv = vv - vc;
                const int32_t bin = __mul24(fu ^ (fu >> 31), P.by) + (fv ^ (fv >> 31));   // fold(), 24-bit products
                const int32_t colr = __mul24(bin, P.col_len) + kPad + t0 + i32;
                const int32_t a = ab + i32;
                const bool in = valid && a < na;
                const float cv = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rc, 4 * (in ? colc + a : 0), 0, 0));
                A = in ? cv : 0.0f;
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    B[nt] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(rt, 4 * (valid ? colr + 32 * nt : 0), 0, 0));
                k += 2;
                vv += dv;
                uu += du;
                colc += step_c;
                const bool wrap = vv > vhi;
                vv = wrap ? vv - nvv : vv;
                uu = wrap ? uu + 1 : uu;
                colc = wrap ? colc + wrap_c : colc;
            };
            auto step = [&](float A, const float (&B)[2]) {
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) D[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(A, B[nt], D[nt], 0, 0, 0);
            };
            const int32_t ks2 = (ncol + 1) >> 1;
            float A0, B0[2], A1, B1[2], A2, B2[2];
            fetch(A0, B0);
            fetch(A1, B1);
            for (int32_t st = 0; st < ks2; st += 3) {
                fetch(A2, B2);
                __builtin_amdgcn_sched_barrier(0);
                step(A0, B0);
                __builtin_amdgcn_sched_barrier(0);
                fetch(A0, B0);
                __builtin_amdgcn_sched_barrier(0);
                step(A1, B1);
                __builtin_amdgcn_sched_barrier(0);
                fetch(A1, B1);
                __builtin_amdgcn_sched_barrier(0);
                step(A2, B2);
                __builtin_amdgcn_sched_barrier(0);
            }
            // Z block to LDS: 32x32 layout, lane l register r holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) Zb[(8 * (r >> 2) + 4 * h + (r & 3)) * kZS + 32 * nt + i32] = D[nt][r];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // anti-diagonal d = t + a' holds the block's part of tick n = t0 + c0 + ab + d
            // (a fixed trip count with clamped indices, so all 32 LDS reads of a diagonal are issued together)
#pragma unroll
            for (int32_t half = 0; half < 2; ++half) {
                const int32_t d = l + 64 * half;
                const int32_t o = t0 + c0 + ab + d - n_w;
                float sum = 0.0f;
#pragma unroll
                for (int32_t ap = 0; ap < kZA; ++ap) {
                    const int32_t t = d - ap;
                    const float z = Zb[ap * kZS + min(max(t, 0), kZT - 1)];
                    sum += (t >= 0 && t < kZT) ? z : 0.0f;
                }
                if (d < kZT + kZA - 1 && o >= 0 && o < kZOut) Ow[o] += sum;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

// Per-pair induction of the sorted variant on the matrix cores: the same pixel-slot work queue, pair order and
// Kahan accumulation in LDS as k_induce_sorted; wavefront w of the workgroup owns ticks nb0 + 512 w .. + 511 of
// each 2048-tick pass over a pair's window, lane l of it ticks + 8 l .. + 7.
__global__ __launch_bounds__(kWG) void k_induce_mfma(DevParams P, const SegInfo *__restrict__ si,
                                                     const float *__restrict__ cells, const float *__restrict__ Rpad,
                                                     const double *__restrict__ prefix,
                                                     const int64_t *__restrict__ slot_off,
                                                     const int32_t *__restrict__ pairs,
                                                     const int32_t *__restrict__ slot_gp, float *__restrict__ wave,
                                                     DevHeader *H, double *report) {
    extern __shared__ float sm[];
    __shared__ int32_t s_slot;
    __shared__ double red[kWG / 64];
    const int NT = P.nticks;
    float *s_sum = sm, *s_cmp = sm + NT;
    const int tid = threadIdx.x;
    const int32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;   // wavefront index (uniform)
    float *Zb = sm + 2 * NT + wv * kZLds, *Ow = Zb + kZA * kZS;
    const int64_t n_slots = H->n_slots;
    const __amdgpu_buffer_rsrc_t rt =
        __builtin_amdgcn_make_buffer_rsrc((void *)Rpad, (short)0, P.bx * P.by * P.col_len * 4, kBufferWord3);
    for (int o = l; o < kZOut; o += 64) Ow[o] = 0.0f;
    for (;;) {
        if (tid == 0) s_slot = (int32_t)atomicAdd(&H->work[0], 1u);
        __syncthreads();
        const int64_t slot = s_slot;
        if (slot >= n_slots) break;
        for (int n = tid; n < NT; n += kWG) { s_sum[n] = 0.0f; s_cmp[n] = 0.0f; }
        const int32_t gp = slot_gp[slot];
        const int32_t e = gp / P.npx, p = gp - e * P.npx;
        const int32_t ix = p % P.nx, iy = p / P.nx;
        const int32_t uc = ix * P.nsub + P.nsub / 2, vc = iy * P.nsub + P.nsub / 2;
        const int64_t pb = slot_off[slot], pe = slot_off[slot + 1];
        double clip = 0.0;
        __syncthreads();
        for (int64_t qq = pb; qq < pe; ++qq) {
            const int32_t s = __builtin_amdgcn_readfirstlane(pairs[qq]);
            const SegInfo &g = si[s];
            const int32_t u0 = g.u0, v0 = g.v0, a0 = g.a0, nv = g.nv, nap = g.na_pad, na = g.na;
            const int32_t ulo = max(u0, uc - P.bx), uhi = min(u0 + g.nu - 1, uc + P.bx - 1);
            const int32_t vlo = max(v0, vc - P.by), vhi = min(v0 + nv - 1, vc + P.by - 1);
            if (ulo > uhi || vlo > vhi) continue;
            const float *cc0 = cells + g.cell_off;
            const int32_t wlo = a0 - (P.t_r - 1), whi = a0 + na - 1;
            if (wlo < 0 || whi >= NT)
                clip += pair_clipped(P, cc0, nv, nap, na, u0, v0, a0, prefix, ulo, uhi, vlo, vhi, uc, vc);
            const int32_t lo = max(wlo, 0), hi = min(whi, NT - 1);
            for (int32_t nb0 = lo; nb0 <= hi; nb0 += 4 * kZOut) {
                const int32_t n_w = nb0 + kZOut * wv;
                if (n_w <= hi) {
                    pair_zgemm(P, cc0, g.nu, nv, nap, na, u0, v0, a0, rt, ulo, uhi, vlo, vhi, uc, vc, n_w, Zb, Ow);
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const int32_t o = 8 * l + r, n = n_w + o;
                        const float x = Ow[o];
                        Ow[o] = 0.0f;
                        if (n <= hi) {                                   // Kahan: s_cmp holds the lost low part
                            const float y = x - s_cmp[n];
                            const float z = s_sum[n] + y;
                            s_cmp[n] = (z - s_sum[n]) - y;
                            s_sum[n] = z;
                        }
                    }
                }
            }
            __syncthreads();
        }
        float *wrow = wave + slot * NT;
        for (int n = tid; n < NT; n += kWG) wrow[n] = s_sum[n] - s_cmp[n];
        const double c = block_sum_double(clip, red);
        if (tid == 0 && c != 0.0) atomicAdd(&report[(int64_t)e * 5 + 3], c);
        __syncthreads();
    }
}

// Atomic variant: one workgroup per segment (dynamic work queue); its pairs in pixel order; FP32 atomics.
template <int RT>
__global__ __launch_bounds__(kWG) void k_induce_atomic(DevParams P, const SegInfo *__restrict__ si, int64_t n_seg,
                                                       const float *__restrict__ cells, const float *__restrict__ Rpad,
                                                       const double *__restrict__ prefix,
                                                       const int32_t *__restrict__ pix_slot, float *wave, DevHeader *H,
                                                       double *report) {
    __shared__ int32_t s_seg;
    __shared__ double red[kWG / 64];
    const int NT = P.nticks;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s_seg = (int32_t)atomicAdd(&H->work[1], 1u);
        __syncthreads();
        const int64_t s = s_seg;
        __syncthreads();
        if (s >= n_seg) break;
        const SegInfo &g = si[s];
        if (g.n_pairs == 0) continue;
        const int32_t u0 = g.u0, v0 = g.v0, a0 = g.a0, nv = g.nv, nap = g.na_pad, na = g.na;
        const float *cc0 = cells + g.cell_off;
        const int32_t wlo = a0 - (P.t_r - 1), whi = a0 + na - 1;
        const int32_t lo = max(wlo, 0), hi = min(whi, NT - 1);
        double clip = 0.0;
        for (int32_t iy = g.iy0; iy <= g.iy1; ++iy)
            for (int32_t ix = g.ix0; ix <= g.ix1; ++ix) {
                const int32_t uc = ix * P.nsub + P.nsub / 2, vc = iy * P.nsub + P.nsub / 2;
                const int32_t ulo = max(u0, uc - P.bx), uhi = min(u0 + g.nu - 1, uc + P.bx - 1);
                const int32_t vlo = max(v0, vc - P.by), vhi = min(v0 + nv - 1, vc + P.by - 1);
                if (ulo > uhi || vlo > vhi) continue;
                const int64_t slot = pix_slot[(int64_t)g.event * P.npx + iy * P.nx + ix];
                float *wrow = wave + slot * NT;
                if (wlo < 0 || whi >= NT)
                    clip += pair_clipped(P, cc0, nv, nap, na, u0, v0, a0, prefix, ulo, uhi, vlo, vhi, uc, vc);
                for (int32_t nb0 = lo; nb0 <= hi; nb0 += kWG * RT) {
                    const int32_t nb = nb0 + tid * RT;
                    if (nb > hi) continue;
                    float acc[RT];
#pragma unroll
                    for (int r = 0; r < RT; ++r) acc[r] = 0.0f;
                    pair_block<RT>(P, cc0, nv, nap, u0, v0, a0, Rpad, ulo, uhi, vlo, vhi, uc, vc, nb, acc);
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        if (nb + r <= hi && acc[r] != 0.0f) atomicAdd(&wrow[nb + r], acc[r]);
                }
            }
        const double c = block_sum_double(clip, red);
        if (tid == 0 && c != 0.0) atomicAdd(&report[(int64_t)g.event * 5 + 3], c);
    }
}

// XCD-sliced sorted variant: workgroup b handles pixel slot slot0 + b / NS and slice x = b % NS of the
// mirror-folded x-bin index (table bins i in [x*bx/NS, (x+1)*bx/NS)).  Workgroups are dispatched to the 8 XCDs
// round-robin by id, so each XCD's L2 only ever holds its slice of the field-response table.  The pixel's per-slice
// waveform (Kahan over its segments in ascending order) goes to part[x][slot - slot0][tick]; k_sum_slices adds the
// slices in a fixed order.  Deterministic and batch-invariant like the unsliced kernel.
template <int RT>
__global__ __launch_bounds__(kWG) void k_induce_slices(DevParams P, int32_t NS, int64_t slot0, int64_t chunk,
                                                       const SegInfo *__restrict__ si, const float *__restrict__ cells,
                                                       const float *__restrict__ Rpad, const double *__restrict__ prefix,
                                                       const int64_t *__restrict__ slot_off,
                                                       const int32_t *__restrict__ pairs,
                                                       const int32_t *__restrict__ slot_gp, float *__restrict__ part,
                                                       const DevHeader *H, double *report) {
    extern __shared__ float sm[];
    __shared__ double red[kWG / 64];
    const int NT = P.nticks;
    float *s_sum = sm, *s_cmp = sm + NT;
    const int tid = threadIdx.x;
    const int64_t local = blockIdx.x / NS;
    const int32_t x = blockIdx.x - (int32_t)local * NS;
    const int64_t slot = slot0 + local;
    if (slot >= H->n_slots) return;
    const int32_t ilo = x * P.bx / NS, ihi = (x + 1) * P.bx / NS - 1;
    for (int n = tid; n < NT; n += kWG) { s_sum[n] = 0.0f; s_cmp[n] = 0.0f; }
    const int32_t gp = slot_gp[slot];
    const int32_t e = gp / P.npx, p = gp - e * P.npx;
    const int32_t ix = p % P.nx, iy = p / P.nx;
    const int32_t uc = ix * P.nsub + P.nsub / 2, vc = iy * P.nsub + P.nsub / 2;
    const int64_t pb = slot_off[slot], pe = slot_off[slot + 1];
    double clip = 0.0;
    __syncthreads();
    if (ilo <= ihi) {
        for (int64_t q = pb; q < pe; ++q) {
            const int32_t s = __builtin_amdgcn_readfirstlane(pairs[q]);
            const SegInfo &g = si[s];
            const int32_t u0 = g.u0, v0 = g.v0, a0 = g.a0, nv = g.nv, nap = g.na_pad, na = g.na;
            const int32_t ue = u0 + g.nu - 1;
            // fold(u - uc) in [ilo, ihi]: u - uc in [ilo, ihi] or in [-ihi-1, -ilo-1]
            const int32_t ua0 = max(u0, uc + ilo), ua1 = min(ue, uc + ihi);
            const int32_t ub0 = max(u0, uc - ihi - 1), ub1 = min(ue, uc - ilo - 1);
            const int32_t vlo = max(v0, vc - P.by), vhi = min(v0 + nv - 1, vc + P.by - 1);
            if ((ua0 > ua1 && ub0 > ub1) || vlo > vhi) continue;
            const float *cc0 = cells + g.cell_off;
            const int32_t wlo = a0 - (P.t_r - 1), whi = a0 + na - 1;
            if (wlo < 0 || whi >= NT) {
                if (ua0 <= ua1) clip += pair_clipped(P, cc0, nv, nap, na, u0, v0, a0, prefix, ua0, ua1, vlo, vhi, uc, vc);
                if (ub0 <= ub1) clip += pair_clipped(P, cc0, nv, nap, na, u0, v0, a0, prefix, ub0, ub1, vlo, vhi, uc, vc);
            }
            const int32_t lo = max(wlo, 0), hi = min(whi, NT - 1);
            for (int32_t nb0 = lo; nb0 <= hi; nb0 += kWG * RT) {
                const int32_t nb = nb0 + tid * RT;
                float acc[RT];
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[r] = 0.0f;
                if (nb <= hi) {
                    if (ua0 <= ua1) pair_block<RT>(P, cc0, nv, nap, u0, v0, a0, Rpad, ua0, ua1, vlo, vhi, uc, vc, nb, acc);
                    if (ub0 <= ub1) pair_block<RT>(P, cc0, nv, nap, u0, v0, a0, Rpad, ub0, ub1, vlo, vhi, uc, vc, nb, acc);
                }
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const int32_t n = nb + r;
                    if (n <= hi) {
                        const float y = acc[r] - s_cmp[n];
                        const float t = s_sum[n] + y;
                        s_cmp[n] = (t - s_sum[n]) - y;
                        s_sum[n] = t;
                    }
                }
            }
            __syncthreads();
        }
    }
    float *prow = part + ((int64_t)x * chunk + local) * NT;
    for (int n = tid; n < NT; n += kWG) prow[n] = s_sum[n] - s_cmp[n];
    const double c = block_sum_double(clip, red);
    if (tid == 0 && c != 0.0) atomicAdd(&report[(int64_t)e * 5 + 3], c);
}

// current[slot][n] = sum over slices x = 0..NS-1 (in that order, Kahan) of part[x][slot - slot0][n].
__global__ __launch_bounds__(kWG) void k_sum_slices(int32_t NS, int32_t NT, int64_t slot0, int64_t chunk,
                                                    const float *__restrict__ part, float *__restrict__ wave,
                                                    const DevHeader *H) {
    const int64_t n_slots = H->n_slots;
    const int64_t nrows = min(chunk, n_slots - slot0);
    const int64_t total = nrows * NT;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < total; i += (int64_t)gridDim.x * kWG) {
        float sum = 0.0f, cmp = 0.0f;
        for (int32_t x = 0; x < NS; ++x) {
            const float y = part[(int64_t)x * chunk * NT + i] - cmp;
            const float t = sum + y;
            cmp = (t - sum) - y;
            sum = t;
        }
        wave[slot0 * NT + i] = sum - cmp;
    }
}

// Largest-first order of the active pixels for the per-pair induction.  A workgroup owns one pixel at a time and
// takes the next from a counter, so pixels of very unequal work taken in pixel order leave the chip idle at the end
// while the last heavy pixels finish; taking them largest first (bucketed by the logarithm of their work, 16 buckets
// per octave) keeps the tail short.  Work of a pixel = sum over its pairs of the charge-box columns in its reach times
// the cell-tick blocks.  The order changes only which workgroup computes a pixel, not any sum.
__global__ void k_slot_work(DevParams P, const SegInfo *__restrict__ si, const int64_t *__restrict__ slot_off,
                            const int32_t *__restrict__ pairs, const int32_t *__restrict__ slot_gp, int64_t n_slots,
                            int32_t *__restrict__ bucket, int32_t *__restrict__ hist) {
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= n_slots) return;
    const int32_t gp = slot_gp[slot];
    const int32_t p = gp % P.npx;
    const int32_t uc = (p % P.nx) * P.nsub + P.nsub / 2, vc = (p / P.nx) * P.nsub + P.nsub / 2;
    double work = 0.0;
    for (int64_t q = slot_off[slot]; q < slot_off[slot + 1]; ++q) {
        const SegInfo &g = si[pairs[q]];
        const int32_t cu = min(g.u0 + g.nu, uc + P.bx) - max(g.u0, uc - P.bx);
        const int32_t cv = min(g.v0 + g.nv, vc + P.by) - max(g.v0, vc - P.by);
        if (cu > 0 && cv > 0) work += (double)cu * cv * (g.na_pad / kAC);
    }
    const int32_t lg = work >= 1.0 ? (int32_t)(16.0 * log2(work)) : 0;
    const int32_t b = kOrderBuckets - 1 - min(lg, kOrderBuckets - 1);          // descending work
    bucket[slot] = b;
    atomicAdd(&hist[b], 1);
}

// bucket offsets (exclusive scan of the histogram) into the cursors
__global__ void k_order_offsets(int32_t *__restrict__ hist, int32_t *__restrict__ cursor) {
    __shared__ int32_t s[kOrderBuckets];
    for (int i = threadIdx.x; i < kOrderBuckets; i += blockDim.x) s[i] = hist[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t run = 0;
        for (int i = 0; i < kOrderBuckets; ++i) {
            const int32_t c = s[i];
            s[i] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kOrderBuckets; i += blockDim.x) cursor[i] = s[i];
}

__global__ void k_order_scatter(const int32_t *__restrict__ bucket, int64_t n_slots, int32_t *__restrict__ cursor,
                                int32_t *__restrict__ order) {
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= n_slots) return;
    order[atomicAdd(&cursor[bucket[slot]], 1)] = (int32_t)slot;
}

// w.order holds [order: n_slots][bucket: n_slots][hist: kOrderBuckets][cursor: kOrderBuckets]
static void launch_slot_order(const DevParams &P, const Work &w, int64_t n_slots, hipStream_t st) {
    int32_t *order = w.order, *bucket = order + n_slots, *hist = bucket + n_slots, *cursor = hist + kOrderBuckets;
    launch_zero(hist, (int64_t)sizeof(int32_t) * kOrderBuckets, st);
    const unsigned g = (unsigned)((n_slots + kWG - 1) / kWG);
    k_slot_work<<<g, kWG, 0, st>>>(P, w.si, w.slot_off, w.pairs, w.slot_gp, n_slots, bucket, hist);
    k_order_offsets<<<1, kWG, 0, st>>>(hist, cursor);
    k_order_scatter<<<g, kWG, 0, st>>>(bucket, n_slots, cursor, order);
}

template <int RT>
static void induce_slices_rt(const DevParams &P, const Work &w, const Table &T, float *wave, int64_t n_slots, int32_t NS,
                             float *part, int64_t chunk, hipStream_t st) {
    const size_t lds = (size_t)2 * P.nticks * sizeof(float);
    for (int64_t s0 = 0; s0 < n_slots; s0 += chunk) {
        const int64_t rows = n_slots - s0 < chunk ? n_slots - s0 : chunk;
        k_induce_slices<RT><<<(unsigned)(rows * NS), kWG, lds, st>>>(P, NS, s0, chunk, w.si, w.cells, T.Rpad, T.prefix,
                                                                   w.slot_off, w.pairs, w.slot_gp, part, w.hdr, w.report);
        int64_t g = (rows * P.nticks + kWG - 1) / kWG;
        if (g > 16384) g = 16384;
        k_sum_slices<<<(unsigned)g, kWG, 0, st>>>(NS, P.nticks, s0, chunk, part, wave, w.hdr);
    }
}

// Ticks per thread of the induction: the smallest of 1, 2, 4, 8 whose 256-thread tile covers a pair's window
// (table length + a typical charge-box extent), unless forced.
static int32_t pick_rt(const DevParams &P, int32_t forced) {
    if (forced == 1 || forced == 2 || forced == 4 || forced == 8) return forced;
    const int32_t win = P.t_r + 32;
    return win <= kWG ? 1 : win <= 2 * kWG ? 2 : win <= 4 * kWG ? 4 : 8;
}

void launch_induce_slices(const DevParams &P, const Work &w, const Table &T, float *wave, int64_t n_slots, int32_t NS,
                          float *part, int64_t chunk, int32_t rt, hipStream_t st) {
    if (n_slots <= 0) return;
    switch (pick_rt(P, rt)) {
        case 1: induce_slices_rt<1>(P, w, T, wave, n_slots, NS, part, chunk, st); break;
        case 2: induce_slices_rt<2>(P, w, T, wave, n_slots, NS, part, chunk, st); break;
        case 4: induce_slices_rt<4>(P, w, T, wave, n_slots, NS, part, chunk, st); break;
        default: induce_slices_rt<8>(P, w, T, wave, n_slots, NS, part, chunk, st); break;
    }
}

template <int RT, bool SHIFT>
static void induce_rt(const DevParams &P, const Work &w, const Table &T, float *wave, int mode, int64_t n_slots,
                      hipStream_t st) {
    const int64_t cap = 2048;
    if (mode == 0) {
        int64_t g = n_slots < 1 ? 1 : (n_slots > cap ? cap : n_slots);
        size_t lds = (size_t)2 * P.nticks * sizeof(float);
        if (w.order && n_slots > 0) launch_slot_order(P, w, n_slots, st);
        k_induce_sorted<RT, SHIFT><<<(unsigned)g, kWG, lds, st>>>(P, w.si, w.cells, T.Rpad, T.prefix, w.slot_off, w.pairs,
                                                          w.slot_gp, n_slots > 0 ? w.order : nullptr, wave, w.hdr,
                                                          w.report);
    } else {
        int64_t g = w.n_seg < 1 ? 1 : (w.n_seg > cap ? cap : w.n_seg);
        k_induce_atomic<RT><<<(unsigned)g, kWG, 0, st>>>(P, w.si, w.n_seg, w.cells, T.Rpad, T.prefix, w.pix_slot, wave,
                                                        w.hdr, w.report);
    }
}

void launch_induce_mfma(const DevParams &P, const Work &w, const Table &T, float *wave, int64_t n_slots,
                        hipStream_t st) {
    const int64_t cap = 2048;
    const int64_t g = n_slots < 1 ? 1 : (n_slots > cap ? cap : n_slots);
    const size_t lds = ((size_t)2 * P.nticks + (size_t)(kWG / 64) * kZLds) * sizeof(float);
    k_induce_mfma<<<(unsigned)g, kWG, lds, st>>>(P, w.si, w.cells, T.Rpad, T.prefix, w.slot_off, w.pairs, w.slot_gp,
                                                  wave, w.hdr, w.report);
}

void launch_induce(const DevParams &P, const Work &w, const Table &T, float *wave, int mode, int64_t n_slots, int32_t rt,
                   bool shift, hipStream_t st) {
    switch (pick_rt(P, rt)) {
        case 1: induce_rt<1, false>(P, w, T, wave, mode, n_slots, st); break;
        case 2: induce_rt<2, false>(P, w, T, wave, mode, n_slots, st); break;
        case 4: induce_rt<4, false>(P, w, T, wave, mode, n_slots, st); break;
        default:
            if (shift) induce_rt<8, true>(P, w, T, wave, mode, n_slots, st);
            else induce_rt<8, false>(P, w, T, wave, mode, n_slots, st);
            break;
    }
}

// ================================================================================================= stage hooks
// The paper's own data flow (Sec. 3.3.2, 3.4): the induced current of every (segment, pixel) pair is materialised as
// its own waveform, then the waveforms of each pixel are summed.  The fused kernels above never write these; the
// hooks below do, for tests and for comparison with the fused path.

// Pair list in stored order (pixel-major, ascending segment within a pixel): segment index and tile pixel id.
__global__ __launch_bounds__(kWG) void k_pair_list(DevParams P, const int64_t *__restrict__ slot_off,
                                                   const int32_t *__restrict__ pairs,
                                                   const int32_t *__restrict__ slot_gp, const DevHeader *H,
                                                   int32_t *pair_seg, int32_t *pair_pix) {
    for (int64_t slot = blockIdx.x; slot < H->n_slots; slot += gridDim.x) {
        const int32_t gp = slot_gp[slot];
        const int32_t p = gp - (gp / P.npx) * P.npx;
        for (int64_t q = slot_off[slot] + threadIdx.x; q < slot_off[slot + 1]; q += kWG) {
            if (pair_seg) pair_seg[q] = pairs[q];
            if (pair_pix) pair_pix[q] = p;
        }
    }
}

void launch_pair_list(const DevParams &P, const Work &w, int64_t n_slots, int32_t *pair_seg, int32_t *pair_pix,
                      hipStream_t st) {
    if (n_slots <= 0) return;
    const unsigned g = (unsigned)std::min<int64_t>(n_slots, 65536);
    k_pair_list<<<g, kWG, 0, st>>>(P, w.slot_off, w.pairs, w.slot_gp, w.hdr, pair_seg, pair_pix);
}

// Per-pixel sum of pair waveforms grouped by pixel: head[q] = 1 where a run of equal pixel ids starts (q < n),
// head[n] = 0; a pixel id below its predecessor sets ST_INVALID (the pairs are not grouped in ascending order).
__global__ void k_run_heads(const int32_t *__restrict__ pix, int64_t n, int64_t *head, DevHeader *H) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q > n) return;
    if (q == n) { head[q] = 0; return; }
    const int32_t prev = q > 0 ? pix[q - 1] : -1;
    head[q] = pix[q] != prev ? 1 : 0;
    if (pix[q] < prev) atomicOr(&H->status, ST_INVALID);
}

// After the exclusive scan of head: start[k] = first pair of run k, start[n_runs] = n; pixel ids of the runs.
__global__ void k_run_starts(const int32_t *__restrict__ pix, int64_t n, const int64_t *__restrict__ idx,
                             int64_t *start, int32_t *pixel_out, int64_t cap) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int64_t k = idx[q];
    if (q == 0 || pix[q] != pix[q - 1]) {
        start[k] = q;
        if (k < cap) pixel_out[k] = pix[q];
    }
    if (q == n - 1) start[idx[n]] = n;
}

// current[k][t] = sum over the run's pairs, in stored order, of their waveforms at tick t (Kahan summation).
__global__ __launch_bounds__(kWG) void k_reduce_runs(const float *__restrict__ pair_current,
                                                     const int64_t *__restrict__ start, int32_t NT, float *current) {
    const int64_t k = blockIdx.x;
    const int32_t t = blockIdx.y * kWG + threadIdx.x;
    if (t >= NT) return;
    float sum = 0.0f, cmp = 0.0f;
    for (int64_t q = start[k]; q < start[k + 1]; ++q) {
        const float y = pair_current[q * NT + t] - cmp;
        const float z = sum + y;
        cmp = (z - sum) - y;
        sum = z;
    }
    current[k * NT + t] = sum - cmp;
}

void launch_run_heads(const int32_t *pix, int64_t n, int64_t *head, DevHeader *H, hipStream_t st) {
    k_run_heads<<<(unsigned)((n + 1 + kWG - 1) / kWG), kWG, 0, st>>>(pix, n, head, H);
}

void launch_run_starts(const int32_t *pix, int64_t n, const int64_t *idx, int64_t *start, int32_t *pixel_out,
                       int64_t cap, hipStream_t st) {
    if (n > 0) k_run_starts<<<(unsigned)((n + kWG - 1) / kWG), kWG, 0, st>>>(pix, n, idx, start, pixel_out, cap);
}

void launch_reduce_runs(const float *pair_current, const int64_t *start, int64_t n_runs, int32_t NT, float *current,
                        hipStream_t st) {
    if (n_runs <= 0 || NT <= 0) return;
    const dim3 g((unsigned)n_runs, (unsigned)((NT + kWG - 1) / kWG));
    k_reduce_runs<<<g, kWG, 0, st>>>(pair_current, start, NT, current);
}

// ================================================================================================= summed induction
// Sum-then-convolve: by linearity of eq. (current), the current on pixel p is the time convolution of each absolute
// sub-pixel column's charge, summed over all segments, with that column's folded table column.  The columns are
// summed once per event (fixed segment order, Kahan) and cut into pieces of at most kPieceTicks ticks; each piece is
// a 1 x 1 x L charge box, and every active pixel's list of pieces in its reach replaces its pair list, so the
// sorted induction kernel runs unchanged on the summed data.

// Sort key of a segment in a column's list: first tick (signed, order-preserving bias) above the segment index.
__device__ __forceinline__ uint64_t sum_key(int32_t a0, int32_t s) {
    return ((uint64_t)((uint32_t)a0 ^ 0x80000000u) << 32) | (uint32_t)s;
}
__device__ __forceinline__ int32_t key_seg(uint64_t k) { return (int32_t)(uint32_t)k; }

// Segments per column.  A segment's reachable columns form a rectangle of the event's column grid, so the counts
// come from a two-dimensional difference array: per segment +1 at the rectangle's first corner and -1 / -1 / +1 at the
// corners one past it (those outside the grid dropped), then prefix sums along each row and down each grid column.
__global__ void k_sum_ranges(DevParams P, const SegInfo *si, int64_t n_seg, SumWork sw) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_seg) return;
    const SegInfo &g = si[s];
    if (g.flags & (SEG_INVALID | SEG_TOO_LONG)) return;
    sw.segc[s] = SumSeg{g.a0, g.na, g.u0, g.v0, g.nv, g.na_pad, g.cell_off};
    const int32_t u_a = max(g.u0, sw.UL), u_b = min(g.u0 + g.nu - 1, sw.UL + sw.CU - 1);
    const int32_t v_a = max(g.v0, sw.VL), v_b = min(g.v0 + g.nv - 1, sw.VL + sw.CV - 1);
    if (u_a > u_b || v_a > v_b) return;
    unsigned long long *cnt = (unsigned long long *)sw.col_seg_off + (int64_t)g.event * sw.CU * sw.CV;
    const int32_t ua = u_a - sw.UL, ub = u_b - sw.UL + 1, va = v_a - sw.VL, vb = v_b - sw.VL + 1;
    atomicAdd(&cnt[(int64_t)ua * sw.CV + va], 1ull);
    if (vb < sw.CV) atomicAdd(&cnt[(int64_t)ua * sw.CV + vb], ~0ull);          // -1
    if (ub < sw.CU) {
        atomicAdd(&cnt[(int64_t)ub * sw.CV + va], ~0ull);
        if (vb < sw.CV) atomicAdd(&cnt[(int64_t)ub * sw.CV + vb], 1ull);
    }
}

void launch_sum_ranges(const DevParams &P, const Work &w, const SumWork &sw, hipStream_t st) {
    if (w.n_seg > 0) k_sum_ranges<<<(unsigned)((w.n_seg + kWG - 1) / kWG), kWG, 0, st>>>(P, w.si, w.n_seg, sw);
    const int64_t n_ev = sw.n_cols / ((int64_t)sw.CU * sw.CV);
    const int64_t rows = n_ev * sw.CU;
    if (rows > 0) {
        k_prefix_rows<<<(unsigned)((rows + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>(sw.col_seg_off, rows, sw.CV);
        launch_prefix_cols(sw.col_seg_off, (int32_t)n_ev, sw.CU, sw.CV, st);
    }
}

// per segment (one wavefront, lanes over its reachable columns: every atomic instruction meets distinct cursors)
__global__ __launch_bounds__(kWG) void k_sum_fill(DevParams P, const SegInfo *si, int64_t n_seg, SumWork sw) {
    const int lane = threadIdx.x & 63;
    const int64_t s = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (s >= n_seg) return;
    const SegInfo &g = si[s];
    if (g.flags & (SEG_INVALID | SEG_TOO_LONG)) return;
    const int32_t u_a = max(g.u0, sw.UL), u_b = min(g.u0 + g.nu - 1, sw.UL + sw.CU - 1);
    const int32_t v_a = max(g.v0, sw.VL), v_b = min(g.v0 + g.nv - 1, sw.VL + sw.CV - 1);
    if (u_a > u_b || v_a > v_b) return;
    const int32_t wv = v_b - v_a + 1, nc = (u_b - u_a + 1) * wv;
    const int64_t base = (int64_t)g.event * sw.CU * sw.CV + (int64_t)(u_a - sw.UL) * sw.CV + (v_a - sw.VL);
    const uint64_t key = sum_key(g.a0, (int32_t)s);
    for (int32_t i = lane; i < nc; i += 64) {
        const int32_t du = i / wv;
        const int64_t c = base + (int64_t)du * sw.CV + (i - du * wv);
        sw.col_tmp[sw.col_seg_off[c] + atomicAdd(&sw.col_cursor[c], 1)] = key;
    }
}

// A column's charge is cut where none of its segments has charge for more than kSumGap ticks: the zero ticks of
// such a gap would otherwise be convolved with the whole table column.  A new piece costs less than ~16 zero ticks.
constexpr int32_t kSumGap = 16;

// Pieces of kPieceTicks ticks of an interval of L ticks, and their summed-charge length (the last one padded to kAC).
__device__ inline void sum_interval_size(int32_t L, int64_t &np, int64_t &ns) {
    np = (L + kPieceTicks - 1) / kPieceTicks;
    const int32_t last = L - (int32_t)(np - 1) * kPieceTicks;
    ns = (np - 1) * kPieceTicks + (last + kAC - 1) / kAC * kAC;
}

// 64-bit value of lane j (j wave-uniform).
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int j) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j);
    return ((uint64_t)hi << 32) | lo;
}

// per column: sort its segment list by key (first tick, segment index) into col_seg, then count the pieces and the
// padded summed-charge length of its merged tick intervals.  For the 512-tick summed induction kernel every
// interval's first tick is moved down to the residue it chooses (it makes every lane's table offsets aligned there);
// the matrix kernel takes intervals as they are (align_res < 0).  The order depends only on the segments' charge
// boxes and their order within the event, so the sums are the same in a batch and alone.  The columns with segments
// are listed first (k_sum_active); persistent wavefronts take them one at a time.  Sort by ranks (a key's place is
// the number of smaller keys; keys are unique): lane i holds key i of a 64-key chunk and compares it with every key
// of the list, taken chunk by chunk from the lanes' registers.  Intervals from the sorted list, 64 entries at a time:
// an entry starts an interval when its first tick lies more than kSumGap ticks beyond the last tick of every earlier
// entry (a prefix maximum over the lanes), and the interval before it ends at that maximum.
__device__ __forceinline__ int32_t key_a0(uint64_t k) { return (int32_t)((uint32_t)(k >> 32) ^ 0x80000000u); }
__device__ __forceinline__ void interval_count(int32_t lo, int32_t hi, int32_t res, int64_t &np, int64_t &ns) {
    if (res >= 0) lo -= ((lo - res) % 8 + 8) % 8;
    int64_t n, m;
    sum_interval_size(hi - lo + 1, n, m);
    np += n;
    ns += m;
}
// columns with segments, listed in any order (one atomic per wavefront of kActiveSpan columns); the others get zero
// counts
constexpr int kActiveSpan = 512;
__global__ __launch_bounds__(kWG) void k_sum_active(SumWork sw) {
    const int lane = threadIdx.x & 63;
    const int64_t c0 = ((int64_t)blockIdx.x * (kWG / 64) + (threadIdx.x >> 6)) * kActiveSpan;
    uint64_t act[kActiveSpan / 64];
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < kActiveSpan / 64; ++i) {
        const int64_t c = c0 + 64 * i + lane;
        bool has = false;
        if (c < sw.n_cols) {
            has = sw.col_seg_off[c + 1] > sw.col_seg_off[c];
            if (!has) {
                sw.piece_off[c] = 0;
                sw.s_off[c] = 0;
            }
        }
        act[i] = __ballot(has);
        total += (uint32_t)__builtin_popcountll(act[i]);
    }
    uint32_t base = 0;
    if (total && lane == 0) base = atomicAdd(sw.n_active, total);
    base = __shfl(base, 0);
#pragma unroll
    for (int i = 0; i < kActiveSpan / 64; ++i) {
        if ((act[i] >> lane) & 1ull)
            sw.active[base + __builtin_popcountll(act[i] & ((1ull << lane) - 1ull))] = (int32_t)(c0 + 64 * i + lane);
        base += (uint32_t)__builtin_popcountll(act[i]);
    }
}

__global__ __launch_bounds__(kWG) void k_sum_columns(int32_t align_res, const SegInfo *__restrict__ si, SumWork sw) {
    const int lane = threadIdx.x & 63;
    const uint64_t *__restrict__ in = sw.col_tmp;
    uint64_t *seg = sw.col_seg;
    const uint32_t n_act = *sw.n_active;
    const uint32_t waves = gridDim.x * (kWG / 64);
    for (uint32_t ia = blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); ia < n_act;
         ia += waves) {
        const int64_t cc = __builtin_amdgcn_readfirstlane(sw.active[ia]);
        const int64_t lb = sw.col_seg_off[cc], n = sw.col_seg_off[cc + 1] - lb;
        int32_t run_hi = 0, cur_lo = 0;                 // last tick of every entry so far; first tick of the open interval
        int64_t np = 0, ns = 0;                         // this lane's share of the column's counts
        // one 64-entry chunk of the sorted list: (first tick, last tick) of entry i0 + lane where `mine`
        auto chunk = [&](int64_t i0, bool mine, int32_t a0, int32_t end) {
            if (!mine) end = INT32_MIN;
            int32_t incl = end;                         // inclusive prefix maximum of the last ticks
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int32_t y = __shfl_up(incl, d);
                if (lane >= d) incl = max(incl, y);
            }
            int32_t excl = __shfl_up(incl, 1);
            if (lane == 0) excl = INT32_MIN;
            if (i0 > 0) excl = max(excl, run_hi);
            const bool st = mine && i0 + lane > 0 && (int64_t)a0 - excl - 1 > kSumGap;
            const uint64_t starts = __ballot(st);
            // the interval that ends before start lane s began at the previous start (or the open one)
            const uint64_t below = starts & ((1ull << lane) - 1ull);
            const int pl = below ? 63 - __builtin_clzll(below) : -1;
            const int32_t prev_lo = __shfl(a0, max(pl, 0));
            if (i0 == 0) cur_lo = __shfl(a0, 0);        // (shuffles in uniform control flow: every lane is a source)
            if (st) interval_count(pl >= 0 ? prev_lo : cur_lo, excl, align_res, np, ns);
            if (starts) cur_lo = __shfl(a0, 63 - __builtin_clzll(starts));
            run_hi = i0 == 0 ? __shfl(incl, 63) : max(run_hi, __shfl(incl, 63));
        };
        if (n <= 64) {
            // the lengths are loaded before the sort and travel with their keys to the lanes of their ranks
            const bool mine = lane < n;
            const uint64_t x = mine ? in[lb + lane] : ~0ull;
            const int32_t na = mine ? sw.segc[key_seg(x)].na : 0;
            int32_t rank = 0;
            for (int j = 0; j < (int)n; ++j) rank += lane_u64(x, j) < x;
            if (!mine) rank = lane;
            if (mine) seg[lb + rank] = x;
            const uint32_t xs_lo = (uint32_t)__builtin_amdgcn_ds_permute(rank * 4, (int)(uint32_t)x);
            const uint32_t xs_hi = (uint32_t)__builtin_amdgcn_ds_permute(rank * 4, (int)(uint32_t)(x >> 32));
            const int32_t nas = __builtin_amdgcn_ds_permute(rank * 4, na);
            const int32_t a0 = key_a0(((uint64_t)xs_hi << 32) | xs_lo);
            chunk(0, mine, a0, a0 + nas - 1);
        } else {
            for (int64_t i0 = 0; i0 < n; i0 += 64) {
                const bool mine = i0 + lane < n;
                const uint64_t x = mine ? in[lb + i0 + lane] : 0;
                int64_t rank = 0;
                for (int64_t j0 = 0; j0 < n; j0 += 64) {
                    const uint64_t y = j0 + lane < n ? in[lb + j0 + lane] : ~0ull;
                    const int jn = (int)min<int64_t>(64, n - j0);
                    for (int j = 0; j < jn; ++j) rank += lane_u64(y, j) < x;
                }
                if (mine) seg[lb + rank] = x;
            }
            // the sorted list before the wavefront reads it back
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            for (int64_t i0 = 0; i0 < n; i0 += 64) {
                const bool mine = i0 + lane < n;
                int32_t a0 = 0, end = 0;
                if (mine) {
                    const uint64_t x = seg[lb + i0 + lane];
                    a0 = key_a0(x);
                    end = a0 + sw.segc[key_seg(x)].na - 1;
                }
                chunk(i0, mine, a0, end);
            }
        }
        if (lane == 0) interval_count(cur_lo, run_hi, align_res, np, ns);     // the last interval
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            np += __shfl_xor(np, o);
            ns += __shfl_xor(ns, o);
        }
        if (lane == 0) {
            sw.piece_off[cc] = np;
            sw.s_off[cc] = ns;
        }
    }
}

void launch_sum_fill(const DevParams &P, const Work &w, const SumWork &sw, hipStream_t st) {
    if (w.n_seg > 0)
        k_sum_fill<<<(unsigned)((w.n_seg + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>(P, w.si, w.n_seg, sw);
    const int64_t span = (int64_t)(kWG / 64) * kActiveSpan;
    k_sum_active<<<(unsigned)((sw.n_cols + span - 1) / span), kWG, 0, st>>>(sw);
    k_sum_columns<<<256 * 16, kWG, 0, st>>>(sw.align_res, w.si, sw);   // persistent waves over the listed columns
}

// Wave-uniform copies of a 64-bit value held by lane l.
__device__ __forceinline__ int64_t uniform_i64(int64_t v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// per column: piece records, and the summed charge of each tick (Kahan over the column's segments in list order).
// Wavefronts take the columns with pieces from the active list, one column at a time; lane j sums tick
// lo + 64 m + j of the current interval over the interval's segments, the same additions per tick, in the same
// order, as a tick-by-tick scan.  For a list of at most kPieceStage segments, the lanes first stage each segment's
// first tick, length and cell base in this column in the wavefront's LDS slice, so the per-segment loops read them
// with one broadcast LDS read into scalar registers and only the (coalesced) cell loads go to memory; longer lists
// read each record in the loop.
constexpr int kPieceStage = 256;
struct SumRec {
    int32_t a0, na;
    int64_t base;                                       // cells index of tick 0 of the segment in this column
};
__global__ __launch_bounds__(kWG) void k_sum_pieces(DevParams P, const SegInfo *si, const float *cells, SumWork sw) {
    __shared__ SumRec stage_all[kWG / 64][kPieceStage];
    __shared__ int32_t rmax_all[kWG / 64][kPieceStage];
    const int lane = threadIdx.x & 63;
    SumRec *rs = stage_all[threadIdx.x >> 6];
    int32_t *rmax = rmax_all[threadIdx.x >> 6];       // last tick of entries 0 .. k (a running maximum)
    const int32_t res = sw.align_res;
    const uint32_t n_act = *sw.n_active;
    const uint32_t waves = gridDim.x * (kWG / 64);
    for (uint32_t ia = blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); ia < n_act;
         ia += waves) {
        const int64_t cc = __builtin_amdgcn_readfirstlane(sw.active[ia]);
        const int32_t e = (int32_t)(cc / ((int64_t)sw.CU * sw.CV));
        const int64_t r = cc - (int64_t)e * sw.CU * sw.CV;
        const int32_t u = sw.UL + (int32_t)(r / sw.CV), v = sw.VL + (int32_t)(r % sw.CV);
        const int64_t sb = sw.col_seg_off[cc], se = sw.col_seg_off[cc + 1], n = se - sb;
        int64_t pk = sw.piece_off[cc], so = sw.s_off[cc];
        const bool staged = n <= kPieceStage;
        // the previous column's reads of the slice are done before it is overwritten
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint64_t smask[kPieceStage / 64] = {};            // interval starts among the staged entries
        if (staged) {
            // records, and the interval starts by the rule k_sum_columns counts by (first tick more than kSumGap
            // beyond the running maximum of the earlier last ticks)
            int32_t carry = INT32_MIN;
#pragma unroll
            for (int w = 0; w < kPieceStage / 64; ++w) {
                if (64 * w >= n) break;
                const int64_t k = 64 * w + lane;
                const bool mine = k < n;
                int32_t a0 = 0, end = INT32_MIN;
                if (mine) {
                    const SumSeg g = sw.segc[key_seg(sw.col_seg[sb + k])];
                    a0 = g.a0;
                    end = g.a0 + g.na - 1;
                    rs[k] = SumRec{g.a0, g.na, g.cell_off + ((int64_t)(u - g.u0) * g.nv + (v - g.v0)) * g.na_pad - g.a0};
                }
                int32_t incl = end;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int32_t y = __shfl_up(incl, d);
                    if (lane >= d) incl = max(incl, y);
                }
                incl = max(incl, carry);
                int32_t excl = __shfl_up(incl, 1);
                if (lane == 0) excl = carry;
                smask[w] = __ballot(mine && (k == 0 || (int64_t)a0 - excl - 1 > kSumGap));
                if (mine) rmax[k] = incl;
                carry = __shfl(incl, 63);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        // the interval starting at entry q of a staged list: its end entry qe (the next start) and last tick
        auto staged_interval = [&](int64_t q, int64_t &qe, int32_t &hi) {
            qe = n;
            for (int w = (int)((q + 1) >> 6); w < kPieceStage / 64 && 64 * w < n; ++w) {
                const uint64_t m = smask[w] & (((q + 1) >> 6) == w ? ~0ull << ((q + 1) & 63) : ~0ull);
                if (m) {
                    qe = 64 * w + __builtin_ctzll(m);
                    break;
                }
            }
            hi = __builtin_amdgcn_readfirstlane(rmax[qe - 1]);
        };
        auto from_lds = [&](int64_t k, int32_t &a0, int32_t &na, int64_t &base) {
            const SumRec x = rs[k];                         // the same address in every lane: a broadcast read
            a0 = __builtin_amdgcn_readfirstlane(x.a0);
            na = __builtin_amdgcn_readfirstlane(x.na);
            base = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)x.base >> 32)) << 32) |
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x.base));
        };
        auto from_global = [&](int64_t k, int32_t &a0, int32_t &na, int64_t &base) {
            const SumSeg g = sw.segc[key_seg(sw.col_seg[sb + k])];
            a0 = g.a0;
            na = g.na;
            base = g.cell_off + ((int64_t)(u - g.u0) * g.nv + (v - g.v0)) * g.na_pad - g.a0;
        };
        auto column = [&](auto seg_at, bool scanned) {
            for (int64_t q = 0; q < n;) {
                // the merged interval starting at list entry q (the rule k_sum_columns counts by)
                int32_t lo, hi, a0, na;
                int64_t base;
                seg_at(q, a0, na, base);
                lo = a0;
                hi = a0 + na - 1;
                int64_t qe = q + 1;
                if (scanned) {
                    staged_interval(q, qe, hi);
                } else {
                    for (; qe < n; ++qe) {
                        seg_at(qe, a0, na, base);
                        if (a0 - hi - 1 > kSumGap) break;
                        hi = max(hi, a0 + na - 1);
                    }
                }
                if (res >= 0) lo -= ((lo - res) % 8 + 8) % 8;
                const int32_t L = hi - lo + 1;
                int64_t np, Lpad;
                sum_interval_size(L, np, Lpad);
                float *S = sw.S + so;
                float top = 0.0f;                       // largest charge of the interval
                for (int32_t a0c = 0; a0c < Lpad; a0c += 64) {
                    const int32_t aa = lo + a0c + lane, ch = min(lo + a0c + 63, hi);
                    float sum = 0.0f, cmp = 0.0f;
                    // eight segments at a time: their cell loads are issued together, then added in list order
                    bool past = false;
                    for (int64_t k0 = q; k0 < qe && !past; k0 += 8) {
                        float val[8];
                        bool use[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            use[i] = false;
                            val[i] = 0.0f;
                            if (k0 + i < qe && !past) {
                                seg_at(k0 + i, a0, na, base);
                                if (a0 > ch) past = true;           // sorted by first tick: no later one reaches
                                else if (aa >= a0 && aa <= a0 + na - 1 && aa <= hi) {
                                    use[i] = true;
                                    val[i] = cells[base + aa];
                                }
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (use[i]) {
                                const float y = val[i] - cmp;
                                const float t = sum + y;
                                cmp = (t - sum) - y;
                                sum = t;
                            }
                    }
                    if (a0c + lane < Lpad) {
                        S[a0c + lane] = sum - cmp;
                        top = fmaxf(top, fabsf(sum - cmp));
                    }
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
                const int32_t ex = __builtin_bit_cast(int32_t, top) >> 23;
                for (int64_t k = lane; k < np; k += 64) {
                    SegInfo g = {};
                    g.u0 = u; g.nu = 1; g.v0 = v; g.nv = 1;
                    g.a0 = lo + (int32_t)k * kPieceTicks;
                    g.na = min(kPieceTicks, L - (int32_t)k * kPieceTicks);
                    g.na_pad = (g.na + kAC - 1) / kAC * kAC;
                    g.cell_off = so + k * kPieceTicks;
                    g.event = e;
                    g.n_pairs = 1;
                    if (sw.piece_lists) sw.piece[pk + k] = g;
                    sw.pdesc[pk + k] = PieceRef{g.a0, g.na, (uint32_t)(g.cell_off / kAC), ex << kBinBits};
                }
                pk += np;
                so += Lpad;
                q = qe;
            }
        };
        if (staged) column(from_lds, true);
        else column(from_global, false);
    }
}

void launch_sum_pieces(const DevParams &P, const Work &w, const SumWork &sw, hipStream_t st) {
    k_sum_pieces<<<256 * 16, kWG, 0, st>>>(P, w.si, w.cells, sw);   // persistent waves over the active columns
}

// per active pixel (one wavefront): number of column pieces in its table reach, then their ids and records in column
// order (row du, then column dv; pieces of a column in tick order).  The lanes take 64 consecutive columns at a time;
// a wavefront prefix sum of their piece counts gives each lane its place in the list.  A record is the piece's
// compact descriptor with the folded table column the pixel sees the column through, fold(du - bx) * by +
// fold(dv - by) for the column at offset (du, dv) of the pixel's reach.
// per active pixel: the number of column pieces in its reach (the columns of its +-bx x +-by sub-pixel window)
__global__ __launch_bounds__(kWG) void k_sum_lists_count(DevParams P, int64_t n_slots, const int32_t *slot_gp,
                                                         SumWork sw) {
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (slot >= n_slots) return;
    const int32_t gp = slot_gp[slot];
    const int32_t e = gp / P.npx, p = gp - e * P.npx;
    const int32_t ix = p % P.nx, iy = p / P.nx;
    const int32_t cu0 = ix * P.nsub + P.nsub / 2 - P.bx - sw.UL, cv0 = iy * P.nsub + P.nsub / 2 - P.by - sw.VL;
    const int64_t base = (int64_t)e * sw.CU * sw.CV;
    // piece_off is the exclusive prefix over the columns in row order: a row's 2 by columns of the reach count
    // piece_off[end] - piece_off[start]
    int64_t x = 0;
    for (int32_t du = lane; du < 2 * P.bx; du += 64) {
        const int64_t row = base + (int64_t)(cu0 + du) * sw.CV + cv0;
        x += sw.piece_off[row + 2 * P.by] - sw.piece_off[row];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) sw.list_off[slot] = x;
}

// per active pixel: its reach's column pieces as records, grouped by the folded table column (bin) the pixel sees
// them through and, within a bin, ascending in first tick (equal first ticks keep the mirror columns in the order
// du >= 0 before du < 0, then dv likewise).  Lane i merges the four tick-sorted piece lists of bin b0 + i.
__global__ __launch_bounds__(kWG) void k_sum_lists_fill(DevParams P, int64_t n_slots, const int32_t *slot_gp,
                                                        SumWork sw) {
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (slot >= n_slots) return;
    const int32_t gp = slot_gp[slot];
    const int32_t e = gp / P.npx, p = gp - e * P.npx;
    const int32_t ix = p % P.nx, iy = p / P.nx;
    const int32_t cu0 = ix * P.nsub + P.nsub / 2 - sw.UL, cv0 = iy * P.nsub + P.nsub / 2 - sw.VL;   // centre column
    const int64_t base = (int64_t)e * sw.CU * sw.CV;
    const int32_t nbin = P.bx * P.by;
    int64_t pos = sw.list_off[slot];
    for (int32_t b0 = 0; b0 < nbin; b0 += 64) {
        const int32_t b = b0 + lane;
        int64_t h[4] = {0, 0, 0, 0}, he[4] = {0, 0, 0, 0};
        int64_t x = 0;
        if (b < nbin) {
            const int32_t fu = b / P.by, fv = b - fu * P.by;
#pragma unroll
            for (int m = 0; m < 4; ++m) {                // the four columns whose offsets fold to (fu, fv)
                const int32_t du = (m & 1) ? -fu - 1 : fu, dv = (m & 2) ? -fv - 1 : fv;
                const int64_t col = base + (int64_t)(cu0 + du) * sw.CV + (cv0 + dv);
                h[m] = sw.piece_off[col];
                he[m] = sw.piece_off[col + 1];
                x += he[m] - h[m];
            }
        }
        int64_t incl = x;                               // inclusive prefix of the lanes' record counts
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        if (x) {
            int32_t ha[4];                              // first tick at each list's head (INT32_MAX when empty)
#pragma unroll
            for (int m = 0; m < 4; ++m) ha[m] = h[m] < he[m] ? sw.pdesc[h[m]].a0 : INT32_MAX;
            for (int64_t q = pos + incl - x; q < pos + incl; ++q) {
                int m = 0;
#pragma unroll
                for (int j = 1; j < 4; ++j) m = ha[j] < (m == 0 ? ha[0] : m == 1 ? ha[1] : ha[2]) ? j : m;
                int64_t k = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j == m) {
                        k = h[j]++;
                        ha[j] = h[j] < he[j] ? sw.pdesc[h[j]].a0 : INT32_MAX;
                    }
                if (sw.piece_lists) sw.list[q] = (int32_t)k;
                PieceRef r = sw.pdesc[k];
                r.bin |= b;
                sw.rec[q] = r;
            }
        }
        pos += __shfl(incl, 63);
    }
}

void launch_sum_lists_count(const DevParams &P, const Work &w, const SumWork &sw, int64_t n_slots, hipStream_t st) {
    if (n_slots > 0)
        k_sum_lists_count<<<(unsigned)((n_slots + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>(P, n_slots, w.slot_gp, sw);
}
void launch_sum_lists_fill(const DevParams &P, const Work &w, const SumWork &sw, int64_t n_slots, int64_t n_list,
                           hipStream_t st) {
    if (n_slots > 0)
        k_sum_lists_fill<<<(unsigned)((n_slots + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>(P, n_slots, w.slot_gp, sw);
    (void)n_list;
}

// Mirror merge.  A pixel convolves every record of one folded table column with the same table column, so a run of
// its list's records with the same bin whose tick spans overlap or lie at most kMergeGap ticks apart is one record
// whose charge is the members' sum, taken in list order (a member's charge sits at its first tick's offset from the
// union's first tick).  Runs are cut at every 64th record of the pixel's
// list (the lanes of one pass), and a run whose union would exceed kPieceMax ticks is not merged; a run of one record
// stays as it is.  Count pass: records and merged-charge floats per pixel; fill pass: the merged records (in list
// order) and their charges.  One wavefront per pixel; the runs of 64 records are found with segmented lane scans.
constexpr int32_t kMergeGap = 8;

// Inclusive segmented scans over the wavefront (a segment starts at a lane whose flag is set).
__device__ __forceinline__ int32_t seg_scan_max(int32_t v, bool start) {
    const int lane = lane_id();
    int f = start;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(v, d);
        const int g = __shfl_up(f, d);
        if (lane >= d && !f) {
            v = max(v, y);
            f |= g;
        }
    }
    return v;
}
__device__ __forceinline__ int32_t seg_scan_min(int32_t v, bool start) {
    const int lane = lane_id();
    int f = start;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(v, d);
        const int g = __shfl_up(f, d);
        if (lane >= d && !f) {
            v = min(v, y);
            f |= g;
        }
    }
    return v;
}
template <bool FILL>
__global__ __launch_bounds__(kWG) void k_sum_merge(int64_t n_slots, SumWork sw) {
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (slot >= n_slots) return;
    const int64_t pb = sw.list_off[slot], pe = sw.list_off[slot + 1];
    int64_t ng = FILL ? sw.mlist_off[slot] : 0, nm = FILL ? sw.m_off[slot] : 0;
    for (int64_t c0 = pb; c0 < pe; c0 += 64) {
        const int32_t n = (int32_t)min<int64_t>(64, pe - c0);
        const bool in = lane < n;
        PieceRef r{0, 0, 0, 0};
        if (in) r = sw.rec[c0 + lane];
        const int32_t end = r.a0 + r.na - 1;
        // runs: a new bin, or a first tick beyond the bin's spans so far (first ticks ascend within a bin) + the gap
        const int32_t bin = r.bin & kBinMask;
        const bool fb = lane == 0 || bin != __shfl_up(bin, 1);
        const int32_t mb = seg_scan_max(end, fb);
        const int32_t mprev = __shfl_up(mb, 1);
        bool st = fb || r.a0 > mprev + 1 + kMergeGap;
        const int32_t ghi = seg_scan_max(end, st);       // the run's last tick so far
        const int32_t glo = seg_scan_min(r.a0, st);      // its first tick
        // each record's natural run ends before the next run start; the verdict on the run's span is read there
        const uint64_t nat = __ballot(in && st);
        const uint64_t nat_after = lane == 63 ? 0ull : nat >> (lane + 1);
        const int32_t run_end = nat_after ? lane + __builtin_ctzll(nat_after) : n - 1;
        const bool ok = __shfl((int)(ghi - glo + 1 <= kPieceMax), max(min(run_end, 63), 0)) != 0;
        st = in && (st || !ok);                         // runs over kPieceMax ticks stay single records
        const uint64_t starts = __ballot(st);
        const uint64_t after = lane == 63 ? 0ull : starts >> (lane + 1);
        const int32_t nxt = after ? lane + 1 + __builtin_ctzll(after) : n;
        const int32_t rhi = __shfl(ghi, max(nxt - 1, 0));
        const bool multi = st && nxt - lane > 1;
        const int32_t L = multi ? rhi - r.a0 + 1 : r.na;
        const int32_t Lp = multi ? (L + kAC - 1) / kAC * kAC : 0;
        // bound of a merged run's charge: its members' largest exponent, raised by the bits of their number
        const int32_t emax = __shfl(seg_scan_max((int32_t)((uint32_t)r.bin >> kBinBits), st), max(nxt - 1, 0));
        const int32_t mexp = min(emax + 32 - __builtin_clz(max(nxt - lane, 2) - 1), 254);
        int64_t incl = Lp;                              // inclusive prefix of the merged-charge floats
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        if (FILL) {
            const int64_t moff = nm + incl - Lp;
            if (st) {
                const int64_t g = ng + __builtin_popcountll(starts & ((1ull << lane) - 1ull));
                sw.mrec[g] = multi ? PieceRef{r.a0, L, sw.nS8 + (uint32_t)(moff / kAC), bin | mexp << kBinBits} : r;
                sw.mstart[g] = c0 + lane;
            }
        }
        ng += __builtin_popcountll(starts);
        nm += __shfl(incl, 63);
    }
    if (!FILL && lane == 0) {
        sw.mlist_off[slot] = ng;
        sw.m_off[slot] = nm;
    }
    if (FILL && lane == 0 && slot == n_slots - 1) sw.mstart[ng] = pe;
}

// The merged records' charges, members in list order: 8 lanes a record, over its ticks.  A pixel's runs are independent of
// each other, so they are spread over the chip by record (in the pass above, a wavefront per pixel, the pixels with the
// longest lists kept it running).  A 20,000-segment event has 13.5 million records of some 30 ticks, whose charges (1.6 GB)
// are what bounds it: the pass and this kernel take 245 + 636 us instead of 1424, for a 500-segment event 37 + 18 instead of
// 345 (16 lanes x 4 ticks a record: 848, 4 x 8: 740).
constexpr int32_t kMergeLanes = 8, kMergeTicks = 8;     // ticks a lane at a time
constexpr int64_t kMergeBlocks = 1 << 17;               // (a large batch has more records than one launch has threads for)
__global__ __launch_bounds__(kWG) void k_sum_merged(int64_t n_rec, SumWork sw) {
    const int lane = threadIdx.x % kMergeLanes;
    const int64_t step = (int64_t)gridDim.x * (kWG / kMergeLanes);
    for (int64_t g = (int64_t)blockIdx.x * (kWG / kMergeLanes) + threadIdx.x / kMergeLanes; g < n_rec; g += step) {
        const PieceRef m = sw.mrec[g];
        if (m.cell8 < sw.nS8) continue;                 // a single piece
        const PieceRef *rec = sw.rec + sw.mstart[g];
        const int32_t n_mem = (int32_t)(sw.mstart[g + 1] - sw.mstart[g]), lp = (m.na + kAC - 1) / kAC * kAC;
        float *out = sw.Sm + (int64_t)(m.cell8 - sw.nS8) * kAC;
        for (int32_t t0 = lane; t0 < lp; t0 += kMergeLanes * kMergeTicks) {
            float v[kMergeTicks];
#pragma unroll
            for (int i = 0; i < kMergeTicks; ++i) v[i] = 0.0f;
            for (int32_t k = 0; k < n_mem; k += 2) {     // two members' loads in flight
                const PieceRef r0 = rec[k], r1 = rec[min(k + 1, n_mem - 1)];
                const uint32_t o0 = (uint32_t)(m.a0 + t0 - r0.a0), n0 = (uint32_t)r0.na;
                const uint32_t o1 = (uint32_t)(m.a0 + t0 - r1.a0), n1 = k + 1 < n_mem ? (uint32_t)r1.na : 0u;
                const float *c0 = sw.S + (int64_t)r0.cell8 * kAC, *c1 = sw.S + (int64_t)r1.cell8 * kAC;
                float x0[kMergeTicks], x1[kMergeTicks];
#pragma unroll
                for (int i = 0; i < kMergeTicks; ++i) {
                    const uint32_t d = (uint32_t)(kMergeLanes * i);
                    x0[i] = o0 + d < n0 ? c0[o0 + d] : 0.0f;
                    x1[i] = o1 + d < n1 ? c1[o1 + d] : 0.0f;
                }
#pragma unroll
                for (int i = 0; i < kMergeTicks; ++i) v[i] = (v[i] + x0[i]) + x1[i];   // an exact zero leaves v unchanged
            }
#pragma unroll
            for (int i = 0; i < kMergeTicks; ++i)
                if (t0 + kMergeLanes * i < lp) out[t0 + kMergeLanes * i] = v[i];
        }
    }
}

void launch_sum_merge(const SumWork &sw, int64_t n_slots, int64_t n_rec, hipStream_t st) {
    if (n_slots <= 0) return;
    const unsigned g = (unsigned)((n_slots + kWG / 64 - 1) / (kWG / 64));
    if (n_rec < 0) {
        k_sum_merge<false><<<g, kWG, 0, st>>>(n_slots, sw);
        return;
    }
    k_sum_merge<true><<<g, kWG, 0, st>>>(n_slots, sw);
    constexpr int64_t per = kWG / kMergeLanes;
    if (n_rec > 0)
        k_sum_merged<<<(unsigned)std::min<int64_t>((n_rec + per - 1) / per, kMergeBlocks), kWG, 0, st>>>(n_rec, sw);
}

// Summed induction, one wavefront per work unit (active pixel, tile of kTileTicks ticks): lane t owns ticks
// t0 + 8t .. +7 of the tile, and the wavefront streams every column piece of the pixel's list whose tick window
// [a0 - T_R + 1, a0 + na - 1] meets the tile through the four-block register ring, three blocks ahead and into the
// next piece (pieces start at the aligning residue, so every lane's table offset is a multiple of 8 and the loads
// are aligned 16-byte loads).  The pieces come as 16-byte records (first tick, length, charge offset, folded table
// column), so the walk needs no dependent loads.  Lanes whose ticks lie outside a piece's window read the table's
// zero padding, so they add exact zeros.  The products are added to the lane's running sums with Kahan
// compensation after every 4 pieces (pieces in list order: deterministic and batch-invariant).  Wavefronts take
// units from a counter and never synchronise with each other; the first tile of a pixel also accounts the charge
// that its pieces induce outside the window.
// A record's summed charge: in the column pieces' buffer, or in the merged records' one.
__device__ __forceinline__ const float *cell_ptr(const float *S, const float *Sm, uint32_t nS8, uint32_t cell8) {
    return cell8 < nS8 ? S + (int64_t)cell8 * kAC : Sm + (int64_t)(cell8 - nS8) * kAC;
}

constexpr int32_t kSumKahanEvery = 4;   // pieces summed in FP32 registers between compensated additions

template <bool SHIFT>
__global__ __launch_bounds__(kWG) void k_induce_summed(DevParams P, const SegInfo *__restrict__ piece,
                                                       const float *__restrict__ S, const float *__restrict__ Sm,
                                                       uint32_t nS8, const float *__restrict__ Rpad,
                                                       const double *__restrict__ prefix,
                                                       const int64_t *__restrict__ list_off,
                                                       const int32_t *__restrict__ list,
                                                       const PieceRef *__restrict__ rec,
                                                       const int32_t *__restrict__ order,
                                                       const int32_t *__restrict__ slot_gp, float *__restrict__ wave,
                                                       DevHeader *H, double *report) {
    const int lane = threadIdx.x & 63;
    const int32_t NT = P.nticks, TR = P.t_r;
    const int32_t n_tiles = (NT + kTileTicks - 1) / kTileTicks;
    const int64_t n_units = H->n_slots * n_tiles;
    for (;;) {
        uint32_t got = 0;
        if (lane == 0) got = atomicAdd(&H->work[2], 1u);
        const int64_t unit = (int64_t)__builtin_amdgcn_readfirstlane(__shfl(got, 0));
        if (unit >= n_units) break;
        const int64_t ui = unit / n_tiles;
        const int64_t slot = order ? order[ui] : ui;                    // largest-first when an order is given
        const int32_t t0 = (int32_t)(unit - ui * n_tiles) * kTileTicks, t1 = t0 + kTileTicks - 1;
        const int32_t gp = slot_gp[slot];
        const int32_t e = gp / P.npx, p = gp - e * P.npx;
        const int32_t uc = (p % P.nx) * P.nsub + P.nsub / 2, vc = (p / P.nx) * P.nsub + P.nsub / 2;
        const int32_t nb = t0 + 8 * lane;
        const int64_t pb = list_off[slot], pe = list_off[slot + 1];
        float acc[8], sum[8], cmp[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) { acc[r] = 0.0f; sum[r] = 0.0f; cmp[r] = 0.0f; }
        auto meets = [&](int64_t k) {
            const SegInfo &g = piece[list[k]];
            return g.a0 + g.na - 1 >= t0 && g.a0 - (TR - 1) <= t1;
        };
        auto colof = [&](int64_t k, const float *&col, const float *&cc, int32_t &nblk) {
            const SegInfo &g = piece[list[k]];
            col = Rpad + (int64_t)(fold(g.u0 - uc) * P.by + fold(g.v0 - vc)) * P.col_len + (nb - g.a0 + TR - 1 + kPad);
            cc = S + g.cell_off;
            nblk = g.na_pad / kAC;
        };
        if constexpr (!SHIFT) {                         // aligned ping-pong per piece, Kahan after every 4 pieces
            auto kahan = [&] {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float y = acc[r] - cmp[r];
                    const float t = sum[r] + y;
                    cmp[r] = (t - sum[r]) - y;
                    sum[r] = t;
                    acc[r] = 0.0f;
                }
            };
            // the pixel's pieces that meet the tile, in list order, streamed through the four-block register ring
            // (three blocks ahead, the next piece's first blocks loaded while the current one runs)
            auto skip = [&](int64_t q) {
                while (q < pe) {
                    const PieceRef r = rec[q];
                    if (r.a0 + r.na - 1 >= t0 && r.a0 - (TR - 1) <= t1) break;
                    ++q;
                }
                return q;
            };
            int32_t pending = 0;
            int64_t q = skip(pb);
            if (q < pe) {
                auto colp = [&](const PieceRef &r) {
                    return Rpad + (int64_t)(r.bin & kBinMask) * P.col_len + (nb - r.a0 + TR - 1 + kPad);
                };
                const PieceRef r0 = rec[q];
                auto adv = [&](const float *&ncol, const float *&ncc, int32_t &nn) {
                    q = skip(q + 1);
                    if (q >= pe) return false;
                    const PieceRef r = rec[q];
                    ncol = colp(r);
                    ncc = cell_ptr(S, Sm, nS8, r.cell8);
                    nn = (r.na + kAC - 1) / kAC;
                    return true;
                };
                auto done = [&] {
                    if (++pending == kSumKahanEvery) {
                        kahan();
                        pending = 0;
                    }
                };
                column_stream<false, true>(colp(r0), cell_ptr(S, Sm, nS8, r0.cell8), (r0.na + kAC - 1) / kAC, adv,
                                           done, acc);
            }
            if (pending) kahan();
        } else {
            int64_t q = pb;
            while (q < pe && !meets(q)) ++q;
            if (q < pe) {
                const float *col, *cc;
                int32_t nblk;
                colof(q, col, cc, nblk);
                auto adv = [&](const float *&ncol, const float *&ncc, int32_t &nn) {
                    do { ++q; } while (q < pe && !meets(q));
                    if (q >= pe) return false;
                    colof(q, ncol, ncc, nn);
                    return true;
                };
                auto done = [&] {
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const float y = acc[r] - cmp[r];
                        const float t = sum[r] + y;
                        cmp[r] = (t - sum[r]) - y;
                        sum[r] = t;
                        acc[r] = 0.0f;
                    }
                };
                column_stream<SHIFT, false>(col, cc, nblk, adv, done, acc);
            }
        }
        float *wrow = wave + slot * NT;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (nb + r < NT) wrow[nb + r] = sum[r] - cmp[r];
        if (t0 == 0) {                                  // charge induced outside [0, NT) by the pixel's pieces
            double clip = 0.0;
            for (int64_t k = pb + lane; k < pe; k += 64) {
                const PieceRef g = rec[k];
                const int32_t wlo = g.a0 - (TR - 1), whi = g.a0 + g.na - 1;
                if (wlo >= 0 && whi < NT) continue;
                const double *pf = prefix + (int64_t)(g.bin & kBinMask) * (TR + 1);
                const float *cv = cell_ptr(S, Sm, nS8, g.cell8);
                for (int32_t a = 0; a < g.na; ++a) {
                    const int32_t aa = g.a0 + a;
                    const int32_t klo = min(max(TR - 1 - aa, 0), TR), khi = min(max(NT + TR - 1 - aa, 0), TR);
                    const double dropped = klo >= khi ? pf[TR] : pf[klo] + (pf[TR] - pf[khi]);
                    clip += (double)cv[a] * dropped;
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) clip += __shfl_xor(clip, o);
            if (lane == 0 && clip != 0.0) atomicAdd(&report[(int64_t)e * 5 + 3], clip);
        }
    }
}

// ------------------------------------------------------------------------------------------ half-pair matrix form
// Summed induction on the FP16 matrix cores.  Every FP32 factor is a pair of halves, x 2^k = h + l with h = half(x 2^k)
// and l = half(x 2^k - h): 22 or more significant bits of x, and h h', h l', l h' are exact in the FP32 accumulator (the
// dropped l l' is below 2^-22 of the product).  2^k puts the largest value of a table column (fixed when the table is
// installed) below 2^15, and a record's largest charge (a bound of it; a record's exponent is stored with its bin): a
// record keeps its bits beside brighter ones, and only ticks below 2^-17 of its own largest keep fewer.
//
// One wavefront per work unit (active pixel, kMmaTiles tiles of 256 ticks), taken from a counter.  A record's current on
// a tile's ticks t0 + 16 j + i is D[i][j] = sum_w A[i][w] B[w][j] with A[i][w] = S[i - w + off] (the charge, a Toeplitz
// matrix) and B[w][j] = R[16 j + w + c], w in [0, off + 16).  off is the smallest value >= L - 1 that makes c a multiple
// of 8, so that a lane's 8 consecutive table values are one aligned 16-byte word; every w is covered 32 at a time by a
// 16x16x32 instruction (lane l gives A[l % 16][8 (l / 16) ..] and B[8 (l / 16) ..][l % 16]).  The table words of a
// record's window are staged in LDS (a tile reads each about 4 times), the charge as eight copies shifted by one value,
// so that every lane's 8 consecutive (reversed) values are one aligned 16-byte word too; A then serves all tiles.
// Tiles outside the record's window are skipped.  Every two parts the products leave the matrix accumulators and are added
// to the lane's sums with Kahan compensation, in list order (deterministic and batch-invariant); the second part first
// takes the accumulators to its own scale.
//
// The vector-ALU form of the same sums (256-tick units, 32 multiply-adds per lane against three LDS reads) took 37.5 ms
// on a module event of 20,000 segments (13.6 million records, 1.37e12 products) and 36.2 ms on a spill tile of 64,000;
// this one 16.7 and 16.6 ms, at an error against FP64 that is 0.7 to 0.95 of its (1.21e-7 against 1.30e-7 of the norm, of
// a pixel at most 8e-7 of itself against 1.1e-6).  One scale for 64 records would save 2 % (16.3 ms), a small event's serial
// chains 8 %, and leave a pixel of little charge beside much with 1.5e-5; an addition after every part costs 2 %.
// It runs at the card's power limit (2.07 GHz against 2.34 GHz), with the matrix cores busy 30 % and LDS about 75 % of
// the time.  3 tiles per unit run 4 wavefronts per SIMD; 4 tiles (3 wavefronts) took 2 to 3 % longer, 2 tiles 10 % and
// 1 tile 40 %: the charge is staged for fewer products.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int32_t kMmaSub = 256;                        // ticks of one tile
constexpr int32_t kMmaTiles = 3;                        // tiles of a work unit
constexpr int32_t kMmaUnit = kMmaTiles * kMmaSub;
constexpr int32_t kMmaPart = 72;                        // charge ticks taken at a time (at most three steps of 32)
constexpr int32_t kMmaLow = 24;                         // staged charge position of a part's last tick
constexpr int32_t kMmaCopy = 144;                       // halves of one shifted copy (288 B: the copies' banks differ by 8)
constexpr int32_t kMmaOct = kMmaTiles * 32 + 16;        // octets (8 table values, 16 bytes) of the longest window
constexpr int32_t kMmaKahanEvery = 2;                   // (more would scale D out of range)
static_assert(kPad >= kMmaSub + kMmaPart + 16 + 96, "summed matrix induction reads");

struct alignas(16) MmaStage {                           // LDS of one wavefront
    u32x4 r[2][kMmaOct];                                // [plane][octet] of the table window
    uint32_t s[2][8][kMmaCopy / 2];                     // [plane][shift] of the reversed charge: copy k has m + k at m
};

// Scale of a table column of zeros: its charge never sets a common scale and becomes zero under any.
constexpr int32_t kZeroColumn = 1 << 20;

// Planes of the response table: half pairs of column b scaled by 2^exps[b], in the layout of the FP32 columns.
__global__ __launch_bounds__(kWG) void k_table_halves(const float *__restrict__ Rpad, int32_t col_len,
                                                      _Float16 *__restrict__ hi, _Float16 *__restrict__ lo,
                                                      int32_t *__restrict__ exps) {
    __shared__ float red[kWG / 64];
    const int64_t base = (int64_t)blockIdx.x * col_len;
    float m = 0.0f;
    for (int32_t k = threadIdx.x; k < col_len; k += kWG) m = fmaxf(m, fabsf(Rpad[base + k]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane_id() == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    for (int i = 0; i < kWG / 64; ++i) m = fmaxf(m, red[i]);
    const int32_t e = m > 0.0f ? 14 - ilogbf(m) : kZeroColumn;
    if (threadIdx.x == 0) exps[blockIdx.x] = e;
    for (int32_t k = threadIdx.x; k < col_len; k += kWG) {
        const float x = ldexpf(Rpad[base + k], e);
        const _Float16 h = (_Float16)x;
        hi[base + k] = h;
        lo[base + k] = (_Float16)(x - (float)h);
    }
}

void launch_table_halves(const float *Rpad, int32_t n_col, int32_t col_len, void *hi, void *lo, int32_t *exps,
                         hipStream_t st) {
    k_table_halves<<<(unsigned)n_col, kWG, 0, st>>>(Rpad, col_len, (_Float16 *)hi, (_Float16 *)lo, exps);
}

// Tiles T0 .. T1 of a staged part (kn steps of 32) into their accumulators; tiles in pairs: two independent chains, few
// registers.
template <int T0, int T1>
__device__ __forceinline__ void mma_tiles(const u32x4 *rl, const u32x4 *sl, int32_t kn, floatx4 (&D)[kMmaTiles]) {
    for (int32_t k = 0; k < kn; ++k) {
        const half8 ah = __builtin_bit_cast(half8, sl[4 * k]), al = __builtin_bit_cast(half8, sl[4 * k + kMmaCopy]);
#pragma unroll
        for (int T = T0; T <= T1; T += 2) {
            const u32x4 *r0 = rl + 32 * (T - T0) + 4 * k;
            const half8 h0 = __builtin_bit_cast(half8, r0[0]), l0 = __builtin_bit_cast(half8, r0[kMmaOct]);
            if (T < T1) {
                const half8 h1 = __builtin_bit_cast(half8, r0[32]), l1 = __builtin_bit_cast(half8, r0[kMmaOct + 32]);
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, h0, D[T], 0, 0, 0);
                D[T + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, h1, D[T + 1], 0, 0, 0);
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, h0, D[T], 0, 0, 0);
                D[T + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, h1, D[T + 1], 0, 0, 0);
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, l0, D[T], 0, 0, 0);
                D[T + 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, l1, D[T + 1], 0, 0, 0);
            } else {
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, h0, D[T], 0, 0, 0);
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, h0, D[T], 0, 0, 0);
                D[T] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, l0, D[T], 0, 0, 0);
            }
        }
    }
}
// The tiles t0 .. t1 of a part (uniform), each range its own straight code (the whole unit first).
template <int T0 = 0, int T1 = kMmaTiles - 1>
__device__ __forceinline__ void mma_dispatch(const u32x4 *rl, const u32x4 *sl, int32_t kn, int32_t t0, int32_t t1,
                                             floatx4 (&D)[kMmaTiles]) {
    if (t0 == T0 && t1 == T1) return mma_tiles<T0, T1>(rl, sl, kn, D);
    if constexpr (T1 > T0) mma_dispatch<T0, T1 - 1>(rl, sl, kn, t0, t1, D);
    else if constexpr (T0 + 1 < kMmaTiles) mma_dispatch<T0 + 1, kMmaTiles - 1>(rl, sl, kn, t0, t1, D);
}

__global__ __launch_bounds__(kWG, 4) void k_induce_summed_mma(DevParams P, const float *__restrict__ S,
                                                              const float *__restrict__ Sm, uint32_t nS8,
                                                              const u32x4 *__restrict__ Rh, const u32x4 *__restrict__ Rl,
                                                              const int32_t *__restrict__ Rexp,
                                                              const int64_t *__restrict__ list_off,
                                                              const PieceRef *__restrict__ rec,
                                                              const int32_t *__restrict__ order,
                                                              float *__restrict__ wave, DevHeader *H) {
    __shared__ MmaStage stage_all[kWG / 64];
    MmaStage &st = stage_all[threadIdx.x >> 6];
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const int32_t NT = P.nticks, TR = P.t_r;
    const int32_t n_tiles = (NT + kMmaUnit - 1) / kMmaUnit;
    const int64_t n_units = H->n_slots * n_tiles;
    // staged charge: positions below kMmaLow - 1 stay zero
    for (int32_t k = lane; k < 2 * 8 * kMmaCopy / 2; k += 64) st.s[0][0][k] = 0u;
    const u32x4 *rl = st.r[0] + 2 * li + lg;             // this lane's octet of tile 0, step 0
    // staging of the charge: lane k holds positions kMmaLow - 1 + k (and + 63 in the second round) and writes them with
    // their upper neighbour, one word per copy of its position's parity
    uint32_t *ws[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int32_t q = kMmaLow - 1 + 63 * r + lane;
        ws[r] = &st.s[0][q & 1][(q - (q & 1)) / 2];
    }
    const int32_t pos0 = 15 - li + 8 * lg + kMmaLow;
    for (;;) {
        uint32_t got = 0;
        if (lane == 0) got = atomicAdd(&H->work[2], 1u);
        const int64_t unit = (int64_t)__builtin_amdgcn_readfirstlane(__shfl(got, 0));
        if (unit >= n_units) break;
        const int64_t ui = unit / n_tiles;
        const int64_t slot = order ? order[ui] : ui;                    // largest-first when an order is given
        const int32_t t0 = (int32_t)(unit - ui * n_tiles) * kMmaUnit, t1 = min(t0 + kMmaUnit, NT) - 1;
        const int64_t pb = list_off[slot], pe = list_off[slot + 1];
        float sum[4 * kMmaTiles], cmp[4 * kMmaTiles];
#pragma unroll
        for (int r = 0; r < 4 * kMmaTiles; ++r) { sum[r] = 0.0f; cmp[r] = 0.0f; }
        floatx4 D[kMmaTiles];
#pragma unroll
        for (int T = 0; T < kMmaTiles; ++T) D[T] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
        for (int64_t c0 = pb; c0 < pe; c0 += 64) {
            // 64 records at a time: each lane prepares one
            PieceRef pr{0, 0, 0, 0};
            const bool in = c0 + lane < pe;
            if (in) pr = rec[c0 + lane];
            const int32_t bin = pr.bin & kBinMask;
            const bool meets = in && pr.a0 + pr.na - 1 >= t0 && pr.a0 - TR + 1 <= t1;
            if (!__ballot(meets)) continue;
            // the record's scales: charge x 2^(N - eb) below 2^15; its products are 2^N times what they stand for
            const int32_t eb = meets ? Rexp[bin] : 0;
            const int32_t N = min(max(min(141 - (int32_t)((uint32_t)pr.bin >> kBinBits), 126) + eb, -126), 126);
            int pending = 0;                             // parts in D, and its scale
            int32_t scale = 0;
            auto flush = [&] {
                const float down = __builtin_bit_cast(float, (127 - scale) << 23);
#pragma unroll
                for (int T = 0; T < kMmaTiles; ++T)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float y = fmaf(D[T][r], down, -cmp[4 * T + r]);
                        const float t = sum[4 * T + r] + y;
                        cmp[4 * T + r] = (t - sum[4 * T + r]) - y;
                        sum[4 * T + r] = t;
                    }
                pending = 0;
            };
            // records longer than kMmaPart ticks go in several rounds over the chunk
            for (int32_t done = 0;; done += kMmaPart) {
                const int32_t L = min(pr.na - done, kMmaPart), a0 = pr.a0 + done;
                const int32_t lo = a0 - TR + 1 - t0, hi = a0 + L - 1 - t0;
                uint64_t mask = __ballot(meets && L > 0 && hi >= 0 && lo <= t1 - t0);
                const int32_t T0 = max(lo, 0) / kMmaSub, T1 = min(hi, t1 - t0) / kMmaSub;
                const int32_t off = L - 1 + ((TR - a0 - L) & 7), kn = (off + 47) / 32;
                // table bytes [v_at, v_end) of a plane are what the tiles read, charge bytes [v_q, v_q + 4 L)
                const uint32_t v_at = (uint32_t)(bin * P.col_len + t0 + T0 * kMmaSub - a0 - off + TR - 1 + kPad) * 2u;
                const uint32_t v_end = v_at + 16u * (uint32_t)(32 * (T1 - T0 + 1) + 4 * kn - 2);
                const int32_t pack = 4 * L | kn << 9 | T0 << 11 | T1 << 13 | (off + 16 - L) << 15;
                const uint64_t v_q = (uint64_t)(cell_ptr(S, Sm, nS8, pr.cell8) + done);
                // a part in hand: its fields and the lane's words of it, loaded one part ahead
                u32x4 gh[2], gl[2];
                float x[2] = {0.0f, 0.0f};
                int32_t qp = 0, qn = 0, qe = 0;
                auto fetch = [&](int i) {
                    qp = __builtin_amdgcn_readlane(pack, i);
                    qe = __builtin_amdgcn_readlane(eb, i);
                    qn = __builtin_amdgcn_readlane(N, i);
                    const int32_t o = __builtin_amdgcn_readlane((int)v_at, i);
                    const int32_t end = __builtin_amdgcn_readlane((int)v_end, i);
                    // loads past the ends return zeros without touching memory
                    const __amdgpu_buffer_rsrc_t rh =
                        __builtin_amdgcn_make_buffer_rsrc((void *)Rh, (short)0, end, kBufferWord3);
                    const __amdgpu_buffer_rsrc_t rw =
                        __builtin_amdgcn_make_buffer_rsrc((void *)Rl, (short)0, end, kBufferWord3);
                    gh[0] = __builtin_amdgcn_raw_buffer_load_b128(rh, 16 * lane, o, 0);
                    gl[0] = __builtin_amdgcn_raw_buffer_load_b128(rw, 16 * lane, o, 0);
                    gh[1] = __builtin_amdgcn_raw_buffer_load_b128(rh, 16 * lane + 1024, o, 0);
                    gl[1] = __builtin_amdgcn_raw_buffer_load_b128(rw, 16 * lane + 1024, o, 0);
                    const int32_t l4 = qp & 511;
                    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
                        (void *)uniform_i64((int64_t)v_q, i), (short)0, l4, kBufferWord3);
                    x[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rq, l4 - 4 * lane, 0, 0));
                    if ((qp >> 9 & 3) > 2)
                        x[1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rq, l4 - 4 * lane - 252, 0, 0));
                };
                // the next part's scale n, the factor that takes D to it (none of D for the first of two parts; exact) and
                // its charge's; a part weaker by 2^-64 than the one before stays in a scale that keeps that one finite
                int32_t n = 0;
                float by = 0.0f, xu = 0.0f;
                auto scales = [&] {
                    n = pending ? min(qn, scale + 64) : qn;
                    by = __builtin_bit_cast(float, pending ? max(127 + n - scale, 0) << 23 : 0);
                    xu = __builtin_bit_cast(float, (127 + max(n - qe, -127)) << 23);
                };
                if (mask) {
                    fetch(__builtin_ctzll(mask));
                    scales();
                }
                while (mask) {
                    mask &= mask - 1ull;
                    const int32_t p = qp, pk = p >> 9 & 3, pT0 = p >> 11 & 3, pT1 = p >> 13 & 3;
                    // the previous part's reads of the slice are done before it is overwritten
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    st.r[0][lane] = gh[0];
                    st.r[1][lane] = gl[0];
                    if (pT1 > pT0 && lane + 64 < kMmaOct) {
                        st.r[0][lane + 64] = gh[1];
                        st.r[1][lane + 64] = gl[1];
                    }
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        if (r == 1 && pk < 3) break;
                        const float y = x[r] * xu;
                        const _Float16 h = (_Float16)y, l = (_Float16)(y - (float)h);
                        const uint32_t w = (uint32_t)__builtin_bit_cast(uint16_t, h) |
                                           (uint32_t)__builtin_bit_cast(uint16_t, l) << 16;
                        // lane + 1's values (DPP wave_shl:1, zero past lane 63: the next round writes that word again)
                        const uint32_t v = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x130, 0xf, 0xf, true);
                        const uint32_t wh = __builtin_amdgcn_perm(v, w, 0x05040100);
                        const uint32_t wl = __builtin_amdgcn_perm(v, w, 0x07060302);
                        if (r == 0 || lane < 40)            // (three steps read up to position 119)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                ws[r][k * (kMmaCopy - 1)] = wh;
                                ws[r][k * (kMmaCopy - 1) + 8 * kMmaCopy / 2] = wl;
                            }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    if (mask) fetch(__builtin_ctzll(mask));
                    // A[i][8g + q] is at position 15 - i + 8g + q + (kMmaLow - (off + 16 - L))
                    const int32_t pos = pos0 - (p >> 15);
                    const u32x4 *sl = (const u32x4 *)&st.s[0][pos & 7][0] + (pos >> 3);
#pragma unroll
                    for (int T = 0; T < kMmaTiles; ++T) D[T] *= by;
                    mma_dispatch(rl, sl, pk, pT0, pT1, D);
                    scale = n;
                    if (++pending == kMmaKahanEvery) flush();
                    scales();
                }
                if (!__ballot(meets && pr.na > done + kMmaPart)) break;
            }
            if (pending) flush();
        }
        float *wrow = wave + slot * NT;
#pragma unroll
        for (int T = 0; T < kMmaTiles; ++T) {
            const int32_t nb = t0 + kMmaSub * T + 16 * li + 4 * lg;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (nb + r < NT) wrow[nb + r] = sum[4 * T + r] - cmp[4 * T + r];
        }
    }
}

// ------------------------------------------------------------------------------------------ pixel products
// Per-pixel induction of a group of segments on the FP16 matrix cores.  The group's charge is summed per table column
// (the columns' mirror images folded onto them) and tick: C[bin][a].  With the bins as the contraction,
// Z[a][tau] = sum_bin C[bin][a] R[bin][tau] is a matrix product with no padding but the rounding of ticks to 16, of
// table ticks to 16 and of the bins to whole octets (8 consecutive j of one i), and the current is the sum along Z's
// anti-diagonals, I[n] = sum_a Z[a][n - a + T_R - 1].  Both factors are half pairs as above.  The charge's scale is one
// per staged tick (a row of Z), the largest that its own values bear, each times its column's scale: a tick of little
// charge keeps its bits beside a bright one, and the scales are taken off before ticks meet in a sum.  The table octets
// are laid out so that 16 table ticks of an octet are 256 consecutive bytes (a 16x16x32 operand of four octets is four
// such runs).  Anti-diagonals: lane (tau, g) holds rows a = 4g .. 4g + 3 of a tile, so row a moves up by a lanes within
// its 16 (DPP row shifts; what leaves the 16 belongs to the next tile), and the four groups are added by lane swaps once
// per 16 output ticks.
// A workgroup stages 32 ticks x 32 octets of C at a time, and each wavefront owns a range of output ticks (it also
// computes the two table tiles below its range), so no sum is shared between wavefronts: the result depends only on
// the segments' order.
//   What bounds it: dense events the table, which every stage streams from beyond L2 (59.6 GB in 8.5 ms for 3000 segments,
// 7.0 TB/s, the matrix cores 21 % busy), so all loads of a tile pair are issued before its products (without that 14.6
// ms); sparse ones the latency of staging, so an octet's images are loaded eight at a time (64 tracks 1.23 ms, four at a
// time 3 % longer).  A group saves work only where its segments share columns: 16 segments and 128 ticks (64 and 256 ticks
// measured the same).  Two workgroups of four wavefronts a CU: three spill (6 % longer).  64 ticks a stage halve the table
// reads but leave one workgroup a CU (3 % less, tracks 40 % more).  Atomic units of 8 segments (4: 4.7 ms, 8: 3.06, 16: 3.3).
//   Measured against the vector kernels (45 x 45 x 1950 table unless said): sorted, 3000 segments 91.3 -> 8.5 ms; atomic,
// 800 segments 50 -> 2.8 ms; one track on 20 x 31 x 1001 1.106 -> 0.073 ms, 64 such tracks 9.2 -> 1.23.
// Error against 64 bits, relative to all currents 1.7e-6 -> 1.5e-7, 9.5e-7 -> 1.4e-7 atomic; of a pixel relative to itself,
// median and largest, 2.3e-6 and 1.0e-5 -> 1.2e-7 and 1.3e-6, a track's 4e-7 and 2.1e-6 -> 1.3e-7 and 7.8e-7.  (With one
// scale for a group, 1 % less time, pixels that only the clouds' tails reach were off by up to 3e-3.)
constexpr int32_t kZgSegs = 16;                         // segments of a group
constexpr int32_t kZgSpan = 128;                        // ticks of a group's charge (unless one segment has more)
constexpr int32_t kZgTicks = 32;                        // ticks and octets staged at a time
constexpr int32_t kZgOct = 32;
constexpr int32_t kZgTop = 127 + 14;                    // biased exponent of a tick's largest scaled charge: below 2^15

struct ZTable {                                         // half planes of the table by octets of bins
    const u32x4 *hi, *lo;                               // [bx * njo][trq]: 8 halves
    const int32_t *exps;                                // [bx * by] scale of a bin
    int32_t njo, trq;
};

struct ZSeg {                                           // a segment of the group, as the staging reads it
    int64_t cells;
    int32_t u0, nu, v0, nv, a0, na, nap, _pad;
};

// One mirror image of a segment's charge box in the pixel's folded bins: the charge of bin (i, j), i0 <= i <= i1 and
// j0 <= j <= j1, at tick a of the box is at byte base + i si + j sj + 4 a of the segment's cells (`bytes` of them).
struct ZJob {
    int64_t cells;
    int32_t bytes, base, si, sj, i0, i1, j0, j1, a0, na;
};

struct alignas(16) ZStage {
    u32x4 c[2][2][kZgOct][16];                          // [plane][16 ticks][octet][tick]: 8 halves (4 FP32 values at first)
    i32x4 ex[kZgOct][2];                                // scales of an octet's bins
    int32_t top[2][kZgTicks];                           // [stage & 1][tick]: largest exponent of charge x column scale
    ZSeg seg[kZgSegs];
    ZJob job[4 * kZgSegs];
    uint32_t at[kZgOct];                                // byte offset of an octet's table column
};

__global__ __launch_bounds__(kWG) void k_table_octets(const float *__restrict__ Rpad, int32_t col_len, int32_t t_r,
                                                      int32_t by, int32_t njo, int32_t trq,
                                                      const int32_t *__restrict__ exps, u32x4 *__restrict__ hi,
                                                      u32x4 *__restrict__ lo) {
    const int32_t o = blockIdx.x, i = o / njo, j0 = (o - i * njo) * 8;
    for (int32_t t = threadIdx.x; t < trq; t += kWG) {
        half8 h, l;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float x = 0.0f;
            if (j0 + q < by && t < t_r) {
                const int32_t b = i * by + j0 + q;
                x = ldexpf(Rpad[(int64_t)b * col_len + kPad + t], exps[b]);
            }
            h[q] = (_Float16)x;
            l[q] = (_Float16)(x - (float)h[q]);
        }
        hi[(int64_t)o * trq + t] = __builtin_bit_cast(u32x4, h);
        lo[(int64_t)o * trq + t] = __builtin_bit_cast(u32x4, l);
    }
}

void launch_table_octets(const float *Rpad, int32_t bx, int32_t by, int32_t t_r, int32_t col_len, int32_t trq,
                         const int32_t *exps, void *hi, void *lo, hipStream_t st) {
    const int32_t njo = (by + 7) / 8;
    k_table_octets<<<(unsigned)(bx * njo), kWG, 0, st>>>(Rpad, col_len, t_r, by, njo, trq, exps, (u32x4 *)hi, (u32x4 *)lo);
}

template <int R>
__device__ __forceinline__ float row_up(float x) {       // lane j of a row of 16 takes lane j - R's value, 0 below
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x110 + R, 0xf, 0xf, true));
}
template <int R>
__device__ __forceinline__ float row_down(float x) {     // lane j of a row of 16 takes lane j + R's value, 0 above
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x100 + R, 0xf, 0xf, true));
}
// Sum over the four rows of 16 lanes, in every row: two copies of y exchange their halves, then their odd and even rows
// (a wait of two states between a register's write and a swap of it).
__device__ __forceinline__ float rows_sum(float y) {
    float z = y;
    asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(y), "+v"(z));
    y += z;
    z = y;
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(y), "+v"(z));
    return y + z;
}

// Z tiles t and t + 1 of the staged octets (KN steps of four octets; steps past the staged ones meet zero charge).
template <int KN, bool TWO>
__device__ __forceinline__ void z_tiles(const ZStage &st, __amdgpu_buffer_rsrc_t rh, __amdgpu_buffer_rsrc_t rl,
                                        uint32_t f0, uint32_t f1, int lj, int lg, floatx4 (&D)[2][2]) {
    u32x4 h0[KN], l0[KN], h1[KN], l1[KN];
#pragma unroll
    for (int k = 0; k < KN; ++k) {                      // all loads first: they come from L2 or beyond
        const uint32_t at = st.at[4 * k + lg] + 16u * (uint32_t)lj;
        h0[k] = __builtin_amdgcn_raw_buffer_load_b128(rh, at, f0, 0);
        l0[k] = __builtin_amdgcn_raw_buffer_load_b128(rl, at, f0, 0);
        h1[k] = __builtin_amdgcn_raw_buffer_load_b128(rh, at, f1, 0);
        l1[k] = __builtin_amdgcn_raw_buffer_load_b128(rl, at, f1, 0);
    }
#pragma unroll
    for (int k = 0; k < KN; ++k)
#pragma unroll
        for (int b = 0; b < (TWO ? 2 : 1); ++b) {
            const half8 ah = __builtin_bit_cast(half8, st.c[0][b][4 * k + lg][lj]);
            const half8 al = __builtin_bit_cast(half8, st.c[1][b][4 * k + lg][lj]);
            const half8 p0 = __builtin_bit_cast(half8, h0[k]), p1 = __builtin_bit_cast(half8, h1[k]);
            D[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, p0, D[b][0], 0, 0, 0);
            D[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, p1, D[b][1], 0, 0, 0);
            D[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, p0, D[b][0], 0, 0, 0);
            D[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, p1, D[b][1], 0, 0, 0);
            D[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, __builtin_bit_cast(half8, l0[k]), D[b][0], 0, 0, 0);
            D[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, __builtin_bit_cast(half8, l1[k]), D[b][1], 0, 0, 0);
        }
}
template <bool TWO>
__device__ __forceinline__ void z_dispatch(int32_t nk, const ZStage &st, __amdgpu_buffer_rsrc_t rh,
                                           __amdgpu_buffer_rsrc_t rl, uint32_t f0, uint32_t f1, int lj, int lg,
                                           floatx4 (&D)[2][2]) {
    if (nk <= 2) z_tiles<2, TWO>(st, rh, rl, f0, f1, lj, lg, D);
    else if (nk <= 4) z_tiles<4, TWO>(st, rh, rl, f0, f1, lj, lg, D);
    else if (nk <= 6) z_tiles<6, TWO>(st, rh, rl, f0, f1, lj, lg, D);
    else z_tiles<8, TWO>(st, rh, rl, f0, f1, lj, lg, D);
}

// Adds the current of the group st.seg[0 .. n_seg) on the pixel with centre bins (uc, vc) through emit(n, value), n in
// [0, n_ticks), called by 32 lanes at a time, never for the same n by two wavefronts between barriers.  All threads of the
// workgroup call it; it starts and ends with a barrier.
template <int WG, class Emit>
__device__ __forceinline__ void z_group(const DevParams &P, const ZTable &Z, ZStage &st, int32_t n_seg, int32_t A0,
                                        int32_t A1, int32_t uc, int32_t vc, const float *__restrict__ cells, Emit emit) {
    const int tid = threadIdx.x, lane = tid & 63, lj = lane & 15, lg = lane >> 4;
    const int32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t TR = P.t_r, NT = P.nticks, n_tau = Z.trq / 16;
    const int32_t plane = P.bx * Z.njo * Z.trq * 16;    // bytes (at most 2^30)
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc((void *)Z.hi, (short)0, plane, kBufferWord3);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void *)Z.lo, (short)0, plane, kBufferWord3);
    constexpr int32_t kNone = -(1 << 24);               // exponent of a tick without charge
    int32_t par = 0;                                    // the stage's half of st.top
    if (tid < 2 * kZgTicks) (&st.top[0][0])[tid] = kNone;
    __syncthreads();                                    // the group's segments are in place
    for (int32_t ac = A0; ac <= A1; ac += kZgTicks) {
        const int32_t n0 = ac - TR + 1;                 // tick of output 0
        if (n0 >= NT || min(ac + kZgTicks - 1, A1) < 0) continue;
        // the mirror images with charge in these ticks (lane = image of a segment; every wavefront finds the same, in
        // the order segment, u side, v side), and the octets they span
        ZJob jb{0, 0, 0, 0, 0, 0, -1, 0, -1, 0, 0};
        int32_t alast = -1;
        if (lane < 4 * n_seg) {
            const ZSeg g = st.seg[lane >> 2];
            const int32_t su = lane >> 1 & 1, sv = lane & 1;
            // bins of the image: u = uc + i (or uc - 1 - i), 0 <= i < bx
            jb.i0 = max(su ? uc - 1 - (g.u0 + g.nu - 1) : g.u0 - uc, 0);
            jb.i1 = min(su ? uc - 1 - g.u0 : g.u0 + g.nu - 1 - uc, P.bx - 1);
            jb.j0 = max(sv ? vc - 1 - (g.v0 + g.nv - 1) : g.v0 - vc, 0);
            jb.j1 = min(sv ? vc - 1 - g.v0 : g.v0 + g.nv - 1 - vc, P.by - 1);
            jb.cells = g.cells;
            jb.bytes = g.nu * g.nv * g.nap * 4;
            jb.si = (su ? -4 : 4) * g.nv * g.nap;
            jb.sj = (sv ? -4 : 4) * g.nap;
            jb.base = (((su ? uc - 1 : uc) - g.u0) * g.nv + ((sv ? vc - 1 : vc) - g.v0)) * g.nap * 4;
            jb.a0 = g.a0;
            jb.na = g.na;
            if (!(g.a0 > ac + kZgTicks - 1 || g.a0 + g.na <= ac)) alast = min(g.a0 + g.na - 1 - ac, kZgTicks - 1);
        }
        const bool has = alast >= 0 && jb.i0 <= jb.i1 && jb.j0 <= jb.j1;
        const uint64_t jobs = __ballot(has);
        if (!jobs) continue;
        const int32_t n_job = __builtin_popcountll(jobs);
        int32_t i0 = has ? jb.i0 : INT32_MAX, i1 = has ? jb.i1 : -1, j0 = has ? jb.j0 : INT32_MAX, j1 = has ? jb.j1 : -1;
        if (!has) alast = -1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            i0 = min(i0, __shfl_xor(i0, o));
            i1 = max(i1, __shfl_xor(i1, o));
            j0 = min(j0, __shfl_xor(j0, o));
            j1 = max(j1, __shfl_xor(j1, o));
            alast = max(alast, __shfl_xor(alast, o));
        }
        i0 = __builtin_amdgcn_readfirstlane(i0);
        i1 = __builtin_amdgcn_readfirstlane(i1);
        j0 = __builtin_amdgcn_readfirstlane(j0);
        j1 = __builtin_amdgcn_readfirstlane(j1);
        alast = __builtin_amdgcn_readfirstlane(alast);
        if (wv == 0 && has) st.job[__builtin_popcountll(jobs & ((1ull << lane) - 1ull))] = jb;
        const int32_t jo0 = j0 / 8, nj = j1 / 8 - jo0 + 1, n_oct = (i1 - i0 + 1) * nj;
        const bool two = alast >= 16;
        // this wavefront's output tiles of 16 ticks
        const int32_t m_first = max(-n0, 0) / 16, m_last = min(TR + alast - 1, NT - 1 - n0) / 16;
        // (an even number: which tiles pair up, and so the order of the sums, must not depend on the wavefronts)
        const int32_t per = ((m_last - m_first + WG / 64) / (WG / 64) + 1) & ~1;
        const int32_t m_lo = m_first + wv * per, m_hi = min(m_lo + per, m_last + 1);
        __syncthreads();                                // the images are in place
        for (int32_t o0 = 0; o0 < n_oct; o0 += kZgOct, par ^= 1) {
            const int32_t no = min(kZgOct, n_oct - o0), nk = (no + 3) / 4, nq = nk <= 2 ? 8 : nk <= 4 ? 16 : nk <= 6 ? 24 : 32;
            // stage: thread (tick, octet) sums its eight bins over the images, in order
            const int32_t a = tid & 31;
            int32_t most = kNone;
            for (int32_t q = tid >> 5; q < nq; q += WG / 32) {
                const int32_t o = o0 + min(q, no - 1), ii = o / nj;
                const int32_t i = i0 + ii, jo = jo0 + o - ii * nj, jb0 = jo * 8;
                if (a == 0) st.at[q] = (uint32_t)((i * Z.njo + jo) * Z.trq) * 16u;
                float c[8];
                int32_t ex[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    c[k] = 0.0f;
                    ex[k] = Z.exps[i * P.by + min(jb0 + k, P.by - 1)];
                }
                // the images with a bin in one of the wavefront's two octets
                bool near = false;
                if (lane < n_job) {
                    const ZJob &g = st.job[lane];
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const int32_t iw = __builtin_amdgcn_readlane(i, 32 * w), jw = __builtin_amdgcn_readlane(jb0, 32 * w);
                        near |= iw >= g.i0 && iw <= g.i1 && jw + 7 >= g.j0 && jw <= g.j1;
                    }
                }
                uint64_t mask = __ballot(near);
                // adds the next kImg images (in order) to c, all their loads in flight at once
                auto add = [&](auto kImg) {
                    uint32_t x[kImg.value][8];
#pragma unroll
                    for (int w = 0; w < kImg.value; ++w) {
                        const bool any = mask != 0;
                        const ZJob &g = st.job[any ? __builtin_ctzll(mask) : 0];
                        mask &= mask - 1ull;
                        const int32_t al = ac + a - g.a0;
                        // bits of the octet's bins that are not in the image; their loads go past the box and return 0
                        uint32_t out = ~0u;
                        if (q < no && any && al >= 0 && al < g.na && i >= g.i0 && i <= g.i1)
                            out = ~(~0u << min(max(g.j0 - jb0, 0), 8)) | ~0u << min(max(g.j1 - jb0 + 1, 0), 8);
                        const int32_t at = g.base + i * g.si + jb0 * g.sj + 4 * al, sj = g.sj;
                        const int64_t box = uniform_i64((int64_t)(cells + g.cells), 0);
                        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
                            (void *)box, (short)0, __builtin_amdgcn_readfirstlane(g.bytes), kBufferWord3);
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            x[w][k] = __builtin_amdgcn_raw_buffer_load_b32(
                                rc, (uint32_t)(at + k * sj) | (uint32_t)((int32_t)(out << (31 - k)) >> 31), 0, 0);
                    }
#pragma unroll
                    for (int w = 0; w < kImg.value; ++w)
#pragma unroll
                        for (int k = 0; k < 8; ++k) c[k] += __builtin_bit_cast(float, x[w][k]);
                };
                while (mask) {
                    if (__builtin_popcountll(mask) > 4) add(std::integral_constant<int, 8>());
                    else add(std::integral_constant<int, 4>());
                }
                st.c[0][a >> 4][q][a & 15] = __builtin_bit_cast(u32x4, (floatx4){c[0], c[1], c[2], c[3]});
                st.c[1][a >> 4][q][a & 15] = __builtin_bit_cast(u32x4, (floatx4){c[4], c[5], c[6], c[7]});
                if (a == 0) {
                    st.ex[q][0] = (i32x4){ex[0], ex[1], ex[2], ex[3]};
                    st.ex[q][1] = (i32x4){ex[4], ex[5], ex[6], ex[7]};
                }
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    most = max(most, c[k] == 0.0f ? kNone : (__builtin_bit_cast(int32_t, fabsf(c[k])) >> 23) - ex[k]);
            }
            most = max(most, __shfl_xor(most, 32));
            if (lane < 32) atomicMax(&st.top[par][a], most);
            __syncthreads();                            // the ticks' exponents are complete
            if (tid < kZgTicks) st.top[par ^ 1][tid] = kNone;
            // the halves, in place
            const int32_t N = kZgTop - st.top[par][a];
            for (int32_t q = tid >> 5; q < nq; q += WG / 32) {
                const i32x4 e0 = st.ex[q][0], e1 = st.ex[q][1];
                const floatx4 c0 = __builtin_bit_cast(floatx4, st.c[0][a >> 4][q][a & 15]);
                const floatx4 c1 = __builtin_bit_cast(floatx4, st.c[1][a >> 4][q][a & 15]);
                half8 h, l;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float y = k < 4 ? ldexpf(c0[k & 3], N - e0[k & 3]) : ldexpf(c1[k & 3], N - e1[k & 3]);
                    h[k] = (_Float16)y;
                    l[k] = (_Float16)(y - (float)h[k]);
                }
                st.c[0][a >> 4][q][a & 15] = __builtin_bit_cast(u32x4, h);
                st.c[1][a >> 4][q][a & 15] = __builtin_bit_cast(u32x4, l);
            }
            __syncthreads();
            if (m_lo < m_hi) {
                int32_t dn[2][4];                       // the lane's rows' scales
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) dn[b][r] = st.top[par][16 * b + 4 * lg + r] - kZgTop;
                float O[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                for (int32_t t = m_lo - 2; t < m_hi; t += 2) {
                    const bool v0 = t >= 0 && t < n_tau, v1 = t + 1 >= 0 && t + 1 < n_tau;
                    if (v0 || v1) {
                        floatx4 D[2][2];
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int y = 0; y < 2; ++y) D[b][y] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
                        const uint32_t f0 = (uint32_t)min(max(t, 0), n_tau - 1) * 256u;
                        const uint32_t f1 = (uint32_t)min(max(t + 1, 0), n_tau - 1) * 256u;
                        if (two) z_dispatch<true>(nk, st, rh, rl, f0, f1, lj, lg, D);
                        else z_dispatch<false>(nk, st, rh, rl, f0, f1, lj, lg, D);
                        // anti-diagonals: tile y of rows b goes to output tiles t + y + b (lo) and the next one (hi)
#pragma unroll
                        for (int b = 0; b < 2; ++b)
#pragma unroll
                            for (int y = 0; y < 2; ++y) {
                                if ((b == 1 && !two) || !(y ? v1 : v0)) continue;
                                floatx4 d;
#pragma unroll
                                for (int r = 0; r < 4; ++r) d[r] = ldexpf(D[b][y][r], dn[b][r]);
                                // (charge that is not finite is no number against the padding past the table's end)
                                if (t + y == n_tau - 1 && 16 * (t + y) + lj >= TR) d = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
                                const float lo = d[0] + row_up<1>(d[1]) + (row_up<2>(d[2]) + row_up<3>(d[3]));
                                const float hi = row_down<15>(d[1]) + (row_down<14>(d[2]) + row_down<13>(d[3]));
                                // row g moves up by 4 g more
                                const float l4 = row_up<4>(lo), l8 = row_up<8>(lo), l12 = row_up<12>(lo);
                                O[y + b] += lg == 0 ? lo : lg == 1 ? l4 : lg == 2 ? l8 : l12;
                                const float s12 = row_down<12>(lo) + row_up<4>(hi), s8 = row_down<8>(lo) + row_up<8>(hi);
                                const float s4 = row_down<4>(lo) + row_up<12>(hi);
                                O[y + b + 1] += lg == 0 ? hi : lg == 1 ? s12 : lg == 2 ? s8 : s4;
                            }
                    }
                    const float y0 = rows_sum(O[0]), y1 = rows_sum(O[1]);
                    const int32_t m = t + (lg & 1), n = n0 + 16 * m + lj;
                    if (lane < 32 && m >= m_lo && m < m_hi && n >= 0 && n < NT) emit(n, lg ? y1 : y0);
                    O[0] = O[2];
                    O[1] = O[3];
                    O[2] = O[3] = 0.0f;
                }
            }
            __syncthreads();
        }
    }
}

// Loads the group that starts at list entry q of [q, end) into st.seg: the longest run of at most kZgSegs entries whose
// ticks span at most kZgSpan (one entry at least).  id(k) is entry k's segment.  Every wavefront finds the same group;
// the first one writes it.  Returns its length; [A0, A1] its ticks (A1 < A0: no charge).
template <class Id>
__device__ __forceinline__ int32_t z_load_group(const DevParams &P, const SegInfo *__restrict__ si, int64_t q, int64_t end,
                                                int32_t uc, int32_t vc, Id id, ZStage &st, int32_t &A0, int32_t &A1) {
    const int lane = lane_id();
    const int32_t cnt = (int32_t)min<int64_t>(kZgSegs, end - q);
    ZSeg z{0, 0, 0, 0, 0, INT32_MAX, 0, 0, 0};
    int32_t lo = INT32_MAX, hi = INT32_MIN;
    if (lane < cnt) {
        const SegInfo &g = si[id(q + lane)];
        const bool any = max(g.u0, uc - P.bx) <= min(g.u0 + g.nu - 1, uc + P.bx - 1) &&
                         max(g.v0, vc - P.by) <= min(g.v0 + g.nv - 1, vc + P.by - 1);
        if (any && !(g.flags & (SEG_INVALID | SEG_TOO_LONG))) {
            z = ZSeg{g.cell_off, g.u0, g.nu, g.v0, g.nv, g.a0, g.na, g.na_pad, 0};
            lo = g.a0;
            hi = g.a0 + g.na - 1;
        }
    }
#pragma unroll
    for (int d = 1; d < kZgSegs; d <<= 1) {              // running span over the entries
        const int32_t x = __shfl_up(lo, d), y = __shfl_up(hi, d);
        if (lane >= d) {
            lo = min(lo, x);
            hi = max(hi, y);
        }
    }
    const bool fits = lane < cnt && (lane == 0 || (int64_t)hi - lo < kZgSpan);
    const int32_t n = __builtin_ctzll(~__ballot(fits));  // the entries that fit are a prefix
    A0 = __builtin_amdgcn_readlane(lo, n - 1);
    A1 = __builtin_amdgcn_readlane(hi, n - 1);
    if (threadIdx.x < 64 && lane < n) st.seg[lane] = z;
    return n;
}

// Sorted variant (automatic choice): one workgroup per active pixel, its segments in ascending id, group by group; the
// groups' currents go into the pixel's waveform in LDS with Kahan compensation.
template <int WG>
__global__ __launch_bounds__(WG, 512 / WG) void k_induce_z(DevParams P, ZTable Z, const SegInfo *__restrict__ si,
                                                  const float *__restrict__ cells, const int64_t *__restrict__ slot_off,
                                                  const int32_t *__restrict__ pairs, const int32_t *__restrict__ slot_gp,
                                                  const int32_t *__restrict__ order, float *__restrict__ wave,
                                                  DevHeader *H) {
    extern __shared__ float sm[];
    __shared__ ZStage st;
    __shared__ int32_t s_slot;
    const int NT = P.nticks, tid = threadIdx.x;
    float *s_sum = sm, *s_cmp = sm + NT;
    const int64_t n_slots = H->n_slots;
    for (;;) {
        if (tid == 0) s_slot = (int32_t)atomicAdd(&H->work[0], 1u);
        __syncthreads();
        const int32_t got = __builtin_amdgcn_readfirstlane(s_slot);
        if (got >= n_slots) break;
        const int64_t slot = order ? order[got] : got;
        for (int n = tid; n < NT; n += WG) { s_sum[n] = 0.0f; s_cmp[n] = 0.0f; }
        const int32_t p = slot_gp[slot] % P.npx;
        const int32_t uc = (p % P.nx) * P.nsub + P.nsub / 2, vc = (p / P.nx) * P.nsub + P.nsub / 2;
        const int64_t pe = slot_off[slot + 1];
        for (int64_t q = slot_off[slot]; q < pe;) {
            int32_t A0, A1;
            const int32_t n = z_load_group(P, si, q, pe, uc, vc, [&](int64_t k) { return pairs[k]; }, st, A0, A1);
            z_group<WG>(P, Z, st, n, A0, A1, uc, vc, cells, [&](int32_t t, float x) {
                const float y = x - s_cmp[t], z = s_sum[t] + y;
                s_cmp[t] = (z - s_sum[t]) - y;
                s_sum[t] = z;
            });
            __syncthreads();                            // before the next group's segments
            q += n;
        }
        float *wrow = wave + slot * NT;
        for (int n = tid; n < NT; n += WG) wrow[n] = s_sum[n] - s_cmp[n];
        __syncthreads();
    }
}

// Atomic variant (automatic choice): the same group products with FP32 atomics.  A work unit is a block of kZaSegs
// consecutive segments and every 16th pixel row of their reach; runs of its segments of one event that lie close together
// form the groups.
constexpr int32_t kZaSegs = 8, kZaRows = 16;
__global__ __launch_bounds__(kWG, 2) void k_induce_z_atomic(DevParams P, ZTable Z, const SegInfo *__restrict__ si,
                                                         int64_t n_seg, const float *__restrict__ cells,
                                                         const int32_t *__restrict__ pix_slot, float *wave,
                                                         DevHeader *H) {
    __shared__ ZStage st;
    __shared__ int32_t s_unit;
    const int NT = P.nticks, tid = threadIdx.x, lane = tid & 63;
    const int64_t n_units = (n_seg + kZaSegs - 1) / kZaSegs * kZaRows;
    for (;;) {
        if (tid == 0) s_unit = (int32_t)atomicAdd(&H->work[1], 1u);
        __syncthreads();
        const int64_t unit = __builtin_amdgcn_readfirstlane(s_unit);
        __syncthreads();
        if (unit >= n_units) break;
        const int64_t blk = unit / kZaRows, end = min(n_seg, (blk + 1) * kZaSegs);
        const int32_t row = (int32_t)(unit - blk * kZaRows);
        for (int64_t q = blk * kZaSegs; q < end;) {
            // the group: entries q .. of one event whose ticks span at most kZgSpan and whose union of pixel rectangles is
            // at most twice the largest one (every wavefront finds the same)
            const int32_t cnt = (int32_t)(end - q);
            ZSeg z{0, 0, 0, 0, 0, INT32_MAX, 0, 0, 0};
            int32_t lo = INT32_MAX, hi = INT32_MIN, x0 = INT32_MAX, x1 = -1, y0 = INT32_MAX, y1 = -1, area = 0, ev = -1;
            if (lane < cnt) {
                const SegInfo &g = si[q + lane];
                ev = g.event;
                if (g.n_pairs > 0) {
                    z = ZSeg{g.cell_off, g.u0, g.nu, g.v0, g.nv, g.a0, g.na, g.na_pad, 0};
                    lo = g.a0;
                    hi = g.a0 + g.na - 1;
                    x0 = g.ix0; x1 = g.ix1; y0 = g.iy0; y1 = g.iy1;
                    area = g.n_pairs;
                }
            }
            const bool same = ev == __builtin_amdgcn_readlane(ev, 0);
#pragma unroll
            for (int d = 1; d < kZaSegs; d <<= 1) {
                const int32_t a = __shfl_up(lo, d), b = __shfl_up(hi, d), c = __shfl_up(x0, d), e = __shfl_up(x1, d);
                const int32_t f = __shfl_up(y0, d), h = __shfl_up(y1, d), k = __shfl_up(area, d);
                if (lane >= d) {
                    lo = min(lo, a); hi = max(hi, b); x0 = min(x0, c); x1 = max(x1, e); y0 = min(y0, f); y1 = max(y1, h);
                    area = max(area, k);
                }
            }
            const bool fits = lane < cnt && (lane == 0 || (same && (int64_t)hi - lo < kZgSpan &&
                                                           (int64_t)(x1 - x0 + 1) * (y1 - y0 + 1) <= 2ll * area));
            const uint64_t out = ~__ballot(fits);
            const int32_t n = __builtin_ctzll(out);
            const int32_t A0 = __builtin_amdgcn_readlane(lo, n - 1), A1 = __builtin_amdgcn_readlane(hi, n - 1);
            const int32_t gx0 = __builtin_amdgcn_readlane(x0, n - 1), gx1 = __builtin_amdgcn_readlane(x1, n - 1);
            const int32_t gy0 = __builtin_amdgcn_readlane(y0, n - 1), gy1 = __builtin_amdgcn_readlane(y1, n - 1);
            const int32_t e = __builtin_amdgcn_readlane(ev, 0);
            q += n;
            if (gx0 > gx1 || gy0 > gy1) continue;       // segments that reach no pixel: no rectangle to walk
            __syncthreads();                            // the previous group's segments are no longer read
            if (tid < n) st.seg[tid] = z;
            for (int32_t iy = gy0 + row; iy <= gy1; iy += kZaRows)
                for (int32_t ix = gx0; ix <= gx1; ++ix) {
                    const int32_t slot = __builtin_amdgcn_readfirstlane(pix_slot[(int64_t)e * P.npx + iy * P.nx + ix]);
                    if (slot < 0) continue;
                    float *wrow = wave + (int64_t)slot * NT;
                    z_group<kWG>(P, Z, st, n, A0, A1, ix * P.nsub + P.nsub / 2, iy * P.nsub + P.nsub / 2, cells,
                            [&](int32_t t, float x) {
                                if (x != 0.0f) atomicAdd(&wrow[t], x);
                            });
                }
        }
    }
}

// Materialised form: row q of `out` (n_ticks floats) receives pair q's current, one pair at a time.
__global__ __launch_bounds__(kWG, 2) void k_induce_z_pairs(DevParams P, ZTable Z, const SegInfo *__restrict__ si,
                                                        const float *__restrict__ cells,
                                                        const int64_t *__restrict__ slot_off,
                                                        const int32_t *__restrict__ pairs,
                                                        const int32_t *__restrict__ slot_gp, const DevHeader *H,
                                                        float *__restrict__ out) {
    extern __shared__ float sm[];
    __shared__ ZStage st;
    const int NT = P.nticks, tid = threadIdx.x;
    for (int n = tid; n < NT; n += kWG) sm[n] = 0.0f;
    for (int64_t slot = blockIdx.x; slot < H->n_slots; slot += gridDim.x) {
        const int32_t p = slot_gp[slot] % P.npx;
        const int32_t uc = (p % P.nx) * P.nsub + P.nsub / 2, vc = (p / P.nx) * P.nsub + P.nsub / 2;
        for (int64_t q = slot_off[slot]; q < slot_off[slot + 1]; ++q) {
            int32_t A0, A1;
            z_load_group(P, si, q, q + 1, uc, vc, [&](int64_t k) { return pairs[k]; }, st, A0, A1);
            z_group<kWG>(P, Z, st, 1, A0, A1, uc, vc, cells, [&](int32_t t, float x) { sm[t] += x; });
            __syncthreads();
            float *row = out + q * NT;
            for (int n = tid; n < NT; n += kWG) {
                row[n] = sm[n];
                sm[n] = 0.0f;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------ charge outside the readout
// The signed induction that falls outside [0, n_ticks), from FP64 prefix sums of the table columns.  Charge in column
// (u, v) at tick a induces on every pixel that reaches the column, and only the sum over an event's pixels is reported, so
// the pixels' prefix sums are added first: for a column whose reaching pixels all lie on the grid they depend only on its
// offset within a pixel (a class of n_sub^2, summed when the table is installed); at the grid's edge the pixels are
// walked.
__global__ __launch_bounds__(kWG) void k_clip_classes(DevParams P, const double *__restrict__ prefix,
                                                      double *__restrict__ cls) {
    const int32_t c = blockIdx.x, ru = c / P.nsub, rv = c - ru * P.nsub, h = P.nsub / 2, n = P.t_r + 1;
    auto first = [&](int32_t r, int32_t b) { return -b + ((r - h + b) % P.nsub + P.nsub) % P.nsub; };
    for (int32_t k = threadIdx.x; k < n; k += kWG) {
        double s = 0.0;
        for (int32_t du = first(ru, P.bx); du < P.bx; du += P.nsub)
            for (int32_t dv = first(rv, P.by); dv < P.by; dv += P.nsub)
                s += prefix[(int64_t)(fold(du) * P.by + fold(dv)) * n + k];
        cls[(int64_t)c * n + k] = s;
    }
}

void launch_clip_classes(const DevParams &P, const double *prefix, double *cls, hipStream_t st) {
    k_clip_classes<<<(unsigned)(P.nsub * P.nsub), kWG, 0, st>>>(P, prefix, cls);
}

// Dropped induction of unit charge in column (u, v) at tick a, summed over the pixels that reach the column.
__device__ __forceinline__ double clip_weight(const DevParams &P, const double *__restrict__ prefix,
                                              const double *__restrict__ cls, int32_t u, int32_t v, int32_t a) {
    const int32_t T = P.t_r, h = P.nsub / 2, n = T + 1;
    const int32_t klo = min(max(T - 1 - a, 0), T);                 // first kept table tick
    const int32_t khi = min(max(P.nticks + T - 1 - a, 0), T);      // one past the last kept tick
    if (klo == 0 && khi == T) return 0.0;
    auto dropped = [&](const double *p) { return klo >= khi ? p[T] : p[klo] + (p[T] - p[khi]); };
    const int32_t xa = ceil_div(u - h - P.bx + 1, P.nsub), xb = floor_div(u - h + P.bx, P.nsub);
    const int32_t ya = ceil_div(v - h - P.by + 1, P.nsub), yb = floor_div(v - h + P.by, P.nsub);
    if (cls && xa >= 0 && xb < P.nx && ya >= 0 && yb < P.ny) {
        const int32_t ru = u - floor_div(u, P.nsub) * P.nsub, rv = v - floor_div(v, P.nsub) * P.nsub;
        return dropped(cls + (int64_t)(ru * P.nsub + rv) * n);
    }
    double s = 0.0;
    for (int32_t x = max(xa, 0); x <= min(xb, P.nx - 1); ++x)
        for (int32_t y = max(ya, 0); y <= min(yb, P.ny - 1); ++y)
            s += dropped(prefix + (int64_t)(fold(u - x * P.nsub - h) * P.by + fold(v - y * P.nsub - h)) * n);
    return s;
}

// Per-pair modes: over the segments' charge cells (a workgroup per segment).
__global__ __launch_bounds__(kWG) void k_clip_cells(DevParams P, const SegInfo *__restrict__ si, int64_t n_seg,
                                                    const float *__restrict__ cells, const double *__restrict__ prefix,
                                                    const double *__restrict__ cls, double *report) {
    __shared__ double red[kWG / 64];
    for (int64_t s = blockIdx.x; s < n_seg; s += gridDim.x) {
        const SegInfo &g = si[s];
        if (g.n_pairs == 0 || (g.a0 >= P.t_r - 1 && g.a0 + g.na <= P.nticks)) continue;
        const int32_t na = g.na, nv = g.nv, nap = g.na_pad;
        const float *c = cells + g.cell_off;
        double acc = 0.0;
        for (int32_t i = threadIdx.x; i < g.nu * nv * na; i += kWG) {
            const int32_t col = i / na, a = i - col * na, u = col / nv;
            const float q = c[(int64_t)col * nap + a];
            if (q != 0.0f) acc += (double)q * clip_weight(P, prefix, cls, g.u0 + u, g.v0 + col - u * nv, g.a0 + a);
        }
        const double t = block_sum_double(acc, red);
        if (threadIdx.x == 0 && t != 0.0) atomicAdd(&report[(int64_t)g.event * 5 + 3], t);
        __syncthreads();
    }
}

// Summed mode: over the column pieces (a wavefront per column at a time).
__global__ __launch_bounds__(kWG) void k_clip_columns(DevParams P, SumWork sw, const double *__restrict__ prefix,
                                                      const double *__restrict__ cls, double *report) {
    const int lane = threadIdx.x & 63;
    const uint32_t n_act = *sw.n_active, waves = gridDim.x * (kWG / 64);
    double acc = 0.0;
    int32_t ev = -1;
    auto flush = [&] {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (lane == 0 && acc != 0.0) atomicAdd(&report[(int64_t)ev * 5 + 3], acc);
        acc = 0.0;
    };
    for (uint32_t ia = blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); ia < n_act;
         ia += waves) {
        const int64_t cc = __builtin_amdgcn_readfirstlane(sw.active[ia]);
        const int32_t e = (int32_t)(cc / ((int64_t)sw.CU * sw.CV));
        const int64_t r = cc - (int64_t)e * sw.CU * sw.CV;
        const int32_t u = sw.UL + (int32_t)(r / sw.CV), v = sw.VL + (int32_t)(r % sw.CV);
        if (e != ev && ev >= 0) flush();
        ev = e;
        for (int64_t k = sw.piece_off[cc]; k < sw.piece_off[cc + 1]; ++k) {
            const PieceRef p = sw.pdesc[k];
            if (p.a0 >= P.t_r - 1 && p.a0 + p.na <= P.nticks) continue;
            const float *S = sw.S + (int64_t)p.cell8 * kAC;
            for (int32_t i = lane; i < p.na; i += 64)
                acc += (double)S[i] * clip_weight(P, prefix, cls, u, v, p.a0 + i);
        }
    }
    if (ev >= 0) flush();
}

static ZTable z_table(const Table &T) {
    return ZTable{(const u32x4 *)T.zhi, (const u32x4 *)T.zlo, T.exps, T.njo, T.trq};
}

// The grid's dynamic LDS may exceed 64 KB with the static stage: the limit is raised once per device.
hipError_t allow_z_lds() {
    const int most = 2 * 8000 * (int)sizeof(float);
    hipError_t e = hipFuncSetAttribute((const void *)k_induce_z<kWG>, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_induce_z<512>, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_induce_z_pairs, hipFuncAttributeMaxDynamicSharedMemorySize, most / 2);
    return e;
}

// Up to 8 pixels a CU those with the most groups keep the kernel running, and a workgroup of 512 threads takes them faster
// than two of 256 take two; with many more the two overlap staging and products.  Measured with 256 and 512 threads: 276
// pixels of a track 74 and 62 us, 663 of 1200 segments 4.2 and 3.2 ms, 2000 pixels 5.4 and 5.4; from 2100 to 2800 it is
// the event that decides, an even one 5.9 to 6.2 and 6.3 to 6.7, one with a crowded place 12.5 to 15.9 and 9.3 to 12.5; 3200
// pixels 8.0 and 8.6, 64 tracks' 12,400 1.18 and 1.68.
constexpr int64_t kZgWide = 2048;
void launch_induce_z(const DevParams &P, const Work &w, const Table &T, float *wave, int mode, int64_t n_slots,
                     hipStream_t st) {
    const ZTable Z = z_table(T);
    if (w.n_seg > 0) {
        const int64_t g = std::min<int64_t>(w.n_seg, 8192);
        k_clip_cells<<<(unsigned)g, kWG, 0, st>>>(P, w.si, w.n_seg, w.cells, T.prefix, T.cls, w.report);
    }
    if (mode == 0) {
        if (n_slots <= 0) return;
        // up to two workgroups a CU all pixels start at once, in any order
        const int32_t *order = n_slots > 512 ? w.order : nullptr;
        if (order) launch_slot_order(P, w, n_slots, st);
        const bool wide = n_slots <= kZgWide;
        auto *k = wide ? k_induce_z<512> : k_induce_z<kWG>;
        k<<<(unsigned)std::min<int64_t>(n_slots, 256 * 4), wide ? 512 : kWG, (size_t)2 * P.nticks * sizeof(float), st>>>(
            P, Z, w.si, w.cells, w.slot_off, w.pairs, w.slot_gp, order, wave, w.hdr);
    } else if (w.n_seg > 0) {
        const int64_t units = (w.n_seg + kZaSegs - 1) / kZaSegs * kZaRows;
        k_induce_z_atomic<<<(unsigned)std::min<int64_t>(units, 256 * 4), kWG, 0, st>>>(P, Z, w.si, w.n_seg, w.cells,
                                                                                      w.pix_slot, wave, w.hdr);
    }
}

void launch_induce_z_pairs(const DevParams &P, const Work &w, const Table &T, int64_t n_slots, float *out,
                           hipStream_t st) {
    if (n_slots <= 0) return;
    k_induce_z_pairs<<<(unsigned)std::min<int64_t>(n_slots, 65536), kWG, (size_t)P.nticks * sizeof(float), st>>>(
        P, z_table(T), w.si, w.cells, w.slot_off, w.pairs, w.slot_gp, w.hdr, out);
}

bool summed_matrix(int32_t rt, bool shift) { return rt == 0 && !shift; }
int32_t summed_align_res(const DevParams &P, int32_t rt, bool shift) {
    if (summed_matrix(rt, shift)) return -1;           // takes intervals at any tick
    return ((P.t_r - 1 + kPad) % 8 + 8) % 8;
}

// Largest-first order of the pixels for the summed induction (the same log-bucketed order as the per-pair kernel's;
// all tiles of a pixel stay together): work of a pixel = the cell-tick blocks of its pieces.
__global__ __launch_bounds__(kWG) void k_slot_work_summed(const PieceRef *__restrict__ rec,
                                                          const int64_t *__restrict__ list_off, int64_t n_slots,
                                                          int32_t *__restrict__ bucket, int32_t *__restrict__ hist) {
    const int lane = threadIdx.x & 63;                  // one wavefront per pixel, lanes over its records
    const int64_t slot = (int64_t)blockIdx.x * (kWG / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (slot >= n_slots) return;
    int64_t blocks = 0;                                 // an integer sum: the same in any order
    for (int64_t q = list_off[slot] + lane; q < list_off[slot + 1]; q += 64) blocks += (rec[q].na + kAC - 1) / kAC;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) blocks += __shfl_xor(blocks, o);
    if (lane == 0) {
        const double work = (double)blocks;
        const int32_t lg = work >= 1.0 ? (int32_t)(16.0 * log2(work)) : 0;
        const int32_t b = kOrderBuckets - 1 - min(lg, kOrderBuckets - 1);
        bucket[slot] = b;
        atomicAdd(&hist[b], 1);
    }
}

const int32_t *launch_summed_order(const Work &w, const SumWork &sw, int64_t n_slots, int32_t rt, bool shift,
                                   hipStream_t st) {
    if ((rt != 0 && rt != 8) || n_slots <= 0 || !w.order || shift) return nullptr;
    int32_t *ord = w.order, *bucket = ord + n_slots, *hist = bucket + n_slots, *cursor = hist + kOrderBuckets;
    launch_zero(hist, (int64_t)sizeof(int32_t) * kOrderBuckets, st);
    const unsigned gs = (unsigned)((n_slots + kWG - 1) / kWG);
    k_slot_work_summed<<<(unsigned)((n_slots + kWG / 64 - 1) / (kWG / 64)), kWG, 0, st>>>(sw.mrec, sw.mlist_off, n_slots,
                                                                                         bucket, hist);
    k_order_offsets<<<1, kWG, 0, st>>>(hist, cursor);
    k_order_scatter<<<gs, kWG, 0, st>>>(bucket, n_slots, cursor, ord);
    return ord;
}

void launch_induce_summed(const DevParams &P, const Work &w, const SumWork &sw, const Table &T, float *wave,
                          int64_t n_slots, int32_t rt, bool shift, const int32_t *order, hipStream_t st) {
    if (rt != 0 && rt != 8) {                           // the per-pair kernel on the summed pieces (tuning option)
        Work ws = w;
        ws.si = sw.piece;
        ws.cells = sw.S;
        ws.slot_off = sw.list_off;
        ws.pairs = sw.list;
        launch_induce(P, ws, T, wave, 0, n_slots, rt, false, st);
        return;
    }
    if (n_slots <= 0) return;
    if (summed_matrix(rt, shift)) {
        k_clip_columns<<<256 * 4, kWG, 0, st>>>(P, sw, T.prefix, T.cls, w.report);
        const int64_t units = n_slots * ((P.nticks + kMmaUnit - 1) / kMmaUnit);
        const int64_t g = std::min<int64_t>((units + kWG / 64 - 1) / (kWG / 64), 256 * 4);
        k_induce_summed_mma<<<(unsigned)g, kWG, 0, st>>>(P, sw.S, sw.Sm, sw.nS8, (const u32x4 *)T.hi, (const u32x4 *)T.lo,
                                                         T.exps, sw.mlist_off, sw.mrec, order, wave, w.hdr);
        return;
    }
    const int64_t units = n_slots * ((P.nticks + kTileTicks - 1) / kTileTicks);
    const int64_t g = std::min<int64_t>((units + kWG / 64 - 1) / (kWG / 64), 256 * 8);
    if (shift)                                          // per piece (the list and the unmerged records)
        k_induce_summed<true><<<(unsigned)g, kWG, 0, st>>>(P, sw.piece, sw.S, sw.Sm, sw.nS8, T.Rpad, T.prefix,
                                                           sw.list_off, sw.list, sw.rec, order, w.slot_gp, wave,
                                                           w.hdr, w.report);
    else                                                // the merged records
        k_induce_summed<false><<<(unsigned)g, kWG, 0, st>>>(P, sw.piece, sw.S, sw.Sm, sw.nS8, T.Rpad, T.prefix,
                                                            sw.mlist_off, sw.list, sw.mrec, order, w.slot_gp, wave,
                                                            w.hdr, w.report);
}

// ================================================================================================= electronics
// Front-end electronics (Sec. 3.4), one wavefront per active pixel.  The per-tick rule: Q += I[n]; when no sample
// is pending and n >= ready, a crossing happens if Q + discriminator noise >= threshold; the sample is taken at
// max(n + hold, last + spacing) with uncorrelated noise added; ADC = clamp(floor(Q_s / q_lsb) + pedestal); the
// integrator restarts from the reset noise after the sample tick; a periodic reset applies before a tick's charge
// when no sample is pending.  The discriminator draw is skipped exactly when Q + |g|max * sigma_disc cannot reach
// the threshold.
//
// The walk goes in 64-tick chunks: the 64 lanes load a chunk at once, the charge and its absolute values since the
// segment start (the chunk start or the last reset) are prefix-summed across the lanes, and the events of the chunk
// (crossings, samples, resets) are found by ballots and handled in tick order; a lane's integrated charge is the
// value carried into the segment plus its prefix sum.  The carried value is a Kahan pair; a prefix sum over one
// segment of at most 64 ticks adds at most six roundings of its absolute sum, well inside the decision margin's
// relative term.  (One thread per pixel walking the ticks in order was 4.4x slower: too few wavefronts, and a
// dependent load per tick.)

// Most chunks have no event: no sample is due, no reset falls into them, and the carried charge plus the sum of the
// chunk's magnitudes stays below the threshold by more than the margins and any noise draw, or at least the 64 draws of
// the chunk.  Such a chunk needs only the two totals its last lane's prefix sums would hold, which the same tree of
// additions gives without a scan: every lane loads 4 ticks, 64 lanes four chunks, and a row of 16 lanes adds up a chunk.
// What bounds the kernel is its instructions, about 250 for a scanned chunk, 100 for one settled by its draws, 30 for one
// that needs none (15,000 pixels x 3000 ticks with 4 pulses and noise: 239 us, every chunk scanned 318; 250 pixels of a
// track 19 us, scanned 46).

// Value of the lane whose number is at / 4 (mod 64).
__device__ __forceinline__ float lane_from(int at, float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(at, __builtin_bit_cast(int, x)));
}

// Sum over the lane's row of 16, in every lane, paired as a prefix sum over its ticks pairs them.
__device__ __forceinline__ float row_tree(float x) {
    auto add = [&](auto c) {
        x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(c)::value, 0xf, 0xf,
                                                                true));
    };
    add(std::integral_constant<int, 0xB1>());            // lane ^ 1, lane ^ 2 (quads), the other quad, the other eight
    add(std::integral_constant<int, 0x4E>());
    add(std::integral_constant<int, 0x141>());
    add(std::integral_constant<int, 0x140>());
    return x;
}

// With `list` the pixels are the header's n_settle entries of it (a second pass over settled currents).  With `settle` a
// pixel one of whose decisions - a crossing, a code, or the margin that flags them - lies within twice the margin is
// appended to it, and its dropped and surplus samples and its current's sum are left to that pass.
template <bool SETTLE>
__global__ __launch_bounds__(kWG) void k_electronics(DevParams P, const float *__restrict__ wave,
                                                     const int32_t *__restrict__ slot_gp,
                                                     const uint64_t *__restrict__ ev_ids, int32_t n_ev,
                                                     const uint8_t *__restrict__ disabled, int64_t n_slots,
                                                     int32_t *pk_tick, uint16_t *pk_adc, uint8_t *pk_flag,
                                                     int64_t *pk_cnt, DevHeader *H, double *report,
                                                     int64_t *ev_cnt, const int32_t *__restrict__ list,
                                                     int32_t *settle) {
    const int64_t n_rows = list ? (int64_t)H->n_settle : n_slots;
    const int32_t NT = P.nticks, RP = P.reset_period;
    const int lane = lane_id();
    const int kWaves = blockDim.x / 64;
    const int32_t wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (int64_t row = (int64_t)blockIdx.x * kWaves + wv; row < n_rows; row += (int64_t)gridDim.x * kWaves) {
        const int64_t slot = list ? __builtin_amdgcn_readfirstlane(list[row]) : row;
        const int32_t gp = __builtin_amdgcn_readfirstlane(slot_gp[slot]);
        if (!(gp >= 0 && gp < n_ev * P.npx)) {                   // ids outside the event grids are skipped
            if (lane == 0) pk_cnt[slot] = 0;
            continue;
        }
        const int32_t e = gp / P.npx;
        const uint32_t pid = (uint32_t)(gp - e * P.npx);
        const bool off = disabled && disabled[pid];                   // disabled channel: no packets
        const uint64_t ev = ev_ids[e];
        const float *w = wave + slot * NT;
        const float disc_inv = P.sig_disc > 0.0f ? 1.0f / P.sig_disc : 0.0f;
        const float reset0 = P.sig_reset > 0.0f ? P.sig_reset * noise_normal(P, pid, kTickInitial, ev, STREAM_RESET)
                                                : 0.0f;
        float Qb = reset0, Qbc = 0.0f, Ab = 0.0f;                     // carried charge (Kahan pair) and |charge|
        bool pending = false, uncertain = false, done = off, close = false;
        int32_t ns = 0, ready = 0, last = -(1 << 28), cnt = 0, dropped = 0, over = 0;
        const int64_t obase = slot * P.max_packets;
        auto carry = [&](float q, float a) {                          // a segment's charge into the next chunk
            const float y = q - Qbc, t = Qb + y;
            Qbc = (t - Qb) - y;
            Qb = t;
            Ab += a;
        };
        double rs = 0.0;
        // four chunks at a time, lane l with ticks 4 l .. + 3 of them: row k of 16 lanes holds chunk k
        auto load = [&](int32_t g0) {
            floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
            const int32_t n = g0 + 4 * lane;
            if (n + 3 < NT) return (floatx4)(*(const floatx4u *)(w + n));
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (n + k < NT) v[k] = w[n + k];
            return v;
        };
        floatx4 ahead = load(0);
        float tot = 0.0f, mag = 0.0f;
        int32_t reset = RP;                                           // the next periodic reset at or after the chunk
        for (int32_t n0 = 0; n0 < NT; n0 += 64) {
            if ((n0 & 255) == 0) {
                const floatx4 v = ahead;
                ahead = load(n0 + 256);
                rs += ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
                tot = row_tree((v[0] + v[1]) + (v[2] + v[3]));
                mag = row_tree((fabsf(v[0]) + fabsf(v[1])) + (fabsf(v[2]) + fabsf(v[3])));
            }
            if (done) continue;
            const float ct = lane_value(tot, (n0 & 255) / 4), ca = lane_value(mag, (n0 & 255) / 4);
            while (RP > 0 && reset < n0) reset += RP;
            bool idle;                                                // no sample, reset or close comparison in the chunk
            if (pending) {
                idle = ns - n0 >= 64;
            } else {
                const float q0 = Qb - Qbc;
                const float most = P.eps_abs + P.eps_rel * ((Ab + ca) + (fabsf(q0) + ca) + P.thr);
                const float room = (P.thr - (q0 + 1.00001f * ca)) - 2.5f * most;     // to the threshold, at least
                const bool no_reset = RP <= 0 || reset - n0 >= 64;
                idle = no_reset && (ready - n0 >= 64 || room > kNormalBound * P.sig_disc);
                if (!idle && no_reset && room * disc_inv > 3.25f) {   // few chunks have a draw that far out
                    float u0, u1;
                    noise_words(P, pid, (uint32_t)(n0 + lane), ev, STREAM_DISC, u0, u1);
                    idle = !__ballot(!normal_below(u0, room * disc_inv));
                }
            }
            if (idle) {
                carry(ct, ca);
                continue;
            }
            const int32_t n = n0 + lane;
            const float x = n < NT ? w[n] : 0.0f;
            float sx, sa;                                             // prefix sums over lanes s..lane
            auto scan = [&](int32_t s) {
                sx = lane >= s ? x : 0.0f;
                sa = fabsf(sx);
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const float yx = lane_from(4 * lane + 256 - 4 * d, sx), ya = lane_from(4 * lane + 256 - 4 * d, sa);
                    sx += lane >= d ? yx : 0.0f;
                    sa += lane >= d ? ya : 0.0f;
                }
            };
            auto restart = [&](uint32_t tick) {                       // integrator reset
                Qb = P.sig_reset > 0.0f ? P.sig_reset * noise_normal(P, pid, tick, ev, STREAM_RESET) : 0.0f;
                Qbc = 0.0f;
                Ab = 0.0f;
            };
            scan(0);
            const int32_t jn = min(64, NT - n0);
            int32_t s = 0;                                            // first lane of the current segment
            bool at_reset = false;                                    // the periodic reset at lane s is applied
            while (true) {
                if (!pending && !at_reset && RP > 0 && n0 + s > 0 && (n0 + s) % RP == 0) restart((uint32_t)(n0 + s));
                const float Qv0 = Qb - Qbc;
                const float Ql = Qv0 + sx, Al = Ab + sa;              // charge and |charge| after this lane's tick
                if (pending) {
                    const int32_t js = ns - n0;
                    if (js >= jn) break;                              // the sample is in a later chunk
                    const float Qv = lane_value(Ql, js), Av = lane_value(Al, js);
                    float qs = Qv;
                    if (P.sig_unc > 0.0f) qs += P.sig_unc * noise_normal(P, pid, (uint32_t)ns, ev, STREAM_SAMPLE);
                    const float xq = __fdiv_rn(qs, P.q_lsb);
                    const float fl = floorf(xq);
                    int32_t code = (int32_t)fmaxf(fminf(fl, 1.0e9f), -1.0e9f) + P.pedestal;
                    uint8_t flag = uncertain ? 2 : 0;
                    if (code < 0) { code = 0; flag |= 4; }
                    if (code > P.adc_max) { code = P.adc_max; flag |= 4; }
                    const float dist = (xq - fl) * P.q_lsb;
                    const float eps = P.eps_abs + P.eps_rel * (Av + fabsf(qs) + P.thr);
                    if (dist < eps || P.q_lsb - dist < eps) flag |= 1;
                    if (SETTLE) close |= dist < 2.0f * eps || P.q_lsb - dist < 2.0f * eps;
                    if (cnt < P.max_packets) {
                        if (lane == 0) {
                            pk_tick[obase + cnt] = ns;
                            pk_adc[obase + cnt] = (uint16_t)code;
                            pk_flag[obase + cnt] = flag;
                        }
                        ++cnt;
                    } else {
                        ++over;
                    }
                    restart((uint32_t)ns);
                    pending = false;
                    ready = ns + 1;
                    last = ns;
                    s = js + 1;
                    at_reset = false;
                    if (s >= jn) break;
                    scan(s);
                    continue;
                }
                // the next periodic reset after lane s ends the lanes compared against this segment's charge
                int32_t r = jn;
                if (RP > 0) {
                    const int32_t t = ((n0 + s) / RP + 1) * RP;       // first multiple of the period after n0 + s
                    if (t - n0 < jn) r = t - n0;
                }
                const int32_t lo = max(s, ready - n0);
                const bool cmp = lane >= lo && lane < r;
                float m = 0.0f, eps = 0.0f;
                if (cmp) {
                    float disc = 0.0f;
                    eps = P.eps_abs + P.eps_rel * (Al + fabsf(Ql) + P.thr);
                    if (P.sig_disc > 0.0f && Ql + kNormalBound * P.sig_disc >= P.thr) {
                        float u0, u1;
                        noise_words(P, pid, (uint32_t)n, ev, STREAM_DISC, u0, u1);
                        if (!normal_below(u0, ((P.thr - Ql) - 2.5f * eps) * disc_inv)) disc = P.sig_disc * box_muller(u0, u1);
                    }
                    m = (Ql + disc) - P.thr;
                }
                const uint64_t cross = __ballot(cmp && m >= 0.0f), near = __ballot(cmp && fabsf(m) < eps);
                const uint64_t near2 = SETTLE ? __ballot(cmp && fabsf(m) < 2.0f * eps) : 0;
                if (cross) {
                    const int32_t c = __ffsll((unsigned long long)cross) - 1;
                    if (near & ((2ull << c) - 1)) uncertain = true;    // lanes up to the crossing (c = 63: all)
                    if (near2 & ((2ull << c) - 1)) close = true;
                    pending = true;
                    ns = max(n0 + c + P.hold, last + P.spacing);
                    if (ns >= NT) { ++dropped; done = true; break; }
                    continue;                                         // the sample may fall in this chunk
                }
                if (near) uncertain = true;
                if (near2) close = true;
                if (r < jn) {                                         // periodic reset at lane r
                    restart((uint32_t)(n0 + r));
                    s = r;
                    at_reset = true;
                    scan(s);
                    continue;
                }
                break;
            }
            if (!done && s < jn) carry(lane_value(sx, jn - 1), lane_value(sa, jn - 1));
        }
        if (lane == 0) pk_cnt[slot] = off ? 0 : cnt;
        if (!(SETTLE && close)) add_report(report, e, 2, rs, true);
        if (SETTLE && close) {
            if (lane == 0) settle[atomicAdd(&H->n_settle, 1u)] = (int32_t)slot;
            continue;
        }
        if (lane == 0 && dropped) {
            atomicAdd((unsigned long long *)&H->dropped, (unsigned long long)dropped);
            if (ev_cnt) atomicAdd((unsigned long long *)&ev_cnt[2 * e], (unsigned long long)dropped);
        }
        if (lane == 0 && over) {
            atomicAdd((unsigned long long *)&H->over, (unsigned long long)over);
            if (ev_cnt) atomicAdd((unsigned long long *)&ev_cnt[2 * e + 1], (unsigned long long)over);
        }
    }
}

void launch_electronics(const DevParams &P, const float *wave, const int32_t *slot_gp, const uint64_t *event_ids,
                        int64_t n_slots, const Work &w, int32_t *settle, hipStream_t st) {
    int64_t g = (n_slots + kWG / 64 - 1) / (kWG / 64);
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    auto *k = settle ? k_electronics<true> : k_electronics<false>;
    k<<<(unsigned)g, kWG, 0, st>>>(P, wave, slot_gp, event_ids, w.n_ev, w.disabled, n_slots, w.pk_tick, w.pk_adc, w.pk_flag,
                                   w.pk_off, w.hdr, w.report, w.ev_cnt, nullptr, settle);
}

// ================================================================================================= settled pixels
// A packet's tick and code are decided by comparing a charge with a threshold or an LSB edge, and a charge that lies on
// the edge to within rounding is decided by the order of the FP32 sum.  So that packets do not depend on which units
// summed the currents, they are stated in one order: a pixel with such a decision (about one in a hundred) gets its
// currents again in that order and passes the front end once more.
//   Order: a pair's (a record's) products column by column, cell tick by cell tick, as one FP32 chain per output tick;
// chains of a pair (of kSumKahanEvery records that meet a 256-tick tile) added with Kahan compensation in list order.
// Per pair that is the vector kernels' order, bit for bit, also for the atomic mode, which has none of its own; for the
// summed mode it is this kernel's (the 512-tick vector kernel cuts intervals and tiles otherwise and agrees to rounding).
//   A round is 16 chains of a (pixel, 256 ticks), one per wavefront (lane t: ticks 4 t .. + 3).  The few pixels of a call
// are spread over the chip round by round: a workgroup computes a round's chains, waits until the round before has been
// added, adds its own to the pixel's sum and compensation in memory and passes on.  Rounds are handed out in order, so a
// round waits only on one that is already running.  Beyond the first kSettleSpread pixels there are enough to take a
// pixel's rounds one after the other in one workgroup.  (One workgroup per pixel and 256 ticks throughout: 4.1 instead
// of 0.66 ms for 4 pixels of 3000 dense segments, as 48 workgroups leave the chip idle; 1.1 instead of 0.86 ms for 14
// pixels of a summed event of 20,000 segments, 3000 ticks.)
constexpr int32_t kSettleWG = 1024, kSettleWaves = kSettleWG / 64, kSettleTile = 256;

// Adds a sequence of (table column, cell column) products to the lane's 4 ticks, in pair_block's order.  next(col, cc, n)
// gives the lane's lag-0 entry of the next table column, its cell column and that one's blocks of kAC ticks.  A block needs
// 8 table values more than the one before (they are read as two 16-byte words, with the block's cells, while the block
// before runs): the reads, not the products, bound the plain loop, which takes 11 words of 4 bytes.
template <class Next>
__device__ __forceinline__ void chain4(Next next, float (&acc)[4]) {
    const float *col;
    cfloat_ptr cc;
    int32_t n;
    if (!next(col, cc, n)) return;
    floatx4 t = *(const floatx4u *)col, a1 = *(const floatx4u *)(col - 4), a0 = *(const floatx4u *)(col - 8);
    float c[kAC];
#pragma unroll
    for (int q = 0; q < kAC; ++q) c[q] = cc[q];
    for (bool more = true; more;) {
        floatx4 nt = a0, na1 = a1, na0 = a0;
        if (--n > 0) {
            col -= 8;
            cc += kAC;
        } else {
            more = next(col, cc, n);
            if (more) nt = *(const floatx4u *)col;
        }
        float nc[kAC];
        if (more) {
            na1 = *(const floatx4u *)(col - 4);
            na0 = *(const floatx4u *)(col - 8);
#pragma unroll
            for (int q = 0; q < kAC; ++q) nc[q] = cc[q];
        }
        const float w[11] = {a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3], t[0], t[1], t[2], t[3]};
#pragma unroll
        for (int q = 0; q < kAC; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = fmaf(c[q], w[r - q + kAC - 1], acc[r]);
        if (more) {
            t = nt;
            a1 = na1;
            a0 = na0;
#pragma unroll
            for (int q = 0; q < kAC; ++q) c[q] = nc[q];
        }
    }
}

struct SettleLds {
    float part[kSettleWaves][kSettleTile];
    int32_t win[kSettleWaves][2];                       // ticks that a chain is added to
    int32_t buf[kSettleWaves * kSumKahanEvery];         // summed form: the round's records
    uint32_t unit;
};

// The chains of round r of pixel `slot`, ticks t0 .. t1, into L.part; returns how many wavefronts have one.
template <bool SUMMED>
__device__ __forceinline__ int32_t settle_chains(const DevParams &P, const Work &w, const SumWork &sw,
                                                 const float *__restrict__ Rpad, SettleLds &L, int64_t slot, int32_t r,
                                                 int32_t t0, int32_t t1) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t TR = P.t_r, nb = t0 + 4 * lane;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int32_t lo = t0, hi = t1, n_chain;
    if constexpr (SUMMED) {
        // the records that meet the tile, number 64 r .. 64 r + 63 of them (every wavefront finds the same)
        constexpr int32_t kEach = kSumKahanEvery, kRound = kSettleWaves * kEach;
        static_assert(kRound == 64, "a round's records");
        const int64_t pb = sw.mlist_off[slot], pe = sw.mlist_off[slot + 1];
        int32_t seen = -64 * r, n = 0;                  // number of the next one, relative to the round
        for (int64_t c0 = pb; c0 < pe && seen < kRound; c0 += 64) {
            const int64_t k = c0 + lane;
            bool in = k < pe;
            if (in) {
                const PieceRef g = sw.mrec[k];
                in = g.a0 + g.na - 1 >= t0 && g.a0 - (TR - 1) <= t0 + kSettleTile - 1;
            }
            const uint64_t mask = __ballot(in);
            const int32_t at = seen + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
            if (wv == 0 && in && at >= 0 && at < kRound) L.buf[at] = (int32_t)(k - pb);
            seen += __builtin_popcountll(mask);
        }
        n = min(max(seen, 0), kRound);
        n_chain = (n + kEach - 1) / kEach;
        __syncthreads();
        int32_t j = wv * kEach;
        const int32_t je = min(j + kEach, n);
        chain4([&](const float *&col, cfloat_ptr &cc, int32_t &nblk) {
            if (j >= je) return false;
            const PieceRef g = sw.mrec[pb + __builtin_amdgcn_readfirstlane(L.buf[j++])];
            cc = uniform_cptr(cell_ptr(sw.S, sw.Sm, sw.nS8, g.cell8));
            col = Rpad + (int64_t)(g.bin & kBinMask) * P.col_len + nb - g.a0 + TR - 1 + kPad;
            nblk = __builtin_amdgcn_readfirstlane((g.na + kAC - 1) / kAC);
            return true;
        }, acc);
    } else {
        const int64_t q = w.slot_off[slot] + (int64_t)r * kSettleWaves;
        n_chain = (int32_t)min<int64_t>(kSettleWaves, w.slot_off[slot + 1] - q);
        if (wv < n_chain) {
            const int32_t p = w.slot_gp[slot] % P.npx;
            const int32_t uc = (p % P.nx) * P.nsub + P.nsub / 2, vc = (p / P.nx) * P.nsub + P.nsub / 2;
            const SegInfo &g = w.si[__builtin_amdgcn_readfirstlane(w.pairs[q + wv])];
            lo = max(t0, g.a0 - (TR - 1));
            hi = min(t1, g.a0 + g.na - 1);
            const int32_t ulo = max(g.u0, uc - P.bx), uhi = min(g.u0 + g.nu - 1, uc + P.bx - 1);
            const int32_t vlo = max(g.v0, vc - P.by), vhi = min(g.v0 + g.nv - 1, vc + P.by - 1);
            if (ulo > uhi || vlo > vhi) hi = -1;
            else if (nb <= hi && nb + 3 >= lo) {
                const int32_t nblk = g.na_pad / kAC;
                cfloat_ptr cells = uniform_cptr(w.cells + g.cell_off);
                const float *row = Rpad + nb - g.a0 + TR - 1 + kPad;
                int32_t u = ulo, v = vlo - 1;
                chain4([&](const float *&col, cfloat_ptr &cc, int32_t &nn) {
                    if (++v > vhi) {
                        v = vlo;
                        if (++u > uhi) return false;
                    }
                    cc = cells + ((int64_t)(u - g.u0) * g.nv + (v - g.v0)) * g.na_pad;
                    col = row + (int64_t)(fold(u - uc) * P.by + fold(v - vc)) * P.col_len;
                    nn = nblk;
                    return true;
                }, acc);
            }
        }
    }
    if (wv < n_chain) {
        *(float4 *)&L.part[wv][4 * lane] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        if (lane == 0) {
            L.win[wv][0] = lo;
            L.win[wv][1] = hi;
        }
    }
    return n_chain;
}

// Adds the round's chains to the sum of tick t.
__device__ __forceinline__ void settle_add(const SettleLds &L, int32_t n_chain, int32_t t0, float &sum, float &cmp) {
    const int32_t i = threadIdx.x, n = t0 + i;
    for (int32_t j = 0; j < n_chain; ++j)
        if (n >= L.win[j][0] && n <= L.win[j][1]) {
            const float y = L.part[j][i] - cmp, t = sum + y;
            cmp = (t - sum) - y;
            sum = t;
        }
}

// token[pixel of the list][tile]: rounds added so far (zero before the launch); comp: the compensations in between.
template <bool SUMMED>
__global__ __launch_bounds__(kSettleWG) void k_settle(DevParams P, Work w, SumWork sw, const float *__restrict__ Rpad,
                                                      const int32_t *__restrict__ list, uint32_t *token, float *comp,
                                                      float *wave) {
    __shared__ __align__(16) SettleLds L;
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t NT = P.nticks, n_tiles = (NT + kSettleTile - 1) / kSettleTile;
    const int32_t n_px = (int32_t)w.hdr->n_settle, n_spread = min(n_px, kSettleSpread);
    if (n_px == 0) return;
    auto rounds = [&](int64_t slot) {
        const int64_t n = SUMMED ? sw.mlist_off[slot + 1] - sw.mlist_off[slot] : w.slot_off[slot + 1] - w.slot_off[slot];
        const int32_t per = SUMMED ? 64 : kSettleWaves;
        return max((int32_t)((n + per - 1) / per), 1);
    };
    // units: the spread pixels' (round, tile) pairs, lane i = pixel i of the list; then (pixel, tile) pairs
    const int32_t mine = lane < n_spread ? rounds(list[lane]) * n_tiles : 0;
    int32_t end = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t x = __shfl_up(end, d);
        if (lane >= d) end += x;
    }
    const int32_t n_spread_units = __builtin_amdgcn_readlane(end, 63);
    const int64_t n_units = n_spread_units + (int64_t)(n_px - n_spread) * n_tiles;
    for (;;) {
        if (tid == 0) L.unit = atomicAdd(&w.hdr->settle_work, 1u);
        __syncthreads();
        const uint32_t unit = __builtin_amdgcn_readfirstlane(L.unit);
        __syncthreads();
        if ((int64_t)unit >= n_units) break;
        if ((int32_t)unit < n_spread_units) {
            const int32_t i = __builtin_ctzll(__ballot(end > (int32_t)unit));
            const int32_t k = (int32_t)unit - (__builtin_amdgcn_readlane(end, i) - __builtin_amdgcn_readlane(mine, i));
            const int32_t r = k / n_tiles, tile = k - r * n_tiles, t0 = tile * kSettleTile;
            const int64_t slot = __builtin_amdgcn_readfirstlane(list[i]);
            const bool last = r + 1 == __builtin_amdgcn_readlane(mine, i) / n_tiles;
            const int32_t n_chain = settle_chains<SUMMED>(P, w, sw, Rpad, L, slot, r, t0, min(t0 + kSettleTile, NT) - 1);
            uint32_t *tk = &token[i * n_tiles + tile];
            if (tid == 0) {
                while (__hip_atomic_load(tk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint32_t)r)
                    __builtin_amdgcn_s_sleep(1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            __syncthreads();                            // the chains are in place, too
            if (tid < kSettleTile && t0 + tid < NT) {
                float *ps = &wave[slot * NT + t0 + tid], *pc = &comp[(int64_t)i * NT + t0 + tid];
                float sum = 0.0f, cmp = 0.0f;
                if (r > 0) {
                    sum = __hip_atomic_load(ps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    cmp = __hip_atomic_load(pc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                settle_add(L, n_chain, t0, sum, cmp);
                __hip_atomic_store(ps, last ? sum - cmp : sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(pc, cmp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            // the workgroup's stores are complete, then the token is released for all of them.  (A release by every writing
            // wavefront writes the L2 back as often: 2.06 instead of 0.86 ms on a summed event of 20,000 segments.)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) __hip_atomic_store(tk, (uint32_t)r + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const int64_t k = (int64_t)unit - n_spread_units;
            const int64_t slot = __builtin_amdgcn_readfirstlane(list[n_spread + k / n_tiles]);
            const int32_t t0 = (int32_t)(k % n_tiles) * kSettleTile, n_round = rounds(slot);
            float sum = 0.0f, cmp = 0.0f;
            for (int32_t r = 0; r < n_round; ++r) {
                const int32_t n_chain = settle_chains<SUMMED>(P, w, sw, Rpad, L, slot, r, t0, min(t0 + kSettleTile, NT) - 1);
                __syncthreads();
                if (tid < kSettleTile) settle_add(L, n_chain, t0, sum, cmp);
                __syncthreads();
            }
            if (tid < kSettleTile && t0 + tid < NT) wave[slot * NT + t0 + tid] = sum - cmp;
        }
        __syncthreads();                                // keeps thread 0's token and its next unit apart: without it the
                                                        // other lanes of its wavefront are sent round the loop alone
    }
}

void launch_settle(const DevParams &P, const Work &w, const SumWork &sw, const Table &T, float *wave,
                   const int32_t *slot_gp, const uint64_t *event_ids, bool summed, int64_t n_slots, const int32_t *list,
                   uint32_t *token, float *comp, hipStream_t st) {
    if (n_slots <= 0) return;
    auto *k = summed ? k_settle<true> : k_settle<false>;
    k<<<256, kSettleWG, 0, st>>>(P, w, sw, T.Rpad, list, token, comp, wave);
    k_electronics<false><<<(unsigned)std::min<int64_t>(n_slots, 256), 64, 0, st>>>(
        P, wave, slot_gp, event_ids, w.n_ev, w.disabled, n_slots, w.pk_tick, w.pk_adc, w.pk_flag, w.pk_off, w.hdr, w.report,
        w.ev_cnt, list, nullptr);
}

__global__ void k_compact(int32_t max_packets, int64_t n_slots, const int64_t *pk_off, const int32_t *slot_gp,
                          int32_t npx, const int32_t *pk_tick, const uint16_t *pk_adc, const uint8_t *pk_flag,
                          int32_t *o_pixel, int32_t *o_tick, uint16_t *o_adc, uint8_t *o_flag, int64_t cap,
                          const DevHeader *H, int64_t *counts, int32_t n_ev, const int64_t *ev_pix_off,
                          int64_t *ev_pkt_off) {
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot == 0 && counts) {
        counts[0] = n_slots;
        counts[1] = pk_off[n_slots];
        counts[2] = H->dropped;
        counts[3] = H->over;
    }
    if (ev_pkt_off && ev_pix_off)
        for (int64_t e = slot; e <= n_ev; e += (int64_t)gridDim.x * blockDim.x) ev_pkt_off[e] = pk_off[ev_pix_off[e]];
    if (slot >= n_slots) return;
    const int64_t off = pk_off[slot], cnt = pk_off[slot + 1] - off;
    const int32_t pid = slot_gp[slot] % npx;
    for (int64_t k = 0; k < cnt && off + k < cap; ++k) {
        const int64_t src = slot * max_packets + k;
        o_pixel[off + k] = pid;
        o_tick[off + k] = pk_tick[src];
        o_adc[off + k] = pk_adc[src];
        o_flag[off + k] = pk_flag[src];
    }
}

void launch_compact_packets(const DevParams &P, const Work &w, int64_t n_slots, int32_t *pkt_pixel, int32_t *pkt_tick,
                            uint16_t *pkt_adc, uint8_t *pkt_flags, int64_t cap_packets, const int64_t *ev_pix_off,
                            int64_t *ev_pkt_off, int64_t *counts, hipStream_t st) {
    scan_exclusive(w.pk_off, n_slots + 1, nullptr, w.scan_tmp, st);
    k_compact<<<(unsigned)std::max<int64_t>((n_slots + kWG - 1) / kWG, 1), kWG, 0, st>>>(
        P.max_packets, n_slots, w.pk_off, w.slot_gp, P.npx, w.pk_tick, w.pk_adc, w.pk_flag, pkt_pixel, pkt_tick, pkt_adc,
        pkt_flags, cap_packets, w.hdr, counts, w.n_ev, ev_pix_off, ev_pkt_off);
}

// ================================================================================================= work statistics
// Algorithmic work of the induction stage of the last pipeline call: for every (segment, pixel) pair, the number of
// charge cells in the pixel's table reach and the number of (cell, tick) products that land in the tick window.
__global__ void k_work_stats(DevParams P, const SegInfo *si, int64_t n_seg, unsigned long long *acc) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_seg) return;
    const SegInfo g = si[s];
    if (g.n_pairs == 0) return;
    // kept table ticks summed over the segment's cell ticks a (independent of the pixel)
    unsigned long long kept = 0;
    for (int32_t a = g.a0; a < g.a0 + g.na; ++a) {
        const int32_t lo = max(a - P.t_r + 1, 0), hi = min(a, P.nticks - 1);
        if (hi >= lo) kept += (unsigned long long)(hi - lo + 1);
    }
    unsigned long long cols = 0;
    for (int32_t iy = g.iy0; iy <= g.iy1; ++iy)
        for (int32_t ix = g.ix0; ix <= g.ix1; ++ix) {
            const int32_t uc = ix * P.nsub + P.nsub / 2, vc = iy * P.nsub + P.nsub / 2;
            const int32_t nu = min(g.u0 + g.nu - 1, uc + P.bx - 1) - max(g.u0, uc - P.bx) + 1;
            const int32_t nv = min(g.v0 + g.nv - 1, vc + P.by - 1) - max(g.v0, vc - P.by) + 1;
            if (nu > 0 && nv > 0) cols += (unsigned long long)nu * nv;
        }
    atomicAdd(&acc[0], (unsigned long long)g.n_pairs);
    atomicAdd(&acc[1], cols * kept);
    atomicAdd(&acc[2], cols * (unsigned long long)g.na);
    atomicAdd(&acc[3], (unsigned long long)g.nu * g.nv * g.na);
}

void launch_work_stats(const DevParams &P, const SegInfo *si, int64_t n_seg, unsigned long long *acc, hipStream_t st) {
    if (n_seg > 0) k_work_stats<<<(unsigned)((n_seg + kWG - 1) / kWG), kWG, 0, st>>>(P, si, n_seg, acc);
}

// Summed induction: per active pixel, the (column-piece tick, table tick) products that land in the window.
// Summed mode: a tick of a piece counts only if it holds charge (the ticks a piece adds for alignment, and the short
// gaps between segments that a piece spans, hold exact zeros and are not algorithmic work).
__global__ void k_work_stats_summed(DevParams P, int64_t n_slots, const int64_t *list_off, const PieceRef *rec,
                                    const float *S, const int64_t *mlist_off, const PieceRef *mrec, bool matrix,
                                    unsigned long long *acc) {
    const int32_t tile = matrix ? kMmaSub : kTileTicks;
    int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= n_slots) return;
    unsigned long long f = 0, cells = 0, issued = 0;
    const int32_t n_tiles = (P.nticks + tile - 1) / tile;
    // algorithmic work: every non-zero summed charge tick of every column piece in reach, times the table ticks
    // that land inside the readout
    for (int64_t q = list_off[slot]; q < list_off[slot + 1]; ++q) {
        const PieceRef g = rec[q];
        const float *sv = S + (int64_t)g.cell8 * kAC;
        for (int32_t a = g.a0; a < g.a0 + g.na; ++a) {
            if (sv[a - g.a0] == 0.0f) continue;
            const int32_t lo = max(a - P.t_r + 1, 0), hi = min(a, P.nticks - 1);
            if (hi >= lo) f += (unsigned long long)(hi - lo + 1);
            ++cells;
        }
    }
    // products the summed kernel computes for the merged records, zeros included: every tile (of `tile` ticks) a
    // record's window meets, all its ticks x every 8-tick charge block (the matrix kernel: every 32-value step of a part)
    for (int64_t q = mlist_off[slot]; q < mlist_off[slot + 1]; ++q) {
        const PieceRef g = mrec[q];
        const int32_t t_lo = max(floor_div(g.a0 - P.t_r + 1, tile), 0);
        const int32_t t_hi = min(floor_div(g.a0 + g.na - 1, tile), n_tiles - 1);
        if (t_hi < t_lo) continue;
        int32_t lags = (g.na + kAC - 1) / kAC * kAC;
        if (matrix) {
            lags = 0;
            for (int32_t done = 0; done < g.na; done += kMmaPart) {
                const int32_t L = min(g.na - done, kMmaPart);
                lags += (L + 46 + ((P.t_r - g.a0 - done - L) & 7)) / 32 * 32;
            }
        }
        issued += (unsigned long long)(t_hi - t_lo + 1) * (unsigned long long)lags * (unsigned long long)tile;
    }
    atomicAdd(&acc[0], (unsigned long long)(mlist_off[slot + 1] - mlist_off[slot]));
    atomicAdd(&acc[1], f);
    atomicAdd(&acc[2], cells);
    atomicAdd(&acc[3], issued);
}

void launch_work_stats_summed(const DevParams &P, int64_t n_slots, const int64_t *list_off, const PieceRef *rec,
                              const float *S, const int64_t *mlist_off, const PieceRef *mrec, bool matrix,
                              unsigned long long *acc, hipStream_t st) {
    if (n_slots > 0)
        k_work_stats_summed<<<(unsigned)((n_slots + kWG - 1) / kWG), kWG, 0, st>>>(
            P, n_slots, list_off, rec, S, mlist_off, mrec, matrix, acc);
}

// ================================================================================================= Philox test hook
__global__ void k_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, uint32_t *out, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint4 c = make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]);
    uint4 x = philox4x32_10(c, k0, k1);
    out[4 * i] = x.x; out[4 * i + 1] = x.y; out[4 * i + 2] = x.z; out[4 * i + 3] = x.w;
}

void launch_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, uint32_t *out, int64_t n, hipStream_t st) {
    if (n > 0) k_philox<<<(unsigned)((n + kWG - 1) / kWG), kWG, 0, st>>>(ctr, k0, k1, out, n);
}

}  // namespace ltsim
