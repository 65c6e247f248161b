// Direct (all-pairs) Stokes kernel sums on gfx950.
//
// Single layer (Stokeslet, paper eq. sl_stokes) and double layer (stresslet,
// stated after eq. double_layer_int_eq), summed over the smooth quadrature of
// eq. smooth_double_layer_int_eq_patches_disc (strength q = w * density),
// with the "other cells only" rule of the explicit step (Sec. 2.2, step 1(d))
// and distance-0 pairs skipped.
//
// Design (CDNA4, wave64):
//   * prep: one thread per source packs {position, q[, normal]} into a padded
//     record array and each wave summarises its 64-source sub-tile (bounding
//     box, group range, near radius).
//   * sum: a workgroup of 4 waves owns 4*64*T targets (T per lane, kept in
//     registers) and one split of the sources.  Sources stream through LDS
//     in steps of 256 records (register prefetch of the next step); every
//     lane of a wave reads the same record, a broadcast LDS read.
//   * per 64-source sub-tile the wave decides, uniformly, whether the fast
//     loop (no per-pair tests) is exact: box far from its targets and no
//     shared group.  Other sub-tiles take a masked loop: in float64 in the same
//     kernel, in mixed precision in a near-pass kernel of its own (which takes
//     the same decision again), whose float64 pairs would cost the main loop its
//     registers.  Mixed precision evaluates pairs in float32
//     on offsets from the sub-tile centre (each rounded once from float64),
//     sums each sub-tile in float32 and adds it into float64 accumulators.
//     In the near pass (possible exclusions or near pairs, or a gap below an eighth of
//     the sub-tile's extent) r is formed from float32 high parts plus float32
//     residues, and pairs within the near radius are evaluated in float64.
//   * work balance (stream-K): the grid holds exactly the resident number of
//     workgroups; the (target block x 64-source sub-tile) units are cut into
//     equal contiguous ranges, one per workgroup (long float64 ranges count a
//     target block's chunks in an order of their own).  A workgroup flushes float64
//     partial sums whenever its range moves to a new target block; segment
//     ids (workgroup + target block) are consecutive, and a second kernel
//     adds each target's segments in fixed order (deterministic, no atomics).
//   * the decision tests every target of the wave against the
//     sub-tile box, after a whole-wave box test that settles most sub-tiles.
#include <float.h>
#include <limits.h>

#include <numeric>
#include <type_traits>

#include "direct_dev.hpp"

namespace stokes {

struct DirectArgs {
    SumInputs in;
    const void* rec;          // packed source records
    const void* aux;          // FP64 path: padded int32 groups; mixed: float4 low parts
    const SubMeta* meta;
    int64_t n_sub;            // source sub-tiles
    int64_t units;            // target blocks x sub-tiles
    int cut;                  // ranges begin at multiples of this many units
    int64_t step;             // float64: a target block takes chunk k * step mod (chunks) k-th
    double* part;             // partial sums, one segment per (block, target block) pair
    double* near_part;        // near-pass sums, (near slices, 3, blocks_x * kBlock * T)
};

// ---------------------------------------------------------------------------
// source prep
// ---------------------------------------------------------------------------
template <int KT, int MIXED>
__global__ __launch_bounds__(kBlock) void prep_sources(SumInputs in, void* rec_out, void* aux_out,
                                                       SubMeta* meta) {
    using Rec = typename SrcRec<KT, MIXED>::type;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;   // grid covers n_src_pad exactly
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t n = in.n_src;
    const bool valid = i < n;
    double y[3] = {kPadPos, kPadPos, kPadPos}, q[3] = {0, 0, 0}, nv[3] = {0, 0, 0};
    double rn = 0.0;
    int32_t g = INT_MIN;
    if (valid) {
        const double w = in.weight[i];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            y[c] = in.src_xyz[c * n + i];
            q[c] = w * in.density[c * n + i];
            if (KT == 1) nv[c] = in.normal[c * n + i];
        }
        if (MIXED == 0) {   // FP64 records hold doubled positions (exact)
            y[0] *= 2.0; y[1] *= 2.0; y[2] *= 2.0;
        }
        g = in.src_group ? in.src_group[i] : 0;
        if (MIXED && in.group_h) {
            if (g >= 0 && g < in.n_groups) {
                rn = in.near_frac * in.group_h[g];
            } else {   // invalid group id: poison this source's strength
                q[0] = q[1] = q[2] = __builtin_nan("");
            }
        }
    }
    double lo[3], hi[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c] = wave_min(valid ? y[c] : DBL_MAX);
        hi[c] = wave_max(valid ? y[c] : -DBL_MAX);
    }
    const int gmin = wave_mini(valid ? g : INT_MAX);
    const int gmax = wave_maxi(valid ? g : INT_MIN);
    const double rmax = wave_max(valid ? rn : 0.0);
    const int count = __popcll(__ballot(valid));
    double ctr[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) ctr[c] = count ? 0.5 * (lo[c] + hi[c]) : 0.0;

    Rec* rec = reinterpret_cast<Rec*>(rec_out);
    if constexpr (MIXED == 0) {
        Rec r;
        r.x = y[0]; r.y = y[1]; r.z = y[2];
        r.qx = q[0]; r.qy = q[1]; r.qz = q[2];
        if constexpr (KT == 0) { r.q4x = 4.0 * q[0]; r.q4y = 4.0 * q[1]; r.q4z = 4.0 * q[2]; r.pad = 0.0; }
        if constexpr (KT == 1) { r.nx = nv[0]; r.ny = nv[1]; r.nz = nv[2]; r.pad = 0.0; }
        rec[i] = r;
        reinterpret_cast<int32_t*>(aux_out)[i] = g;
    } else {
        // offset from the sub-tile centre as float32 high part + float32 residue
        float hi3[3], lo3[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double off = y[c] - ctr[c];
            hi3[c] = valid ? (float)off : kPadOff;
            lo3[c] = valid ? (float)(off - (double)hi3[c]) : 0.0f;
        }
        reinterpret_cast<float4*>(aux_out)[i] = make_float4(lo3[0], lo3[1], lo3[2], 0.0f);
        Rec r;
        r.ox = hi3[0];
        r.oy = hi3[1];
        r.oz = hi3[2];
        r.qx = (float)q[0]; r.qy = (float)q[1]; r.qz = (float)q[2];
        r.t2 = (float)(rn * rn);
        r.g = g;
        if constexpr (KT == 1) { r.nx = (float)nv[0]; r.ny = (float)nv[1]; r.nz = (float)nv[2]; r.pad = 0.f; }
        rec[i] = r;
    }
    if (lane == 0) {
        SubMeta m;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            m.lo[c] = count ? lo[c] : 0.0;
            m.hi[c] = count ? hi[c] : 0.0;
            m.ctr[c] = ctr[c];
        }
        m.rnear = rmax;
        m.gmin = gmin; m.gmax = gmax; m.count = count; m.pad = 0;
        meta[i / kSub] = m;
    }
}

template <int T>
__device__ __forceinline__ void flush_segment(const DirectArgs& a, int64_t tbk, int wave, int lane,
                                              const double (&ax)[T], const double (&ay)[T],
                                              const double (&az)[T]) {
    constexpr int BT = kBlock * T;
    double* seg = a.part + (int64_t)(blockIdx.x + tbk) * 3 * BT;
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const int li = wave * (kWave * T) + k * kWave + lane;
        seg[li] = ax[k];
        seg[BT + li] = ay[k];
        seg[2 * BT + li] = az[k];
    }
}

// Launch-shape tuning: targets per lane (T) and the minimum number of waves
// per SIMD that the register allocation must allow, for each precision.
#ifndef STOKES_DIRECT_T64
#define STOKES_DIRECT_T64 4
#endif
#ifndef STOKES_DIRECT_W64
#define STOKES_DIRECT_W64 3
#endif
#ifndef STOKES_DIRECT_T32
#define STOKES_DIRECT_T32 2
#endif
// The mixed kernel's float32 loop is sensitive to the register assignment (an FMA
// whose three operands share a bank takes longer), which the occupancy bound
// steers; measured at 3, 4, 5 and 6 waves: single layer, 69,632 points 2.21,
// 2.23, 2.15, 2.15 ms; double layer, 294,912 wall nodes at 48,000 targets 8.15,
// 8.02, 8.56, 8.54 ms.
#ifndef STOKES_DIRECT_W32SL
#define STOKES_DIRECT_W32SL 6
#endif
#ifndef STOKES_DIRECT_W32DL
#define STOKES_DIRECT_W32DL 4
#endif

// Targets per lane and waves per SIMD of long double-layer sums.
constexpr int kT64Long = 8, kW64Long = 2;

// FP64 kernel.  Sub-tiles that need the rules take the masked loop here: its
// compares and select add about a fifth to a pair, where a pass of its own finds
// them again and brings its own partial sums (6.4e7 double-layer pairs of a
// check-point quadrature 197 us with such a pass, 141 here; 16,001 tracers at
// 34,816 sources 550 and 428, 60,001 at 108,800 4.94 and 4.65 ms).  Where targets
// lie among their own sources those sub-tiles follow each other, so a range takes
// its chunks spread over all sources (see spread_step).
template <int KT, int T>
__global__ __launch_bounds__(kBlock, T == kT64Long ? kW64Long : STOKES_DIRECT_W64) void direct_f64(DirectArgs a) {
    using Rec = typename SrcRec<KT, 0>::type;
    constexpr int BT = kBlock * T;
    __shared__ Rec s_rec[kTile];
    __shared__ int32_t s_grp[kTile];

    const int64_t U = a.units, C = a.n_sub, G = gridDim.x;
    const int64_t u0 = range_begin(blockIdx.x, U, G, a.cut), u1 = range_begin(blockIdx.x + 1, U, G, a.cut);
    if (u0 >= u1) return;                      // whole workgroup idle (uniform)
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const bool excl = a.in.excl != 0;
    const Rec* rec = reinterpret_cast<const Rec*>(a.rec);
    const int32_t* grp = reinterpret_cast<const int32_t*>(a.aux);

    Targets<T> t;
    Box wbox{};
    bool wave_active = false;
    int64_t tbk = -1;
    double ax[T], ay[T], az[T];
#pragma unroll
    for (int k = 0; k < T; ++k) ax[k] = ay[k] = az[k] = 0.0;

    int64_t ub = u0 / C, sub = u0 % C;         // unit position, advanced by up to four sub-tiles
    const int64_t chunks = (C + 3) >> 2;
    int64_t chunk = (sub >> 2) * a.step % chunks;
    for (int64_t u = u0; u < u1;) {
        const int s0 = (int)(sub & 3), s1 = (int)min((int64_t)4, s0 + min(u1 - u, C - sub));
        __syncthreads();                       // previous step's readers are done
        if (ub != tbk) {
            if (tbk >= 0) flush_segment<T>(a, tbk, wave, lane, ax, ay, az);
            tbk = ub;
            const int64_t tb = tbk * BT + (int64_t)wave * (kWave * T);
            wave_active = tb < a.in.n_trg;
            wbox = load_targets<T>(a.in, wave_active ? tb : 0, lane, t);
            double_targets<T>(t, &wbox);
#pragma unroll
            for (int k = 0; k < T; ++k) ax[k] = ay[k] = az[k] = 0.0;
        }
        const int64_t first = chunk * 4;       // the chunk's first sub-tile
        if (wave >= s0 && wave < s1) {
            s_rec[threadIdx.x] = rec[first * kSub + threadIdx.x];
            s_grp[threadIdx.x] = grp[first * kSub + threadIdx.x];
        }
        __syncthreads();
        if (wave_active) {
#pragma unroll 1
            for (int s = s0; s < s1; ++s) {
                const SubMeta m = a.meta[first + s];
                if (m.count == 0) continue;
                const Rec* base = s_rec + s * kSub;
                if (!needs_near<T, false>(wbox, t, m, excl)) {
#pragma unroll 2
                    for (int j = 0; j < kSub; ++j) {
                        const Rec sr = base[j];
#pragma unroll
                        for (int k = 0; k < T; ++k)
                            pair_f64<KT, false>(sr, t.x[k], t.y[k], t.z[k], false, ax[k], ay[k], az[k]);
                    }
                    continue;
                }
#pragma unroll 2
                for (int j = 0; j < kSub; ++j) {
                    const Rec sr = base[j];
                    const int32_t gs = s_grp[s * kSub + j];
#pragma unroll
                    for (int k = 0; k < T; ++k)
                        pair_f64<KT, true>(sr, t.x[k], t.y[k], t.z[k], excl && gs == t.g[k], ax[k], ay[k], az[k]);
                }
            }
        }
        u += s1 - s0;
        sub += s1 - s0;
        if (sub == C) { sub = chunk = 0; ++ub; }
        else if ((sub & 3) == 0 && (chunk += a.step) >= chunks) chunk -= chunks;
    }
    flush_segment<T>(a, tbk, wave, lane, ax, ay, az);
}

// Main mixed kernel: float32 fast loop only; sub-tiles needing care are
// skipped (direct_near_mixed takes them).  CNT: also record each pair's class
// (test-only instantiation).
template <int KT, int T, bool CNT = false>
__global__ __launch_bounds__(kBlock, KT == 0 ? STOKES_DIRECT_W32SL : STOKES_DIRECT_W32DL) void direct_mixed(DirectArgs a) {
    using Rec = typename SrcRec<KT, 1>::type;
    constexpr int BT = kBlock * T;
    __shared__ Rec s_rec[kTile];

    const int64_t U = a.units, C = a.n_sub, G = gridDim.x;
    const int64_t u0 = range_begin(blockIdx.x, U, G, a.cut), u1 = range_begin(blockIdx.x + 1, U, G, a.cut);
    if (u0 >= u1) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const bool excl = a.in.excl != 0;
    const Rec* rec = reinterpret_cast<const Rec*>(a.rec);

    Targets<T> t;
    Box wbox{};
    bool wave_active = false;
    int64_t tbk = -1;
    double ax[T], ay[T], az[T];
#pragma unroll
    for (int k = 0; k < T; ++k) ax[k] = ay[k] = az[k] = 0.0;

    int64_t ub = u0 / C, sub = u0 % C;
    Rec pre = rec[(sub & ~(int64_t)3) * kSub + threadIdx.x];
    for (int64_t u = u0; u < u1;) {
        const int s0 = (int)(sub & 3), s1 = (int)min((int64_t)4, s0 + min(u1 - u, C - sub));
        const int64_t first = sub - s0;        // the chunk's first sub-tile
        __syncthreads();
        if (ub != tbk) {
            if (tbk >= 0) flush_segment<T>(a, tbk, wave, lane, ax, ay, az);
            tbk = ub;
            const int64_t tb = tbk * BT + (int64_t)wave * (kWave * T);
            wave_active = tb < a.in.n_trg;
            wbox = load_targets<T>(a.in, wave_active ? tb : 0, lane, t);
#pragma unroll
            for (int k = 0; k < T; ++k) ax[k] = ay[k] = az[k] = 0.0;
        }
        s_rec[threadIdx.x] = pre;
        __syncthreads();
        u += s1 - s0;
        sub += s1 - s0;
        if (sub == C) { sub = 0; ++ub; }
        if (u < u1) pre = rec[sub * kSub + threadIdx.x];
        if (wave_active) {
#pragma unroll 1
            for (int s = s0; s < s1; ++s) {
                const SubMeta m = a.meta[first + s];
                if (m.count == 0 || needs_near<T, true>(wbox, t, m, excl)) continue;
                // target offsets from the sub-tile centre, rounded once from float64
                float xs[T], ys[T], zs[T], bx[T], by[T], bz[T];
#pragma unroll
                for (int k = 0; k < T; ++k) {
                    xs[k] = (float)(t.x[k] - m.ctr[0]);
                    ys[k] = (float)(t.y[k] - m.ctr[1]);
                    zs[k] = (float)(t.z[k] - m.ctr[2]);
                    bx[k] = by[k] = bz[k] = 0.0f;
                }
                const Rec* base = s_rec + s * kSub;
#pragma unroll 2
                for (int j = 0; j < kSub; ++j) {
                    const Rec sr = base[j];
#pragma unroll
                    for (int k = 0; k < T; ++k)
                        pair_f32<KT>(sr, xs[k] - sr.ox, ys[k] - sr.oy, zs[k] - sr.oz, false, false,
                                     bx[k], by[k], bz[k]);
                }
#pragma unroll
                for (int k = 0; k < T; ++k) {
                    ax[k] += (double)bx[k];
                    ay[k] += (double)by[k];
                    az[k] += (double)bz[k];
                }
                if constexpr (CNT) {
                    const int64_t i0 = (first + s) * kSub;
                    for (int k = 0; k < T; ++k) {
                        const int64_t ti = tbk * BT + (int64_t)wave * (kWave * T) + k * kWave + lane;
                        if (ti < a.in.n_trg)
                            for (int j = 0; j < m.count; ++j)
                                atomicAdd(a.in.pair_class + ti * a.in.n_src + i0 + j, kPairF32);
                    }
                }
            }
        }
    }
    flush_segment<T>(a, tbk, wave, lane, ax, ay, az);
}

// Sub-tiles up to which the near pass notes near pairs in its float32 loop: a wave's
// targets spread over few clusters then, and most sub-tiles have some.  With a second
// pass where there are any / noted in the loop, whole calls of cells among 120,001
// tracers: 9 sub-tiles 123 / 108 us, 18 178 / 157, 34 260 / 267; 64 cells (544) among 8,001 234 / 243.
constexpr int kFewSubs = 24;

// Near pass (mixed): the skipped sub-tiles with r from high + low float32 parts,
// the same-group mask, and pairs inside the near radius in float64.  FEW: see
// kFewSubs.  CNT:
// also record each pair's class (test-only instantiation).
template <int KT, int T, bool FEW, bool CNT = false>
__global__ __launch_bounds__(kBlock) void direct_near_mixed(DirectArgs a) {
    using Rec = typename SrcRec<KT, 1>::type;
    constexpr int BT = kBlock * T, kLoop = FEW ? 32 : kSub;
    // each wave stages its current sub-tile in its own slice (read back by
    // broadcast into VGPRs; only that wave touches it, and a wave's LDS
    // operations complete in order, so no workgroup barrier is needed)
    __shared__ Rec s_src[4][kSub];
    __shared__ float4 s_res[4][kSub];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int64_t tbk = blockIdx.x;
    const int64_t tb = tbk * BT + (int64_t)wave * (kWave * T);
    if (tb >= a.in.n_trg) return;
    const bool excl = a.in.excl != 0;
    const Rec* rec = reinterpret_cast<const Rec*>(a.rec);
    const float4* lo = reinterpret_cast<const float4*>(a.aux);
    Targets<T> t;
    const Box wbox = load_targets<T>(a.in, tb, lane, t);
    double ax[T], ay[T], az[T];
#pragma unroll
    for (int k = 0; k < T; ++k) ax[k] = ay[k] = az[k] = 0.0;
    for_each_near<T, true>(wbox, t, a.meta, a.n_sub, lane, (int)blockIdx.y, (int)gridDim.y, excl,
                           [&](int64_t sub, const SubMeta& m) {
        float xs[T], ys[T], zs[T], xl[T], yl[T], zl[T], bx[T], by[T], bz[T];
#pragma unroll
        for (int k = 0; k < T; ++k) {
            const double hx = t.x[k] - m.ctr[0], hy = t.y[k] - m.ctr[1], hz = t.z[k] - m.ctr[2];
            xs[k] = (float)hx; ys[k] = (float)hy; zs[k] = (float)hz;
            xl[k] = (float)(hx - (double)xs[k]);
            yl[k] = (float)(hy - (double)ys[k]);
            zl[k] = (float)(hz - (double)zs[k]);
            bx[k] = by[k] = bz[k] = 0.0f;
        }
        s_src[wave][lane] = rec[sub * kSub + lane];
        s_res[wave][lane] = lo[sub * kSub + lane];
        __builtin_amdgcn_wave_barrier();
        // r = (x_hi - y_hi) + (x_lo - y_lo): the high difference is rounded
        // relative to rho, the residues carry the rest
        auto offset = [&](const Rec& sr, const float4& sl, int k, float& dx, float& dy, float& dz) {
            dx = (xs[k] - sr.ox) + (xl[k] - sl.x);
            dy = (ys[k] - sr.oy) + (yl[k] - sl.y);
            dz = (zs[k] - sr.oz) + (zl[k] - sl.z);
            return __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
        };
        // The float64 pairs come after the float32 loop, which so has no branches: a
        // lane notes its own as bits, and the lanes take theirs side by side,
        // whatever the sources (a branch per source ran them one source after
        // another: 576 sources at 120,001 tracers 81 us here, 64 so).  FEW notes
        // them in the loop, 32 sources at a time; else a second pass over the
        // offsets does, where any lane has one.
        auto take = [&](uint32_t (&set)[T], int j0) {
#pragma unroll
            for (int k = 0; k < T; ++k)
                for (; set[k] != 0; set[k] &= set[k] - 1)
                    near_pair_f64<KT>(a.in, sub * kSub + j0 + __builtin_ctz(set[k]), t.x[k], t.y[k], t.z[k], ax[k],
                                      ay[k], az[k]);
        };
        bool any = false;
#pragma unroll 1
        for (int j0 = 0; j0 < kSub; j0 += kLoop) {
            uint32_t set[T] = {};
#pragma unroll 2
            for (int j = 0; j < kLoop; ++j) {
                const Rec sr = s_src[wave][j0 + j];
                const float4 sl = s_res[wave][j0 + j];
#pragma unroll
                for (int k = 0; k < T; ++k) {
                    float dx, dy, dz;
                    const float r2 = offset(sr, sl, k, dx, dy, dz);
                    const bool excluded = excl && sr.g == t.g[k];
                    const bool near = r2 <= sr.t2;
                    if constexpr (FEW) set[k] |= (uint32_t)(near && !excluded) << j;
                    else any |= near && !excluded;
                    pair_f32<KT>(sr, dx, dy, dz, excluded || near, true, bx[k], by[k], bz[k]);
                    if constexpr (CNT) {
                        const int64_t si = sub * kSub + j0 + j, ti = tb + k * kWave + lane;
                        if (si < a.in.n_src && ti < a.in.n_trg) {
                            // near_pair_f64 takes nothing at zero distance (float64)
                            const int64_t ns = a.in.n_src;
                            const bool zero = t.x[k] == a.in.src_xyz[si] && t.y[k] == a.in.src_xyz[ns + si] &&
                                              t.z[k] == a.in.src_xyz[2 * ns + si];
                            const int32_t cls = excluded ? kPairSkip : !near ? kPairF32 : zero ? kPairSkip : kPairF64;
                            atomicAdd(a.in.pair_class + ti * ns + si, cls);
                        }
                    }
                }
            }
            if constexpr (FEW) take(set, j0);
        }
        if constexpr (!FEW) {
            if (__ballot(any) != 0)
#pragma unroll 1
                for (int j0 = 0; j0 < kSub; j0 += 32) {
                    uint32_t set[T] = {};
#pragma unroll 2
                    for (int j = 0; j < 32; ++j) {
                        const Rec sr = s_src[wave][j0 + j];
                        const float4 sl = s_res[wave][j0 + j];
#pragma unroll
                        for (int k = 0; k < T; ++k) {
                            float dx, dy, dz;
                            const bool near = offset(sr, sl, k, dx, dy, dz) <= sr.t2;
                            set[k] |= (uint32_t)(near && !(excl && sr.g == t.g[k])) << j;
                        }
                    }
                    take(set, j0);
                }
        }
#pragma unroll
        for (int k = 0; k < T; ++k) {
            ax[k] += (double)bx[k];
            ay[k] += (double)by[k];
            az[k] += (double)bz[k];
        }
        __builtin_amdgcn_wave_barrier();   // reads of this sub-tile precede the next writes
    });
    const int64_t np = (int64_t)gridDim.x * BT;
    double* np_slice = a.near_part + (int64_t)blockIdx.y * 3 * np;
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const int64_t gi = tbk * BT + wave * (kWave * T) + k * kWave + lane;
        np_slice[gi] = ax[k];
        np_slice[np + gi] = ay[k];
        np_slice[2 * np + gi] = az[k];
    }
}

// ---------------------------------------------------------------------------
// segment reduction and fills
// ---------------------------------------------------------------------------
// out[c][i] (=|+=) pref * (sum of target i's segments in workgroup order and of
// its near-pass sums).  A call with few target blocks has many of both per
// target (4,352 targets: about 150 segments and 64 near rows), so there P =
// kRedParts threads share a target, each taking a contiguous share, and the shares
// are added in order; with few (see launch_typed) one thread takes them all.
constexpr int kRedParts = 8;
template <int T, int P>
__global__ __launch_bounds__(kBlock) void reduce_segments(const double* __restrict__ part,
                                                          const double* __restrict__ near_part,
                                                          int64_t n_trg, int64_t units,
                                                          int64_t n_sub, int64_t grid, int cut, int slices,
                                                          int64_t np, double pref, double* out,
                                                          int accumulate) {
    constexpr int BT = kBlock * T, kTrg = kBlock / P;
    __shared__ double s_sum[P][3][kTrg];
    const int t = threadIdx.x % kTrg, q = threadIdx.x / kTrg;
    const int64_t i = (int64_t)blockIdx.x * kTrg + t;
    double s[3] = {0.0, 0.0, 0.0};
    if (i < n_trg) {
        const int64_t tbk = i / BT, li = i % BT;
        const int64_t b0 = range_owner(tbk * n_sub, units, grid, cut);
        const int64_t b1 = range_owner((tbk + 1) * n_sub - 1, units, grid, cut) + 1;
        const int64_t e0 = b0 + (b1 - b0) * q / P, e1 = b0 + (b1 - b0) * (q + 1) / P;
#pragma unroll 4
        for (int64_t b = e0; b < e1; ++b) {
            const double* seg = part + (b + tbk) * 3 * BT;
#pragma unroll
            for (int c = 0; c < 3; ++c) s[c] += seg[c * BT + li];
        }
        const int l0 = slices * q / P, l1 = slices * (q + 1) / P;
#pragma unroll 4
        for (int sl = l0; sl < l1; ++sl)
#pragma unroll
            for (int c = 0; c < 3; ++c) s[c] += near_part[(sl * 3 + c) * np + i];
    }
    if constexpr (P == 1) {
        if (i < n_trg)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int64_t o = c * n_trg + i;
                out[o] = accumulate ? out[o] + pref * s[c] : pref * s[c];
            }
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) s_sum[q][c][t] = s[c];
        __syncthreads();
        if (q < 3 && i < n_trg) {
            double v = s_sum[0][q][t];
#pragma unroll
            for (int p = 1; p < P; ++p) v += s_sum[p][q][t];
            const int64_t o = q * n_trg + i;
            out[o] = accumulate ? out[o] + pref * v : pref * v;
        }
    }
}

// ---------------------------------------------------------------------------
// small sums: one kernel
// ---------------------------------------------------------------------------
// The whole float64 sum of a small call in one launch, straight from the
// caller's arrays.  Such a call is bound by latency, not by its pairs: the
// kernels above are three dependent launches, and a few target blocks leave
// most of the chip idle (4,352 points: 51 us there, 44 us here, of which the
// 1.9e7 pairs need 13 at the rate of a full chip; 1,088 points 36 and 18).  Here a
// workgroup owns TW targets and the 256 / TW threads of a target share the
// sources, 256 staged at a time; every pair carries the masks.  The last tile
// has no steps of padding alone (64 sources at 400,000 targets: 107 us with them,
// 39 without).  A target's partial sums are added in a fixed order.
template <int KT, int TW>
__global__ __launch_bounds__(kBlock) void direct_small(SumInputs in, double pref, double* __restrict__ out,
                                                       int accumulate) {
    constexpr int H = kBlock / TW, NC = KT == 0 ? 6 : 9;
    __shared__ double s_src[NC][kBlock];
    __shared__ int32_t s_grp[kBlock];
    const int tid = threadIdx.x, t = tid % TW, h = tid / TW;
    const int64_t n = in.n_src, nt = in.n_trg, i = (int64_t)blockIdx.x * TW + t, ic = min(i, nt - 1);
    const double x = 2.0 * in.trg_xyz[ic], y = 2.0 * in.trg_xyz[nt + ic], z = 2.0 * in.trg_xyz[2 * nt + ic];
    const bool excl = in.excl != 0;
    const int32_t tg = in.trg_group ? in.trg_group[ic] : 0;
    double u[3] = {0.0, 0.0, 0.0};
    auto tile = [&](int64_t b, auto whole) {
        const int64_t m = b + tid;
        double v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = c < 3 ? kPadPos : 0.0;
        int32_t g = INT_MIN;
        if (m < n) {
            const double w = in.weight[m];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                v[c] = 2.0 * in.src_xyz[c * n + m];
                v[3 + c] = w * in.density[c * n + m];
                if constexpr (KT == 1) v[6 + c] = in.normal[c * n + m];
            }
            g = in.src_group ? in.src_group[m] : 0;
        }
        __syncthreads();                       // readers of the previous tile are done
#pragma unroll
        for (int c = 0; c < NC; ++c) s_src[c][tid] = v[c];
        s_grp[tid] = g;
        __syncthreads();
        auto pair = [&](int j) {
            typename SrcRec<KT, 0>::type r;
            r.x = s_src[0][j]; r.y = s_src[1][j]; r.z = s_src[2][j];
            r.qx = s_src[3][j]; r.qy = s_src[4][j]; r.qz = s_src[5][j];
            if constexpr (KT == 0) {
                r.q4x = 4.0 * r.qx; r.q4y = 4.0 * r.qy; r.q4z = 4.0 * r.qz;
            } else {
                r.nx = s_src[6][j]; r.ny = s_src[7][j]; r.nz = s_src[8][j];
            }
            pair_f64<KT, true>(r, x, y, z, excl && s_grp[j] == tg, u[0], u[1], u[2]);
        };
        if constexpr (decltype(whole)::value || TW <= 4) {
#pragma unroll 4
            for (int k = 0; k < TW; ++k) pair(k * H + h);
        } else {                               // no steps of padding alone
            for (int k = 0; k * H < n - b; ++k) pair(k * H + h);
        }
    };
    int64_t b = 0;
    for (; b < (TW <= 4 ? n : n - kBlock + 1); b += kBlock) tile(b, std::true_type{});
    if (b < n) tile(b, std::false_type{});     // (a few steps save nothing: TW > 4)
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) s_src[c][tid] = u[c];
    for (int o = H / 2; o > 0; o >>= 1) {
        __syncthreads();
        if (h < o)
#pragma unroll
            for (int c = 0; c < 3; ++c) s_src[c][tid] += s_src[c][tid + o * TW];
    }
    __syncthreads();
    if (tid < TW && i < nt)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double val = pref * s_src[c][tid];
            out[c * nt + i] = accumulate ? out[c * nt + i] + val : val;
        }
}

// Targets per workgroup: the power of two with the least work on the fullest CU
// (rounds of workgroups times a tile's TW pair steps and its staging, about two
// more; a CU with one workgroup waits on latency as long as one with two).
// 4,352 points on 256 CUs take 79, 50, 41, 49, 62 and 93 us with TW = 1, 2, 4, 8,
// 16 and 32 by this order: 51, 36, 30, 30, 36, 68.
static int small_targets(int64_t n_trg, int n_cu) {
    int best = 1;
    int64_t least = INT64_MAX;
    for (int tw = 1; tw <= kWave; tw *= 2) {
        const int64_t cost = std::max<int64_t>(2, ceil_div(ceil_div(n_trg, tw), n_cu)) * (tw + 2);
        if (cost < least) {
            least = cost;
            best = tw;
        }
    }
    return best;
}

template <int KT>
static void launch_small_kt(const SumInputs& in, double* out, int accumulate, int n_cu, hipStream_t stream) {
    const double pref = (KT == 0 ? 0.25 : 0.125) * in.pref;       // doubled positions, as above
    auto go = [&](auto tw) {
        constexpr int TW = decltype(tw)::value;
        direct_small<KT, TW><<<dim3((unsigned)ceil_div(in.n_trg, TW)), dim3(kBlock), 0, stream>>>(in, pref, out,
                                                                                               accumulate);
    };
    switch (small_targets(in.n_trg, n_cu)) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 8: go(std::integral_constant<int, 8>{}); break;
        case 16: go(std::integral_constant<int, 16>{}); break;
        case 32: go(std::integral_constant<int, 32>{}); break;
        default: go(std::integral_constant<int, 64>{}); break;
    }
}

// The line lies where the other path (the each-pair-once one on shared sets)
// catches up, measured on cells, tracers and walls (this kernel / that path, us).
// A workgroup walks all sources 256 at a time, 0.6 us a tile, however few targets
// there are: 1 target at 13,056 sources 36 / 37, at 26,112 67 / 52, at 984,064 3,120 /
// 359.  Up to there pairs count: 8,704 x 2,000 45 / 56, x 4,001 74 / 66, 4,400 x 8,001 69 / 63,
// shared 5,440 64 / 63 and 6,528 98 / 64.  Few tiles are staged so seldom that it keeps
// up longer: 600 x 128,001 92 / 111, 128 x 1,000,000 142 / 147, 1,100 x 128,001 160 / 157.  The
// double layer lies within 5% of these.  Mixed sums keep their sub-tiles' float32
// partial sums and stay on the other path.
bool direct_is_small(int mixed, int64_t n_src, int64_t n_trg) {
    constexpr int64_t kTiles = 72, kPairs = 26'000'000, kFewTiles = 5, kPairsFewTiles = 120'000'000;
    const int64_t tiles = ceil_div(n_src, (int64_t)kBlock);
    return !mixed && tiles <= kTiles && n_src <= (tiles <= kFewTiles ? kPairsFewTiles : kPairs) / n_trg;
}

hipError_t launch_direct_small(const SumInputs& in, double* out, int accumulate, int n_cu, hipStream_t stream,
                               const KernelTimer& timer) {
    if (timer.on()) (void)hipEventRecord(timer.start, stream);
    if (in.kernel == 0) launch_small_kt<0>(in, out, accumulate, n_cu, stream);
    else launch_small_kt<1>(in, out, accumulate, n_cu, stream);
    const hipError_t e = hipGetLastError();
    if (timer.on()) (void)hipEventRecord(timer.stop, stream);
    return e;
}

hipError_t launch_prep(const SumInputs& in, int64_t n_pad, void* rec, void* aux, SubMeta* meta,
                       hipStream_t stream) {
    const dim3 grid((unsigned)(n_pad / kBlock)), block(kBlock);
    if (in.kernel == 0) {
        if (in.mixed) prep_sources<0, 1><<<grid, block, 0, stream>>>(in, rec, aux, meta);
        else prep_sources<0, 0><<<grid, block, 0, stream>>>(in, rec, aux, meta);
    } else {
        if (in.mixed) prep_sources<1, 1><<<grid, block, 0, stream>>>(in, rec, aux, meta);
        else prep_sources<1, 0><<<grid, block, 0, stream>>>(in, rec, aux, meta);
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void fill_zero(double* out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) out[i] = 0.0;
}

hipError_t launch_fill_zero(double* out, int64_t n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    fill_zero<<<dim3((unsigned)ceil_div(n, kBlock)), dim3(kBlock), 0, stream>>>(out, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// planning and launch
// ---------------------------------------------------------------------------
constexpr int kT64 = STOKES_DIRECT_T64;
constexpr int kT32 = STOKES_DIRECT_T32;

static size_t rec_bytes(int kernel, int mixed) {
    if (!mixed) return kernel == 0 ? sizeof(SrcSL64x) : sizeof(SrcDL64);
    return kernel == 0 ? sizeof(SrcSL32) : sizeof(SrcDL32);
}

int direct_blocks_per_cu(int kernel, int mixed) {
    int nb = 0;
    hipError_t e;
    if (kernel == 0)
        e = mixed ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, direct_mixed<0, kT32>, kBlock, 0)
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, direct_f64<0, kT64>, kBlock, 0);
    else
        e = mixed ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, direct_mixed<1, kT32>, kBlock, 0)
                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, direct_f64<1, kT64>, kBlock, 0);
    return (e == hipSuccess && nb > 0) ? nb : 1;
}

// Targets per lane.  A long double-layer sum runs at the clock that the power
// limit leaves it, and half the LDS reads per pair raise that: 294,912 wall nodes
// at 115,217 targets 27.9 ms with 4, 27.1 with 8; 32,768 at 30,720 811 and 801 us.
// Below about 9e8 pairs the waves in flight count for more (16,384 at 30,720 414
// and 428 us), and so does more padding of the last target block than the
// difference (32,768 at 15,360 414 and 433).
static int targets_per_lane(int kernel, int mixed, int64_t n_src, int64_t n_trg) {
    if (mixed) return kT32;
    if (kernel == 0 || n_src <= 900'000'000 / n_trg) return kT64;
    const int64_t b4 = ceil_div(n_trg, (int64_t)kBlock * kT64), b8 = ceil_div(n_trg, (int64_t)kBlock * kT64Long);
    return (kT64Long * b8 - kT64 * b4) * 64 <= kT64 * b4 ? kT64Long : kT64;
}

// Workgroups with at least this many 256-source chunks each take whole chunks.
constexpr int64_t kWholeChunks = 16;

// Step through a target block's n chunks that deals any run of them evenly to its
// ranges: coprime to n, near its golden section.  Check points lie in the boxes of
// their own patch's sources, so one range of eight had the block's masked sub-tiles;
// a boundary product of 6,144 nodes (98,304 sources at 55,296 check points) 5.78 ms
// in order, 4.86 so; of 13,824 nodes (2.75e10 pairs) 24.2 and 22.6; sources and
// targets apart, 98,304 at 55,296, 4.44 and 4.47.
static int64_t spread_step(int64_t n) {
    int64_t s = std::max<int64_t>(1, (int64_t)(0.618034 * (double)n));
    while (std::gcd(s, n) != 1) ++s;
    return s;
}

DirectPlan plan_direct(int kernel, int mixed, int64_t n_src, int64_t n_trg, int resident_blocks,
                       int forced_grid, size_t max_bytes) {
    DirectPlan p{};
    p.T = targets_per_lane(kernel, mixed, n_src, n_trg);
    p.n_src_pad = ceil_div(n_src, kTile) * kTile;
    p.blocks_x = ceil_div(n_trg, (int64_t)kBlock * p.T);
    const int64_t subs = ceil_div(n_src, (int64_t)kSub), chunks = p.n_src_pad / kTile;
    const size_t bt = (size_t)kBlock * p.T;
    size_t off = 0;
    p.off_src = off;
    off = align_up(off + (size_t)p.n_src_pad * rec_bytes(kernel, mixed), 256);
    p.off_grp = off;
    off = align_up(off + (size_t)p.n_src_pad * (mixed ? sizeof(float4) : sizeof(int32_t)), 256);
    p.off_meta = off;
    off = align_up(off + (size_t)(p.n_src_pad / kSub) * sizeof(SubMeta), 256);
    p.off_part = off;
    int64_t g = forced_grid > 0 ? forced_grid : std::max(1, resident_blocks);
    if (forced_grid <= 0 && p.T == kT64Long) g = std::max<int64_t>(1, g * kW64Long / STOKES_DIRECT_W64);
    // Units are the sub-tiles that hold sources, not those that pad the last chunk:
    // with 64 sources those were three of four workgroups and of four partial sums a
    // target (64 x 1,000,000 mixed 164 us with them, 122 without).  Ranges of whole
    // chunks keep them, as they begin at multiples of four.
    auto partials = [&](int64_t workgroups, int slices) {
        p.grid = std::max<int64_t>(1, workgroups);
        p.near_slices = slices;
        p.cut = chunks * p.blocks_x >= kWholeChunks * p.grid ? kTile / kSub : 1;
        p.n_sub = p.cut > 1 ? p.n_src_pad / kSub : subs;
        p.step = p.cut > 1 && !mixed ? spread_step(chunks) : 1;
        p.units = p.n_sub * p.blocks_x;
        p.off_near = align_up(p.off_part + (size_t)(p.grid + p.blocks_x) * 3 * bt * sizeof(double), 256);
        p.total = align_up(p.off_near + (size_t)slices * p.blocks_x * 3 * bt * sizeof(double), 256);
    };
    partials(std::min(g, subs * p.blocks_x), mixed ? near_slices(p.blocks_x, subs) : 0);
    // few near-pass rows and no more workgroups than 256-source chunks where the
    // partial sums would not fit, and for the small calls that run as one kernel; then
    // as many workgroups as fit
    const int64_t whole = std::min(g, chunks * p.blocks_x);
    const int rows = mixed ? (int)std::min<int64_t>(kNearSlices, subs) : 0;
    if ((max_bytes > 0 && p.total > max_bytes) || direct_is_small(mixed, n_src, n_trg))
        partials(whole, rows);
    if (max_bytes > 0 && p.total > max_bytes) {
        const size_t row = 3 * bt * sizeof(double), fixed = p.off_part + 512 + (size_t)rows * p.blocks_x * row;
        const int64_t fit = fixed < max_bytes ? (int64_t)((max_bytes - fixed) / row) - p.blocks_x : 1;
        partials(std::max<int64_t>(1, std::min(whole, fit)), rows);
    }
    return p;
}

// The measure that the static-scratch entry point accepts sizes by: the lean
// layout's records and partial sums with 3 (float64) or 4 (mixed) workgroups per
// CU, and a byte per (wave, 256-source chunk).  plan_direct with max_bytes fits
// wherever this does.
size_t direct_scratch_measure(int kernel, int mixed, int64_t n_src, int64_t n_trg, int n_cu, int forced_grid) {
    const DirectPlan p = plan_direct(kernel, mixed, n_src, n_trg, 1, 1);
    const int64_t chunks = p.n_src_pad / kTile, units = chunks * p.blocks_x;
    const int64_t g = forced_grid > 0 ? forced_grid : (int64_t)(mixed ? 4 : 3) * n_cu;
    const size_t row = (size_t)3 * kBlock * p.T * sizeof(double);
    size_t off = align_up(p.off_part + (std::max<int64_t>(1, std::min(g, units)) + p.blocks_x) * row, 256);
    off = align_up(off + kNearSlices * p.blocks_x * row, 256);
    return align_up(off + (size_t)p.blocks_x * 4 * (size_t)chunks, 256);
}

template <int KT, int MIXED, int T = MIXED ? kT32 : kT64>
static hipError_t launch_typed(const SumInputs& in, const DirectPlan& p, double* out, int accumulate,
                               void* ws, hipStream_t stream, const KernelTimer& timer) {
    char* base = static_cast<char*>(ws);
    void* rec = base + p.off_src;
    void* aux = base + p.off_grp;
    SubMeta* meta = reinterpret_cast<SubMeta*>(base + p.off_meta);
    prep_sources<KT, MIXED><<<dim3((unsigned)(p.n_src_pad / kBlock)), dim3(kBlock), 0, stream>>>(
        in, rec, aux, meta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    DirectArgs a;
    a.in = in;
    a.rec = rec;
    a.aux = aux;
    a.meta = meta;
    a.n_sub = p.n_sub;
    a.units = p.units;
    a.cut = p.cut;
    a.step = p.step;
    a.part = reinterpret_cast<double*>(base + p.off_part);
    a.near_part = reinterpret_cast<double*>(base + p.off_near);
    if (timer.on()) (void)hipEventRecord(timer.start, stream);
    if constexpr (MIXED != 0) {
        if (in.pair_class)
            direct_mixed<KT, T, true><<<dim3((unsigned)p.grid), dim3(kBlock), 0, stream>>>(a);
        else
            direct_mixed<KT, T><<<dim3((unsigned)p.grid), dim3(kBlock), 0, stream>>>(a);
    } else
        direct_f64<KT, T><<<dim3((unsigned)p.grid), dim3(kBlock), 0, stream>>>(a);
    e = hipGetLastError();
    if (timer.on()) (void)hipEventRecord(timer.stop, stream);
    if (e != hipSuccess) return e;
    if constexpr (MIXED != 0) {
        const dim3 near_grid((unsigned)p.blocks_x, (unsigned)p.near_slices);
        auto near = [&](auto few) {
            constexpr bool F = decltype(few)::value;
            if (in.pair_class)
                direct_near_mixed<KT, T, F, true><<<near_grid, dim3(kBlock), 0, stream>>>(a);
            else
                direct_near_mixed<KT, T, F><<<near_grid, dim3(kBlock), 0, stream>>>(a);
        };
        if (p.n_sub <= kFewSubs) near(std::true_type{});
        else near(std::false_type{});
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // FP64 pair sums are 4x (single layer) or 8x (double layer) the bare sums
    const double pref = MIXED ? in.pref : (KT == 0 ? 0.25 : 0.125) * in.pref;
    auto reduce = [&](auto parts) {
        constexpr int P = decltype(parts)::value;
        reduce_segments<T, P><<<dim3((unsigned)ceil_div(in.n_trg, kBlock / P)), dim3(kBlock), 0, stream>>>(
            a.part, a.near_part, in.n_trg, p.units, p.n_sub, p.grid, p.cut, p.near_slices,
            p.blocks_x * (int64_t)kBlock * T, pref, out, accumulate);
    };
    // threads that share a target pay from about two partial sums each on (400,000 targets
    // with 4 or 5: 20 us shared, 10 alone)
    if (p.grid + p.near_slices * p.blocks_x < 2 * kRedParts * p.blocks_x) reduce(std::integral_constant<int, 1>{});
    else reduce(std::integral_constant<int, kRedParts>{});
    return hipGetLastError();
}

hipError_t launch_direct(const SumInputs& in, const DirectPlan& p, double* out, int accumulate,
                         void* ws, hipStream_t stream, const KernelTimer& timer) {
    if (in.n_trg <= 0) return hipSuccess;
    if (in.n_src <= 0) return accumulate ? hipSuccess : launch_fill_zero(out, 3 * in.n_trg, stream);
    if (in.kernel == 0) {
        return in.mixed ? launch_typed<0, 1>(in, p, out, accumulate, ws, stream, timer)
                        : launch_typed<0, 0>(in, p, out, accumulate, ws, stream, timer);
    }
    return in.mixed ? launch_typed<1, 1>(in, p, out, accumulate, ws, stream, timer)
           : p.T == kT64Long
               ? launch_typed<1, 0, kT64Long>(in, p, out, accumulate, ws, stream, timer)
               : launch_typed<1, 0>(in, p, out, accumulate, ws, stream, timer);
}

}  // namespace stokes
