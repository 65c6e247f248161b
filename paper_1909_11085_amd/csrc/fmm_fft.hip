// Multipole-to-local translations as lattice convolutions.
//
// The upward equivalent and downward check surfaces of all boxes of a level
// lie on one lattice: p points per edge at 1.05 half-widths, the same spacing
// for both.  So the check velocity at lattice point a of a target box from the
// density at lattice point b of a source box at offset o (in box widths)
// depends on a - b only,
//     V_a = sum_o sum_b K_o(a - b) q_b,
// a convolution, diagonal in the Fourier basis of the lattice padded to
// N = 2 p - 1 points per axis (a - b takes 2 p - 1 values, so nothing wraps).
// Against one dense (3 ns x 3 ns) product per offset this does 9 complex
// products per frequency: at p = 6 about 24,000 multiply-adds instead of
// 208,000 per box pair.
//
//   fft_forward_kernel    spectra of the source octets (the 8 children of a box
//                         together), separable over the axes, plane by plane
//                         in kz; HBM-bound writes, 384 contiguous bytes per
//                         (frequency, octet)
//   fft_translate_kernel  per frequency, the products with the 26 neighbouring
//                         octets as FP64 MFMA tiles (see there)
//   fft_inverse_kernel    back to the check points
//
// Measured (all M2L kernels of one evaluation): order 4 on the 261,120 points of
// 480 cells at depth 5, 1.11 ms of dense products before, 0.33 ms; order 6, the
// leaf level (depth 6) of the double layer of 1,048,576 wall nodes at 522,240 points,
// 8.0 ms of pair sums before, 2.8 ms, and 0.4 ms of the exact pseudo-inverse product.
//
// The spectra buffers hold a batch of kz planes, and at the targets a share of
// the octets; a level whose octets could be too many runs several.  Every sum has
// a fixed order, which the batches do not change.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "fmm_fft.hpp"

namespace stokes {
namespace {

// Bytes of the source octets' spectra before planes are split, and of the target
// octets' before those are.  More batches cost launches and reads of the densities:
// 1,048,576 wall nodes at 522,240 points, order 6, depth 6, 10.3 ms with these, 10.6
// with 1 GiB and 640 MiB; order 4, 300,000 points of a shell at depth 6, 3.74 and 3.90.
constexpr size_t kFftSrcBytes = (size_t)3200 << 20, kFftTrgBytes = (size_t)3200 << 20;
constexpr int kFftSplitMax = 512;                    // octets up to which the four waves of a workgroup share a tile
constexpr int kFftNT = 2;                            // 16-column tiles per wave when they do not

typedef double v4d __attribute__((ext_vector_type(4)));

// Surface point number of lattice point (i, j, k), x slowest (the order of the
// cube-surface template); -1 inside.
template <int P>
__device__ __forceinline__ int surf_index(int i, int j, int k) {
    if (i == 0) return j * P + k;
    if (i == P - 1) return P * P + (P - 2) * 4 * (P - 1) + j * P + k;
    const int ring = P * P + (i - 1) * 4 * (P - 1);
    if (j == 0) return ring + k;
    if (j == P - 1) return ring + P + 2 * (P - 2) + k;
    if (k == 0) return ring + P + 2 * (j - 1);
    if (k == P - 1) return ring + P + 2 * (j - 1) + 1;
    return -1;
}

// ------------------------------------------------------------------ the plan
// One workgroup per offset o: the spectra of the six entries of the symmetric
// kernel block and of the point-source velocity, each entry as a plain
// separable transform of its samples.  Per entry (re, im, -im), so that a lane
// of the translation picks its real coefficient by address; the flux column
// (re, im).  Offsets of adjacent boxes are zero.
__global__ __launch_bounds__(256) void spectra_kernel(int p, double alpha, const double* __restrict__ tw,
                                                      double* __restrict__ khat) {
    constexpr int kN = fft_n(kFftMaxOrder);
    __shared__ double2 A[kN * kN], B[kN * kN], w[kN];
    const int N = fft_n(p), o = blockIdx.x;
    const int ox[3] = {o / 49 - 3, o / 7 % 7 - 3, o % 7 - 3};
    const bool adjacent = abs(ox[0]) <= 1 && abs(ox[1]) <= 1 && abs(ox[2]) <= 1;
    const double step = 2.0 * alpha / (p - 1);
    if ((int)threadIdx.x < N) w[threadIdx.x] = make_double2(tw[2 * threadIdx.x], tw[2 * threadIdx.x + 1]);
    for (int e = 0; e < 9; ++e) {                       // xx xy xz yy yz zz, then the flux columns x y z
        const int ea = e < 3 ? 0 : e < 5 ? 1 : e == 5 ? 2 : e - 6, eb = e < 3 ? e : e < 5 ? e - 2 : 2;
        for (int kz = 0; kz < p; ++kz) {
            __syncthreads();
            for (int t = threadIdx.x; t < N * N; t += 256) {
                const int n[2] = {t / N, t % N};
                double2 s = make_double2(0.0, 0.0);
                for (int z = 0; z < N && !adjacent; ++z) {
                    double r[3];
                    bool in = true;
                    for (int c = 0; c < 3; ++c) {
                        const int m = c < 2 ? n[c] : z;
                        r[c] = e < 6 ? step * (m < p ? m : m - N) - 2.0 * ox[c] : (step * m - alpha) - 2.0 * ox[c];
                        in = in && (e < 6 || m < p);
                    }
                    if (!in) continue;
                    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2], ri = 1.0 / sqrt(r2);
                    const double k = e < 6 ? (ea == eb ? ri : 0.0) + r[ea] * r[eb] * (ri * ri * ri)
                                           : 2.0 * r[ea] * (ri * ri * ri);
                    const double2 c = w[kz * z % N];
                    s.x += k * c.x;
                    s.y -= k * c.y;
                }
                A[t] = s;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < N * N; t += 256) {    // over y
                const int ix = t / N, ky = t % N;
                double2 s = make_double2(0.0, 0.0);
                for (int y = 0; y < N; ++y) {
                    const double2 v = A[ix * N + y], c = w[ky * y % N];
                    s.x += v.x * c.x + v.y * c.y;
                    s.y += v.y * c.x - v.x * c.y;
                }
                B[t] = s;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < N * N; t += 256) {    // over x
                const int ky = t / N, kx = t % N;
                int f = fft_first(p, kz);
                if (kz > 0) f += t;
                else if (ky == 0 && kx < p) f += kx;
                else if (ky > 0 && ky < p) f += p + (ky - 1) * N + kx;
                else continue;
                double2 s = make_double2(0.0, 0.0);
                for (int x = 0; x < N; ++x) {
                    const double2 v = B[x * N + ky], c = w[kx * x % N];
                    s.x += v.x * c.x + v.y * c.y;
                    s.y += v.y * c.x - v.x * c.y;
                }
                double* out = khat + (int64_t)f * kFftOpStride;
                if (e < 6) {
                    out += o * 18 + e * 3;
                    out[0] = s.x;
                    out[1] = s.y;
                    out[2] = -s.y;
                } else {
                    out += kFftOffsets * 18 + o * 6 + (e - 6) * 2;
                    out[0] = s.x;
                    out[1] = s.y;
                }
            }
        }
    }
}

__global__ void twiddle_kernel(int N, double* tw) {
    const int k = threadIdx.x;
    if (k < N) sincospi(2.0 * k / N, &tw[2 * k + 1], &tw[2 * k]);
}

// ------------------------------------------------------------------ forward
__host__ __device__ constexpr int fft_threads(int p) { return (24 * fft_n(p) + kWave - 1) / kWave * kWave; }

// One source octet at a time, planes k0 .. k1 - 1; octet *n_soct is a record of
// zeros that stands for missing neighbours.  Series cc = 3 child + component.
template <int P>
__global__ __launch_bounds__(fft_threads(P)) void fft_forward_kernel(FftLevel a, const double* __restrict__ tw,
                                                                     int k0, int k1) {
    constexpr int N = fft_n(P), NT = fft_threads(P);
    __shared__ double2 A[24 * P * P], B[24 * P * N];
    const int64_t n = *a.n_soct;
    const int tid = threadIdx.x;
    const int f0 = fft_first(P, k0);
    for (int64_t i = blockIdx.x; i <= n; i += gridDim.x) {
        const int64_t box0 = i < n ? (int64_t)a.soct[i] * 8 : -1;
        if (a.sig && tid < 8)
            a.sigq[i * 8 + tid] =
                box0 >= 0 && a.sslot[box0 + tid] >= 0 ? a.sig[box0 + tid] * a.inv_h : 0.0;
        for (int kz = k0; kz < k1; ++kz) {
            if (box0 >= 0) {
                for (int e = tid; e < 24 * P * P; e += NT) {                  // over z
                    const int cc = e / (P * P), ix = e / P % P, iy = e % P;
                    const int64_t box = box0 + cc / 3;
                    double2 s = make_double2(0.0, 0.0);
                    if (a.sslot[box] >= 0) {
                        const double* d = a.ue + box * a.n3 + cc % 3;
                        const bool rim = ix == 0 || iy == 0 || ix == P - 1 || iy == P - 1;
                        const int iz_step = rim ? 1 : P - 1;
                        for (int iz = 0; iz < P; iz += iz_step) {
                            const double v = d[3 * surf_index<P>(ix, iy, iz)];
                            const int k = kz * iz % N;
                            s.x = __builtin_fma(v, tw[2 * k], s.x);
                            s.y = __builtin_fma(-v, tw[2 * k + 1], s.y);
                        }
                    }
                    A[e] = s;
                }
                __syncthreads();
                for (int e = tid; e < 24 * P; e += NT) {                      // over y: e = cc * P + ix
                    double2 v[P];
#pragma unroll
                    for (int y = 0; y < P; ++y) v[y] = A[e * P + y];
#pragma unroll
                    for (int ky = 0; ky < N; ++ky) {
                        double2 s = make_double2(0.0, 0.0);
#pragma unroll
                        for (int y = 0; y < P; ++y) {
                            const double c = tw[2 * (ky * y % N)], w = tw[2 * (ky * y % N) + 1];
                            s.x = __builtin_fma(v[y].x, c, __builtin_fma(v[y].y, w, s.x));
                            s.y = __builtin_fma(v[y].y, c, __builtin_fma(-v[y].x, w, s.y));
                        }
                        B[e * N + ky] = s;
                    }
                }
                __syncthreads();
            }
            const int cc = tid % 24, ky = tid / 24;
            if (ky < N && (kz > 0 || ky < P)) {                               // over x
                double2 v[P];
#pragma unroll
                for (int x = 0; x < P; ++x) v[x] = box0 >= 0 ? B[(cc * P + x) * N + ky] : make_double2(0.0, 0.0);
                const int f = fft_first(P, kz) - f0 + (kz > 0 ? ky * N : ky == 0 ? 0 : P + (ky - 1) * N);
                const int m = kz > 0 || ky > 0 ? N : P;
                double* q = a.q + ((int64_t)f * (n + 1) + i) * kFftRow + 2 * cc;
#pragma unroll
                for (int kx = 0; kx < N; ++kx) {
                    double2 s = make_double2(0.0, 0.0);
#pragma unroll
                    for (int x = 0; x < P; ++x) {
                        const double c = tw[2 * (kx * x % N)], w = tw[2 * (kx * x % N) + 1];
                        s.x = __builtin_fma(v[x].x, c, __builtin_fma(v[x].y, w, s.x));
                        s.y = __builtin_fma(v[x].y, c, __builtin_fma(-v[x].x, w, s.y));
                    }
                    if (kx < m) *reinterpret_cast<double2*>(q + (int64_t)kx * (n + 1) * kFftRow) = s;
                }
            }
            // the next plane or octet rewrites A, last read before the second barrier, and B after its own first
        }
    }
}

// ------------------------------------------------------------------ translate
// Per frequency the 8 x 3 complex check values of a target octet are a real
// 48 x 48 matrix times the 48 values of each neighbouring source octet, for
// each of the 26 directions d, the matrix of direction d built from the 343
// offsets' symmetric 3 x 3 spectra (o = 2 d + source child - target child; the
// adjacent offsets hold zeros: 9% of the work).  MFMA 16 x 16 x 4 with octets as
// columns:
//   rows     tile a = component; row r of a tile: (c', child) with c' = re / im
//            = (r >> 2) & 1 and child = (r & 3) + 4 (r >> 3), so that the four
//            accumulator entries of a lane are (re, im) of children g and g + 4,
//            g = lane >> 4, and every lane stores whole complex values;
//   K steps  (child z bit, b, c): lane group g supplies source child g + 4 sz, so
//            a lane's B entries are consecutive complex values of its column;
//   A        the frequency's spectra in LDS (49 KB, with the flux columns 66 KB).
//            With this order the LDS address is a per-lane constant plus the
//            direction's base plus compile-time offsets.
// A wave owns 16 NT columns and keeps the next direction's B in registers while
// it multiplies; a direction that no column has is skipped.  FP64 vector and
// matrix instructions share the issue port here (their times add when both
// run), so the loop holds nothing but MFMAs, LDS reads and loads.  SPLIT (few
// octets): the four waves share one tile, each takes every fourth direction and
// the partial sums are added in wave order.  Workgroups take equal ranges of
// (frequency, tile) units; consecutive ranges sit on one XCD, so the spectra of
// the frequencies in work stay in its L2.
template <int NT, bool SPLIT, bool FLUX>
__global__ __launch_bounds__(256, 2) void fft_translate_kernel(FftLevel a, int64_t f0, int64_t nf) {
    constexpr int kOp = kFftOffsets * 18, kOpAll = kOp + (FLUX ? kFftOffsets * 6 : 0);
    constexpr int COLS = SPLIT ? 16 * NT : 64 * NT;
    constexpr int kPart = 3 * NT * 4 * kWave;               // doubles of a wave's accumulators
    __shared__ __attribute__((aligned(16))) double s_op[kOpAll];
    __shared__ double s_red[SPLIT ? 3 * kPart : 1];
    const int64_t nt = *a.n_toct, ns = *a.n_soct, t1 = min(nt, a.t0 + a.tn);
    if (t1 <= a.t0) return;
    const int64_t tiles = (t1 - a.t0 + COLS - 1) / COLS, U = tiles * nf, G = gridDim.x;
    const int64_t idx = (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);     // G is a multiple of 8
    const int64_t u0 = idx * U / G, u1 = (idx + 1) * U / G;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int g = lane >> 4, row = lane & 15;
    // A address of this lane: offset index of (source child g, target child t) relative to the direction's
    const int t = (row & 3) + 4 * (row >> 3), cim = (row >> 2) & 1;
    const int rel = ((g & 1) * 49 + (g >> 1) * 7) - ((t & 1) * 49 + ((t >> 1) & 1) * 7 + (t >> 2));
    const int a0 = rel * 18 + (cim ? 1 : 0), a1 = rel * 18 + (cim ? 0 : 2), as = kOp + rel * 6 + cim;
    const int nd = SPLIT ? (26 - wave + 3) / 4 : 26;

    int64_t f = u0 / tiles, tile = u0 % tiles, loaded = -1;
    for (int64_t u = u0; u < u1; ++u) {
        if (f != loaded) {
            __syncthreads();
            const double2* src = reinterpret_cast<const double2*>(a.khat + (f0 + f) * kFftOpStride);
            for (int e = threadIdx.x; e < kOpAll / 2; e += 256) reinterpret_cast<double2*>(s_op)[e] = src[e];
            loaded = f;
            __syncthreads();
        }
        const int64_t col0 = a.t0 + tile * COLS + (SPLIT ? 0 : wave * 16 * NT);
        v4d acc[3][NT];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < NT; ++k) acc[i][k] = v4d{0.0, 0.0, 0.0, 0.0};
        const double* q = a.q + f * (ns + 1) * kFftRow + g * 6;
        auto direction = [&](int i) { return SPLIT ? wave + 4 * i : i; };
        auto slots = [&](int i, int32_t (&s)[NT]) {
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const int64_t col = col0 + 16 * k + row;
                s[k] = i < nd && col < t1 ? a.nbr[direction(i) * nt + col] : (int32_t)ns;
            }
        };
        struct Frag { double2 b[NT][6]; double s[NT][2]; };
        auto fetch = [&](const int32_t (&s)[NT], Frag& r) {
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const double2* p = reinterpret_cast<const double2*>(q + (int64_t)s[k] * kFftRow);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    r.b[k][j] = p[j];
                    r.b[k][3 + j] = p[12 + j];
                }
                if constexpr (FLUX) {
                    r.s[k][0] = a.sigq[(int64_t)s[k] * 8 + g];
                    r.s[k][1] = a.sigq[(int64_t)s[k] * 8 + g + 4];
                }
            }
        };
        auto multiply = [&](int i, const int32_t (&s)[NT], const Frag& r) {
            bool any = false;
#pragma unroll
            for (int k = 0; k < NT; ++k) any = any || s[k] != (int32_t)ns;
            if (__ballot(any) == 0) return;
            const int dd = direction(i), id = dd + (dd >= 13 ? 1 : 0);
            const int base = ((2 * (id / 9) + 1) * 7 + 2 * (id / 3 % 3) + 1) * 7 + 2 * (id % 3) + 1;
            const double* p0 = s_op + base * 18 + a0;
            const double* p1 = s_op + base * 18 + a1;
            constexpr int sym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
            for (int sz = 0; sz < 2; ++sz)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    double x0[3], x1[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        x0[c] = p0[sz * 18 + sym[c][b] * 3];
                        x1[c] = p1[sz * 18 + sym[c][b] * 3];
                    }
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int k = 0; k < NT; ++k)
                            acc[c][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0[c], r.b[k][sz * 3 + b].x, acc[c][k], 0,
                                                                             0, 0);
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int k = 0; k < NT; ++k)
                            acc[c][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[c], r.b[k][sz * 3 + b].y, acc[c][k], 0,
                                                                             0, 0);
                }
            if constexpr (FLUX) {
                const double* ps = s_op + base * 6 + as;
#pragma unroll
                for (int sz = 0; sz < 2; ++sz)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int k = 0; k < NT; ++k)
                            acc[c][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(ps[sz * 6 + c * 2], r.s[k][sz], acc[c][k],
                                                                             0, 0, 0);
            }
        };
        if (SPLIT || col0 < t1) {
            int32_t s0[NT], s1[NT];
            Frag r0, r1;
            slots(0, s0);
            slots(1, s1);
            fetch(s0, r0);
            for (int i = 0; i < nd; i += 2) {
                int32_t n0[NT], n1[NT];
                fetch(s1, r1);
                slots(i + 2, n0);
                multiply(i, s0, r0);
                fetch(n0, r0);
                slots(i + 3, n1);
                if (i + 1 < nd) multiply(i + 1, s1, r1);
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                    s0[k] = n0[k];
                    s1[k] = n1[k];
                }
            }
        }
        if constexpr (SPLIT) {
            if (wave > 0) {
                double* p = s_red + (wave - 1) * kPart + lane;
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int k = 0; k < NT; ++k)
#pragma unroll
                        for (int r = 0; r < 4; ++r) p[((c * NT + k) * 4 + r) * kWave] = acc[c][k][r];
            }
            __syncthreads();
            if (wave == 0)
                for (int w = 0; w < 3; ++w)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int k = 0; k < NT; ++k)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                acc[c][k][r] += s_red[w * kPart + ((c * NT + k) * 4 + r) * kWave + lane];
            __syncthreads();
        }
        if (!SPLIT || wave == 0)
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const int64_t col = col0 + 16 * k + row;
                if (col >= t1) continue;
                double2* o = reinterpret_cast<double2*>(a.v + (f * a.tn + col - a.t0) * kFftRow + g * 6);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    o[c] = make_double2(acc[c][k][0], acc[c][k][1]);
                    o[12 + c] = make_double2(acc[c][k][2], acc[c][k][3]);
                }
            }
        if (++tile == tiles) {
            tile = 0;
            ++f;
        }
    }
}

// ------------------------------------------------------------------ inverse
// One target octet at a time: the planes' contributions to the check points,
// added into the boxes' columns plane by plane (plane 0 writes unless a.add).
template <int P>
__global__ __launch_bounds__(fft_threads(P)) void fft_inverse_kernel(FftLevel a, const double* __restrict__ tw,
                                                                     int k0, int k1) {
    constexpr int N = fft_n(P), NT = fft_threads(P);
    __shared__ double2 A[24 * P * P], B[24 * P * N];
    const int64_t t1 = min(*a.n_toct, a.t0 + a.tn), n = a.tn;
    const int tid = threadIdx.x;
    const int f0 = fft_first(P, k0);
    for (int64_t i = a.t0 + blockIdx.x; i < t1; i += gridDim.x) {
        const int64_t box0 = (int64_t)a.toct[i] * 8;
        for (int kz = k0; kz < k1; ++kz) {
            const int cc = tid % 24, ky = tid / 24;
            if (ky < N) {                                                     // over x
                // the half of plane 0 that is not kept is the conjugate of (-kx, -ky)
                const bool mirror = kz == 0 && ky >= P;
                const int kyr = mirror ? N - ky : ky;
                const int f = fft_first(P, kz) - f0 + (kz > 0 ? ky * N : kyr == 0 ? 0 : P + (kyr - 1) * N);
                const double* v = a.v + ((int64_t)f * n + i - a.t0) * kFftRow + 2 * cc;
                double2 s[P];
#pragma unroll
                for (int x = 0; x < P; ++x) s[x] = make_double2(0.0, 0.0);
#pragma unroll
                for (int kx = 0; kx < N; ++kx) {
                    const bool conj = mirror || (kz == 0 && ky == 0 && kx >= P);
                    const int kr = conj && kx > 0 ? N - kx : kx;
                    double2 t = *reinterpret_cast<const double2*>(v + (int64_t)kr * n * kFftRow);
                    if (conj) t.y = -t.y;
#pragma unroll
                    for (int x = 0; x < P; ++x) {
                        const double c = tw[2 * (kx * x % N)], w = tw[2 * (kx * x % N) + 1];
                        s[x].x = __builtin_fma(t.x, c, __builtin_fma(-t.y, w, s[x].x));
                        s[x].y = __builtin_fma(t.y, c, __builtin_fma(t.x, w, s[x].y));
                    }
                }
#pragma unroll
                for (int x = 0; x < P; ++x) B[(cc * P + x) * N + ky] = s[x];
            }
            __syncthreads();
            for (int e = tid; e < 24 * P; e += NT) {                          // over y
                double2 s[P];
#pragma unroll
                for (int y = 0; y < P; ++y) s[y] = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const double2 t = B[e * N + k];
#pragma unroll
                    for (int y = 0; y < P; ++y) {
                        const double c = tw[2 * (k * y % N)], w = tw[2 * (k * y % N) + 1];
                        s[y].x = __builtin_fma(t.x, c, __builtin_fma(-t.y, w, s[y].x));
                        s[y].y = __builtin_fma(t.y, c, __builtin_fma(t.x, w, s[y].y));
                    }
                }
#pragma unroll
                for (int y = 0; y < P; ++y) A[e * P + y] = s[y];
            }
            __syncthreads();
            const double wk = (kz > 0 ? 2.0 : 1.0) / (double)(N * N * N);
            for (int e = tid; e < 24 * P * P; e += NT) {                      // over z, real part
                const int c3 = e / (P * P), ix = e / P % P, iy = e % P;
                const int64_t col = a.tslot[box0 + c3 / 3];
                if (col < 0) continue;
                double* out = a.vbuf + col * a.mp + c3 % 3;
                const double2 t = make_double2(wk * A[e].x, wk * A[e].y);
                const bool rim = ix == 0 || iy == 0 || ix == P - 1 || iy == P - 1;
                const int iz_step = rim ? 1 : P - 1;
                for (int iz = 0; iz < P; iz += iz_step) {
                    const int k = kz * iz % N;
                    const double val = __builtin_fma(t.x, tw[2 * k], -t.y * tw[2 * k + 1]);
                    double* o = out + 3 * surf_index<P>(ix, iy, iz);
                    *o = kz > 0 || a.add ? *o + val : val;
                }
            }
            if (kz == 0 && !a.add)
                for (int e = tid; e < 8 * (a.mp - a.n3); e += NT) {           // the rows past n3
                    const int64_t col = a.tslot[box0 + e / (a.mp - a.n3)];
                    if (col >= 0) a.vbuf[col * a.mp + a.n3 + e % (a.mp - a.n3)] = 0.0;
                }
            // the next plane or octet rewrites B, last read before the second barrier, and A after its own first
        }
    }
}

template <typename F>
bool with_order(int p, F&& f) {
    switch (p) {
        case 2: f(std::integral_constant<int, 2>{}); return true;
        case 3: f(std::integral_constant<int, 3>{}); return true;
        case 4: f(std::integral_constant<int, 4>{}); return true;
        case 5: f(std::integral_constant<int, 5>{}); return true;
        case kFftMaxOrder: f(std::integral_constant<int, kFftMaxOrder>{}); return true;
        default: return false;
    }
}
static_assert(kFftMaxOrder == 6, "with_order covers 2 .. kFftMaxOrder");

size_t plane_bytes(int p, int64_t octets) { return (size_t)fft_n(p) * fft_n(p) * (size_t)octets * kFftRow * 8; }

// Most frequencies of a batch of `planes` consecutive planes.
size_t batch_freqs(int p, int planes) {
    return planes >= p ? (size_t)fft_freqs(p) : (size_t)planes * fft_n(p) * fft_n(p);
}

}  // namespace

size_t fft_spectra_bytes(int p) { return (size_t)fft_freqs(p) * kFftOpStride * 8; }

hipError_t fft_build_spectra(int p, double alpha, double* khat, double* tw, hipStream_t st) {
    hipLaunchKernelGGL(twiddle_kernel, dim3(1), dim3(kWave), 0, st, fft_n(p), tw);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(spectra_kernel, dim3(kFftOffsets), dim3(256), 0, st, p, alpha, tw, khat);
    return hipGetLastError();
}

FftBatches fft_batches(int p, int64_t max_soct, int64_t max_toct) {
    FftBatches r{};
    r.planes = (int)std::min<size_t>(p, std::max<size_t>(1, kFftSrcBytes / plane_bytes(p, max_soct + 1)));
    const size_t freqs = batch_freqs(p, r.planes), octet = freqs * kFftRow * 8;
    const int64_t fit = (int64_t)(kFftTrgBytes / octet) / 128 * 128;   // whole tiles; 13,056 octets or more
    r.tcols = std::min(max_toct, fit);
    r.q_bytes = (size_t)(max_soct + 1) * octet;
    r.v_bytes = (size_t)r.tcols * octet;
    return r;
}

hipError_t launch_fft_m2l(const FftLevel& level, int64_t max_soct, int64_t max_toct, int cus, hipStream_t st) {
    FftLevel a = level;
    const FftBatches bt = fft_batches(a.p, max_soct, max_toct);
    // grid-stride over the octets: enough workgroups to fill the chip with the smaller ones
    const unsigned gs = (unsigned)std::min<int64_t>(max_soct + 1, 8 * (int64_t)cus);
    const unsigned gt = (unsigned)std::min<int64_t>(bt.tcols, 8 * (int64_t)cus);
    // two workgroups fit a CU (registers); a level with few octets still has a unit per frequency
    const dim3 g((unsigned)((2 * cus + 7) / 8 * 8));
    const bool split = max_toct <= kFftSplitMax;
    hipError_t e = hipSuccess;
    for (int k0 = 0; k0 < a.p; k0 += bt.planes) {
        const int k1 = std::min(a.p, k0 + bt.planes);
        const int64_t f0 = fft_first(a.p, k0), nf = fft_first(a.p, k1) - f0;
        if (!with_order(a.p, [&](auto o) {
                hipLaunchKernelGGL(fft_forward_kernel<decltype(o)::value>, dim3(gs),
                                   dim3(fft_threads(decltype(o)::value)), 0, st, a, a.tw, k0, k1);
            }))
            return hipErrorInvalidValue;
        if ((e = hipGetLastError()) != hipSuccess) return e;
        for (a.t0 = 0; a.t0 < max_toct; a.t0 += bt.tcols) {
            a.tn = std::min(bt.tcols, max_toct - a.t0);
            if (split && a.sig) hipLaunchKernelGGL((fft_translate_kernel<1, true, true>), g, dim3(256), 0, st, a, f0, nf);
            else if (split) hipLaunchKernelGGL((fft_translate_kernel<1, true, false>), g, dim3(256), 0, st, a, f0, nf);
            else if (a.sig)
                hipLaunchKernelGGL((fft_translate_kernel<kFftNT, false, true>), g, dim3(256), 0, st, a, f0, nf);
            else hipLaunchKernelGGL((fft_translate_kernel<kFftNT, false, false>), g, dim3(256), 0, st, a, f0, nf);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            (void)with_order(a.p, [&](auto o) {
                hipLaunchKernelGGL(fft_inverse_kernel<decltype(o)::value>, dim3(gt),
                                   dim3(fft_threads(decltype(o)::value)), 0, st, a, a.tw, k0, k1);
            });
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return e;
}

}  // namespace stokes
