// Multipole-to-local translations of the FMM as convolutions on the surface
// lattice (discrete Fourier transforms of the densities, products per
// frequency on the FP64 matrix cores).  Internal, not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace stokes {

// Lattice of an order-p surface: p points per edge, N = 2 p - 1 per axis of the
// padded transform.  The half spectrum of real data is kept plane by plane in
// kz = 0 .. p - 1: planes kz > 0 whole (N^2 frequencies), plane 0 the half with
// ky = 0, kx < p or 0 < ky < p.
__host__ __device__ constexpr int fft_n(int p) { return 2 * p - 1; }
__host__ __device__ constexpr int fft_plane0(int p) { return (fft_n(p) * fft_n(p) + 1) / 2; }
__host__ __device__ constexpr int fft_first(int p, int kz) {      // frequencies before plane kz
    return kz == 0 ? 0 : fft_plane0(p) + (kz - 1) * fft_n(p) * fft_n(p);
}
__host__ __device__ constexpr int fft_freqs(int p) { return fft_first(p, p); }

constexpr int kFftMaxOrder = 6;                   // the highest order with a convolution level
constexpr int kFftOffsets = 343;                  // source minus target box, -3 .. 3 per axis
constexpr int kFftOpStride = kFftOffsets * 24;    // doubles per frequency: 18 per offset, then 6 (flux)
constexpr int kFftRow = 48;                       // doubles per octet and frequency: 8 children x 3 complex

// The translation spectra of order p on the device (fft_freqs(p) x
// kFftOpStride doubles) and the twiddles (fft_n(p) x (cos, sin)).
size_t fft_spectra_bytes(int p);
hipError_t fft_build_spectra(int p, double alpha, double* khat, double* tw, hipStream_t st);

// One level's translation.  Boxes are named by their Morton index in their
// level; octets are the boxes of the level above.
struct FftLevel {
    int p, n3, mp;
    const double* khat;
    const double* tw;
    const double* ue;            // n3 per box of the level
    const int32_t* sslot;        // per box of the level: >= 0 when it holds sources
    const int32_t* tslot;        // per box of the level: its column of vbuf, -1 when it holds no targets
    const int32_t* soct;         // octets holding sources, *n_soct of them
    const int64_t* n_soct;
    const int32_t* toct;         // octets holding targets
    const int64_t* n_toct;
    const int32_t* nbr;          // (26, *n_toct): source octet next to a target octet, *n_soct when none
    const double* sig;           // per box of the level: point-source flux (double layer), else null
    double inv_h;                // 1 / box half-width
    double* q;                   // spectra of the source octets of a batch of planes (plan.q_bytes)
    double* sigq;                // flux over h, 8 per source octet
    double* v;                   // spectra at a batch's share of the target octets (plan.v_bytes)
    int64_t t0, tn;              // that share: target octets t0 .. t0 + tn - 1 (set by the launch)
    double* vbuf;                // check vectors times h, mp per column
    bool add;                    // add to vbuf's columns instead of writing them
};

// The batches of a level with at most max_soct source and max_toct target
// octets: planes per batch, target octets at a time, and the bytes of the two
// spectra buffers.  The source octets' spectra take up to 3,200 MiB, or one plane's
// (2 p - 1)^2 x 384 bytes an octet where that is more; the target octets' up to
// 3,200 MiB.  The batches change no sum and no order of one.
struct FftBatches { int planes; int64_t tcols; size_t q_bytes, v_bytes; };
FftBatches fft_batches(int p, int64_t max_soct, int64_t max_toct);

// Writes (or adds) into the vbuf column of every box of the level that holds
// targets h times its check vector from the interaction lists; when writing,
// rows past n3 are set to zero.
hipError_t launch_fft_m2l(const FftLevel& a, int64_t max_soct, int64_t max_toct, int cus, hipStream_t st);

}  // namespace stokes
