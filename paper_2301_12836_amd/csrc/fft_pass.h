// Shared by the FFT passes of the x and y axes (fft.hip) and of the z axis (fft_z.hip).
#pragma once

#include <cstring>

#include "fft_reg.h"

namespace ls {

constexpr int kThreads = 256;   // threads per block of the LDS Stockham kernels

// Supported FFT lengths: multiples of 16 whose quotient has register DFTs.  A grid of n cells per axis takes the
// smallest one >= 2 n - 1; neighbours differ by at most a quarter above 64 (a third at 192 with only 2^a and 3 2^a).
#define LS_FOR_LENGTHS(X)                                                                              \
    X(16) X(32) X(48) X(64) X(80) X(96) X(112) X(128) X(144) X(160) X(192) X(224) X(256) X(288) X(320) \
    X(384) X(448) X(512)
// lengths L = A x 16 whose A is no power of two: the asymmetric four-step kernels (k_fs_*3 to 256, k_fs_*3p above)
constexpr bool asym_length(int L) { return (L & (L - 1)) != 0; }

// Adjacent columns (lines, in the x passes) of a register four-step block: 128-byte row segments.
template <typename T>
constexpr int seg_cols() {
    return 128 / (int)sizeof(cpx<T>);
}

// Whether the x and y passes take the square four-step kernels (k_fs_strided, k_fs_contig): powers of two whose transpose
// buffer stays within 64 KB.  The other lengths have the asymmetric ones (asym_length).
template <typename T, int L>
constexpr bool fs_ok() {
    return (L & (L - 1)) == 0 && L * seg_cols<T>() * (int)sizeof(cpx<T>) <= 65536;
}

// Twiddles e^{-2 pi i m / L} copied to LDS once per block (cheaper than per-use global loads).
template <typename T, int L>
__device__ __forceinline__ void stage_twiddles(cpx<T>* tws, const cpx<T>* __restrict__ tw, int tid, int nthreads) {
    for (int m = tid; m < L; m += nthreads) tws[m] = tw[m];
}

// LS_FFT=stockham in the environment selects the LDS Stockham kernels everywhere (both paths are
// kept under test); otherwise the register four-step kernels run wherever they fit.
bool use_fourstep();

template <typename T>
const cpx<T>* twiddles(const Ctx* c, int L);
template <>
inline const z128* twiddles<double>(const Ctx* c, int L) { return c->twiddle128(L); }
template <>
inline const z64* twiddles<float>(const Ctx* c, int L) { return c->twiddle64(L); }

// The z pass over the positions of a set: forward z FFT, k-space Green's multiply, inverse z FFT, in place in the
// padded work buffer, with kernel variant 0 (registers) or 1 (LDS Stockham); see fft_z.hip.
template <typename T>
int z_green_pass(Ctx* c, const RhsSet& set, cpx<T>* work, int variant);

}  // namespace ls
