// Time-domain seismograms from the frequency-domain solutions: receiver sampling of solved fields and the
// inverse Fourier transform over the solved frequencies (the paper's frequency loop up to Nyquist followed
// by an inverse transform; Ricker source wavelet of its Tables 1 and 3).
//
// Conventions: time dependence e^{-i w t}, spectra S(w) = int s(t) e^{i w t} dt; a real medium gives
// u(-w) = conj u(w), so only w_k = 2 pi k / (nt dt) >= 0 is solved and
//   u(t_n) = (1/(nt dt)) sum_k c_k Re[S(w_k) U_k e^{-i w_k t_n}],  c_k = 1 for k = 0 or 2k = nt, else 2.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace ls {

namespace {

// out[r][m][c] = u[r][c][cell_m]
__global__ void k_sample(const z128* __restrict__ u, const int* __restrict__ rec, z128* __restrict__ out, int nrhs,
                         int nrec, int N1, int N2, int N3) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (long long)nrhs * nrec * 3) return;
    const int c = (int)(q % 3), m = (int)((q / 3) % nrec), r = (int)(q / (3LL * nrec));
    const long long n = (long long)N1 * N2 * N3;
    const long long p = ((long long)rec[3 * m + 2] * N2 + rec[3 * m + 1]) * N1 + rec[3 * m];
    out[q] = u[((long long)r * 3 + c) * n + p];
}

// wavelet factor of each solved frequency: c_k S(w_k) / (nt dt), S the delayed Ricker spectrum
// (4 sqrt(pi) w^2 / wp^3) e^{-w^2/wp^2} e^{i w ts} (fp > 0) or 1 (fp <= 0: the traces of the fields)
__global__ void k_wavelet(const int* __restrict__ k, int nf, int nt, double dt, double fp, double ts,
                          z128* __restrict__ s) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nf) return;
    const double scale = ((k[q] == 0 || 2 * k[q] == nt) ? 1.0 : 2.0) / (nt * dt);
    if (fp <= 0.0) {
        s[q] = {scale, 0.0};
        return;
    }
    const double w = 2.0 * M_PI * k[q] / (nt * dt), wp = 2.0 * M_PI * fp;
    const double amp = scale * 4.0 * sqrt(M_PI) * w * w / (wp * wp * wp) * exp(-(w / wp) * (w / wp));
    double sn, cs;
    sincos(w * ts, &sn, &cs);
    s[q] = {amp * cs, amp * sn};
}

// traces[j][n] = sum_q Re[s_q U[q][j] e^{-2 pi i (k_q n mod nt) / nt}]
//
// Bound by the sines: one pair per sample and frequency serves COLS traces (their spectra are wave-uniform), and the four
// wavefronts of a block take a quarter of the frequencies each and are summed in order.  IDX: products k n in 32 bits
// where they fit (k <= nt / 2).  n0, j0: first sample and trace of the launch.
constexpr int kTraceWaves = 4;
template <typename IDX, int COLS>
__global__ __launch_bounds__(64 * kTraceWaves) void k_traces(const z128* __restrict__ U, const z128* __restrict__ s,
                                                             const int* __restrict__ k, int nf, int ntr, int nt, int n0,
                                                             int j0, double* __restrict__ tr) {
    __shared__ double part[kTraceWaves][COLS][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = n0 + (int)blockIdx.x * 64 + lane;
    j0 += (int)blockIdx.y * COLS;
    const int per = (nf + kTraceWaves - 1) / kTraceWaves, f1 = min(nf, (wave + 1) * per);
    double acc[COLS] = {};
    for (int f = wave * per; f < f1; ++f) {
        const IDX kn = ((IDX)k[f] * (IDX)n) % (IDX)nt;
        double sn, cs;
        sincospi(2.0 * (double)kn / nt, &sn, &cs);
        const z128 t = s[f] * z128{cs, -sn};
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const z128 a = U[(long long)f * ntr + min(j0 + j, ntr - 1)];
            acc[j] += a.x * t.x - a.y * t.y;
        }
    }
#pragma unroll
    for (int j = 0; j < COLS; ++j) part[wave][j][lane] = acc[j];
    __syncthreads();
    for (int j = wave; j < COLS; j += kTraceWaves) {
        double sum = 0.0;
        for (int w = 0; w < kTraceWaves; ++w) sum += part[w][j][lane];
        if (n < nt && j0 + j < ntr) tr[(long long)(j0 + j) * nt + n] = sum;
    }
}

int ensure_ints(Ctx* c, int count) {
    if (count <= c->ints_cap) return LS_OK;
    if (c->ints) LS_HIP(hipFree(c->ints));
    c->ints = nullptr;
    c->ints_cap = 0;
    LS_HIP(hipMalloc((void**)&c->ints, sizeof(int) * (size_t)count));
    c->ints_cap = count;
    return LS_OK;
}

}  // namespace

int sample_launch(Ctx* c, const z128* u, int nrhs, const int* rec_host, int nrec, z128* out) {
    int rc = ensure_ints(c, 3 * nrec);
    if (rc) return rc;
    LS_HIP(hipMemcpyAsync(c->ints, rec_host, sizeof(int) * 3 * (size_t)nrec, hipMemcpyHostToDevice, c->stream));
    const long long m = (long long)nrhs * nrec * 3;
    hipLaunchKernelGGL(k_sample, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, c->stream, u, c->ints, out, nrhs, nrec,
                       c->n1, c->n2, c->n3);
    LS_HIP(hipGetLastError());
    LS_HIP(hipStreamSynchronize(c->stream));  // the staged receiver list may be replaced by the next call
    return LS_OK;
}

int synthesize_launch(Ctx* c, const z128* U, const int* k_host, int nf, int ntr, int nt, double dt, double fp, double ts,
                      double* traces) {
    // staging: k [nf] ints, then the nf complex wavelet factors (16-byte aligned)
    const int kints = (nf + 3) / 4 * 4;
    int rc = ensure_ints(c, kints + 4 * nf);
    if (rc) return rc;
    int* dk = c->ints;
    z128* ds = (z128*)(c->ints + kints);
    LS_HIP(hipMemcpyAsync(dk, k_host, sizeof(int) * (size_t)nf, hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(k_wavelet, dim3((unsigned)((nf + 63) / 64)), dim3(64), 0, c->stream, dk, nf, nt, dt, fp, ts, ds);
    LS_HIP(hipGetLastError());
    // 16 traces a block where that still gives every CU a block, else 8.  Repeated calls with 8 / 16: 60 frequencies, 576
    // traces of 800 samples 39 / 36 us; 120, 1152 traces of 2000 139 / 108; 60, 9 traces of 800 31 / 32.  (The first of
    // these, single calls: 140 us with a pair of sines per trace, now 59.)  One launch covers 2^20 samples of 65535
    // tiles of traces.
    const int cols = (long long)((nt + 63) / 64) * ((ntr + 15) / 16) >= 256 ? 16 : 8;
    const auto kernel = nt <= 65536 ? (cols == 16 ? k_traces<unsigned, 16> : k_traces<unsigned, 8>)
                                    : (cols == 16 ? k_traces<unsigned long long, 16> : k_traces<unsigned long long, 8>);
    const long long samples = 1 << 20, cap = 65535LL * cols;
    for (long long j0 = 0; j0 < ntr; j0 += cap)
        for (long long n0 = 0; n0 < nt; n0 += samples) {
            const dim3 g((unsigned)((std::min(samples, nt - n0) + 63) / 64),
                         (unsigned)((std::min(cap, ntr - j0) + cols - 1) / cols));
            hipLaunchKernelGGL(kernel, g, dim3(64 * kTraceWaves), 0, c->stream, U, ds, dk, nf, ntr, nt, (int)n0, (int)j0,
                               traces);
        }
    LS_HIP(hipGetLastError());
    LS_HIP(hipStreamSynchronize(c->stream));
    return LS_OK;
}

}  // namespace ls
