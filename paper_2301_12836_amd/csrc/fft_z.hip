// The z pass of the zero-padded convolution (Eq 21): forward z FFT of the three components of the padded work
// buffer, product with the k-space Green's tensor, inverse z FFT, in place (layout and pruning as in fft.hip).
#include "fft_pass.h"

namespace ls {

namespace {

// Adjacent columns per block of the LDS z pass (three components resident in LDS).
template <typename T, int L>
constexpr int zpass_cols() {
    constexpr int budget = 49152;  // bytes of LDS
    constexpr int tx = budget / (3 * L * (int)sizeof(cpx<T>));
    return tx >= 8 ? 8 : (tx >= 4 ? 4 : (tx >= 2 ? 2 : 1));
}

// k-space Green's table of each launch position (z passes), by value
template <typename T>
struct GreenTabs {
    const cpx<T>* g[kMaxRhs];
};

// Visit y and its mirror L2 - y in consecutive blocks so both read the same octant rows of G^: a
// permutation of 0..L2-1 for any count (an even count ends on its self-mirrored middle row L2/2).
__device__ __forceinline__ int paired_row(int by, int L2) {
    if (by == 0) return 0;
    if (L2 % 2 == 0 && by == L2 - 1) return L2 / 2;
    const int m = (by + 1) >> 1;
    return (by & 1) ? m : L2 - m;
}

// the six table entries (green_index) of the k-point whose row starts at byte `o` of the table for k_x = 0 plus the
// 16-byte offset of its column; GP = green_pitch
__device__ __forceinline__ void load_g6(const z64* __restrict__ ghat, size_t o, int GP, z64 g[6]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(ghat) + (size_t)k * GP * 16 + o);
        g[2 * k] = {a.x, a.y};
        g[2 * k + 1] = {a.z, a.w};
    }
}
__device__ __forceinline__ void load_g6(const z128* __restrict__ ghat, size_t o, int GP, z128 g[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double2 a = *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(ghat) + (size_t)k * GP * 16 + o);
        g[k] = {a.x, a.y};
    }
}
// 16-byte units per row and column of the table: 6 (FP64) or 3 (FP32) times the pitch
template <typename T>
constexpr int kGreenUnits = sizeof(T) == 8 ? 6 : 3;

// LDS Stockham z pass: forward z FFT of the three components, v^ = G^(k) f^, inverse z FFT.
// G^ holds the octant [L3/2+1][L2/2+1][6][green_pitch] (Voigt order 11,22,33,23,13,12); under
// k_a -> L_a - k_a an off-diagonal component ij changes sign once for each of i, j equal to a.
// HALF: G^ holds the half-space [L3][L2][6][green_pitch] (backgrounds without the mirror planes) and
// k_x > L1/2 reads the entry at -k (G^ is even), with no sign change.
template <typename T, int L, int TX, bool HALF = false, int ZBS = 0>
__global__ __launch_bounds__(kThreads) void k_fft_zgreen(cpx<T>* __restrict__ data, int nrhs, int L1, int L2,
                                                         long long CS, long long RS, long long ES, int n3,
                                                         GreenTabs<T> gt, const cpx<T>* __restrict__ tw) {
    constexpr int zbs = ZBS;   // work buffer layout (zplane_offset), fixed at compile time
    constexpr int NL = 3 * TX;
    __shared__ cpx<T> s[L * NL];
    const int tid = threadIdx.x;
    const int rhs = blockIdx.x % nrhs;
    const int x0 = (blockIdx.x / nrhs) * TX;
    const int y = paired_row(blockIdx.y, L2);
    const cpx<T>* __restrict__ ghat = gt.g[rhs];
    (void)ES;   // the plane pitch: element offsets follow zplane_offset
    cpx<T>* base = data + (long long)rhs * RS + zrow_offset(y, zbs, L1) + x0;
    for (int idx = tid; idx < L * NL; idx += kThreads) {
        const int t = idx % TX, c = (idx / TX) % 3, e = idx / NL;
        cpx<T> val = {T(0), T(0)};
        if (e < n3) val = base[c * CS + zplane_offset(e, zbs, L2, L1) + t];
        s[e * NL + c * TX + t] = val;
    }
    __syncthreads();
    lds_fft<T, L, NL, NL, kThreads, -1>(s, tw, tid);

    const int GP = green_pitch(L1), O2 = L2 / 2 + 1;
    const bool fy = y > L2 / 2;
    const int ky = fy ? L2 - y : y;
    for (int idx = tid; idx < L * TX; idx += kThreads) {
        const int t = idx % TX, kz0 = idx / TX;
        const int kx0 = x0 + t;
        cpx<T> g[6];
        if constexpr (HALF) {
            const bool neg = kx0 > L1 / 2;
            const int hx = neg ? L1 - kx0 : kx0, hy = neg ? (L2 - y) % L2 : y, hz = neg ? (L - kz0) % L : kz0;
            load_g6(ghat, (((size_t)hz * L2 + hy) * kGreenUnits<T> * GP + hx) * 16, GP, g);
        } else {
            const bool fx = kx0 > L1 / 2, fz = kz0 > L / 2;
            const int kx = fx ? L1 - kx0 : kx0, kz = fz ? L - kz0 : kz0;
            load_g6(ghat, (((size_t)kz * O2 + ky) * kGreenUnits<T> * GP + kx) * 16, GP, g);
            if (fy != fz) g[3] = T(-1) * g[3];
            if (fx != fz) g[4] = T(-1) * g[4];
            if (fx != fy) g[5] = T(-1) * g[5];
        }
        const cpx<T> g11 = g[0], g22 = g[1], g33 = g[2], g23 = g[3], g13 = g[4], g12 = g[5];
        cpx<T>* row = s + kz0 * NL + t;
        const cpx<T> f1 = row[0], f2 = row[TX], f3 = row[2 * TX];
        row[0] = g11 * f1 + g12 * f2 + g13 * f3;
        row[TX] = g12 * f1 + g22 * f2 + g23 * f3;
        row[2 * TX] = g13 * f1 + g23 * f2 + g33 * f3;
    }
    __syncthreads();
    lds_fft<T, L, NL, NL, kThreads, +1>(s, tw, tid);
    for (int idx = tid; idx < L * NL; idx += kThreads) {
        const int t = idx % TX, c = (idx / TX) % 3, e = idx / NL;
        if (e < n3) base[c * CS + zplane_offset(e, zbs, L2, L1) + t] = s[e * NL + c * TX + t];
    }
}

__device__ __forceinline__ void fold_index(int k, int L, int& kf, bool& flipped) {
    flipped = k > L / 2;
    kf = flipped ? L - k : k;
}

// a b + c with one rounding
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// g1 f1 + g2 f2 + g3 f3 as two chains of fused multiply-adds (12 operations instead of 16)
template <typename T>
__device__ __forceinline__ cpx<T> cdot3(cpx<T> g1, cpx<T> f1, cpx<T> g2, cpx<T> f2, cpx<T> g3, cpx<T> f3) {
    T re = g1.x * f1.x, im = g1.x * f1.y;
    re = fmadd(-g1.y, f1.y, re);
    im = fmadd(g1.y, f1.x, im);
    re = fmadd(g2.x, f2.x, re);
    im = fmadd(g2.x, f2.y, im);
    re = fmadd(-g2.y, f2.y, re);
    im = fmadd(g2.y, f2.x, im);
    re = fmadd(g3.x, f3.x, re);
    im = fmadd(g3.x, f3.y, im);
    re = fmadd(-g3.y, f3.y, re);
    im = fmadd(g3.y, f3.x, im);
    return {re, im};
}

// ------------------------------------------------------------------------------------------
// Register z pass.
//
// Four-step split of a z line of L = A x B points (n = n1 + A n2, k = k2 + B k1; n1, k1 < A; n2, k2 < B):
//   X[k2 + B k1] = sum_{n1} W_A^{n1 k1} W_L^{n1 k2} sum_{n2} W_B^{n2 k2} x[n1 + A n2].
// Threads q < A run the length-B DFT of the elements q + A n2 (n2 < B/2: the data occupy z < L/2) and the twiddles
// W_L^{q k2}; after one LDS transpose thread q < B holds the A inputs of its length-A DFT and ends with X[q + B k1]
// in slot k1.  Above 256 the second stage is shared by thread pairs (PAIR): thread p = 2 k2 + h transforms the
// H = A/2 values n1 = 2 m + h, and the radix-2 step that joins the halves exchanges values with thread p ^ 1, TX
// lanes away in the same wavefront: thread p ends with X[k2 + B (i + H h)] in slot i.  The inverse runs the steps
// backwards.  Every thread holds all three components of its points, so the 3 x 3 product needs no exchange.
//
// What bounds it: the field's 24 values per cell read and written (4.83 GB for 6 right-hand sides in FP64 at 128^3, 0.97
// ms at the 5 TB/s of a copy), overlapped with about 3300 vector instructions per wavefront only as far as waves are
// resident.  Registers set that: three components of 16 FP64 values take 192 of them, so a second wave per SIMD
// (256) leaves 64 for everything else.  What it takes to stay within them: loads and stores through a bounds-checked
// buffer (branches around each element kept both sides' registers alive: 160-490 spilled), scheduling fences between
// the short DFTs, table entries requested one value ahead only, and store offsets computed again.  FP64 still
// spills 10 to 16 registers at 192 and 256, 3 to 5 at 320 and 31 at 512 with the octant table, FP32 14 to 16 at 224: two
// waves (three) with them measured faster than one (two) without.  The table's layout (green_index) gives every load of a
// wavefront whole lines in 16-byte pieces; entries of a k-point side by side, 48 or 96 bytes per lane, or 8-byte loads
// cost the FP32 pass 0.12 ms at 128^3.
// Measured before (one FP64 wave per SIMD; LDS Stockham kernels at 48 and 96) -> now, 6 right-hand sides: FP64 0.145
// -> 0.083 ms at 48^3, 0.205 -> 0.175 at 64^3, 0.778 -> 0.59 at 96^3, 1.817 -> 1.30 at 128^3; FP32 0.109 -> 0.097 at
// 64^3, 0.338 -> 0.305 at 96^3, 0.736 -> 0.612 at 128^3; one right-hand side at 256^3 FP64 3.72 -> 2.62, FP32 1.72 ->
// 1.50 ms.  Splitting the components over three thread groups (a third of the registers per thread, the product through
// LDS) measured 2.5 ms at 128^3 in FP64 and 1.5 ms in FP32: half the data in flight per compute unit.
template <int L>
struct ZLine {
    static constexpr bool PAIR = L > 256;
    static constexpr int B = L <= 16 ? 4 : L <= 64 ? 8 : 16;
    static constexpr int A = L / B;
    static constexpr int NT = PAIR ? 2 * B : B;   // threads per line and component
    static constexpr int H = PAIR ? A / 2 : A;    // values per thread between the stages
    static_assert(A * B == L && A <= NT && (!PAIR || A % 2 == 0), "unsupported length");
};

// Waves per SIMD of the register z pass.  FP64 at 384 needs 75 registers more than two waves leave: 3.02 ms (2
// right-hand sides at 192^3) against 2.54 ms with one wave; 224 (3 at 112^3: 0.61 against 0.54 ms) and 448 60 and 170;
// the half-space table's index work at 512 as many.  At 320 the two waves pay (160^3 0.72 against 0.81 ms).  FP32: three
// up to 256 (four spill as well, 0.86 against 0.74 ms at 128^3; two are slower at 224, 3 right-hand sides at 112^3 0.310
// against 0.294 ms); above, blocks of 512 threads are two waves a SIMD, and a second block would need four (a cap of three
// spills 29-57 registers at 448: one right-hand side at 224^3 1.37 against 1.17 ms; 288 to 384 and 512 take the same time).
template <typename T, int L, bool HALF>
constexpr int z_waves() {
    return sizeof(T) == 8 ? (L == 224 || L == 384 || L == 448 || (L == 512 && HALF) ? 1 : 2) : (L > 256 ? 2 : 3);
}

// Scheduling fence between the components of the register z pass: above 256 it saves the registers of the second wave
// (one right-hand side at 256^3 in FP64 2.90 -> 2.62 ms); shorter lines lose by it (3 right-hand sides at 96^3 0.317
// against 0.299 ms).
template <int L>
__device__ __forceinline__ void fence() {
    if constexpr (L > 256) __builtin_amdgcn_sched_barrier(0);
}

template <typename T, int L, int TX, bool HALF, int ZBS>
__global__ __launch_bounds__((TX * ZLine<L>::NT), (z_waves<T, L, HALF>())) void k_zgreen(
    cpx<T>* __restrict__ data, int nrhs, int L1, int L2, long long CS, long long RS, long long ES, int n3, GreenTabs<T> gt,
    const cpx<T>* __restrict__ tw, long long nb_real) {
    using Z = ZLine<L>;
    constexpr int A = Z::A, B = Z::B, NT = Z::NT, H = Z::H, V = B > H ? B : H;
    __shared__ cpx<T> lds[L * TX];
    __shared__ cpx<T> tws[L];
    const int lb = xcd_logical_block(blockIdx.x, (unsigned)nb_real);
    if (lb < 0) return;
    const int tid = threadIdx.x, t = tid % TX, q = tid / TX;
    stage_twiddles<T, L>(tws, tw, tid, TX * NT);
    const int ntx = L1 / TX;
    // right-hand side fastest, then x tiles and y rows, both in mirror pairs (unsigned 32-bit divisions: the 64-bit ones
    // took 550 scalar instructions)
    const unsigned col = (unsigned)lb / (unsigned)nrhs, yb = col / (unsigned)ntx;
    const int rhs = (int)((unsigned)lb - col * (unsigned)nrhs);
    const cpx<T>* __restrict__ ghat = gt.g[rhs];   // this position's frequency
    const int xt = paired_row((int)(col - yb * (unsigned)ntx), ntx);
    const int y = paired_row((int)yb, L2);
    const int kx0 = xt * TX + t;
    const bool s1 = A == NT || q < A;                       // a first-stage thread
    const int qa = s1 ? q : A - 1;
    const int k2 = Z::PAIR ? q >> 1 : q, h = Z::PAIR ? q & 1 : 0;
    const T sgn = h ? T(-1) : T(1);

    // Byte offset of element q + A j of a component's line.  Elements from n3 on lie beyond the component's CS values
    // (whole z planes or blocks follow one another), so the buffer's bounds check gives the zeros of the padding.
    const unsigned row = (unsigned)(zrow_offset(y, ZBS, L1) + (long long)xt * TX) + (unsigned)t;
    const unsigned idle = s1 ? 0u : 0x80000000u;   // past the end (the host keeps the data below 2^31 bytes)
    auto off = [&](int q, int j) __attribute__((always_inline)) {
        const unsigned e = (unsigned)(q + A * j);
        return ((e >> ZBS) * ((unsigned)ES << ZBS) + (e & ((1u << ZBS) - 1)) * (unsigned)L1 + row) * (unsigned)sizeof(cpx<T>) + idle;
    };
    cpx<T>* const base = data + (long long)rhs * RS;
    const unsigned bytes = (unsigned)CS * (unsigned)sizeof(cpx<T>);

    cpx<T> v[3][V];
    // the field is streamed once: non-temporal loads and stores leave the caches to the table
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const Buffer<T> in(base + c * CS, bytes);
#pragma unroll
        for (int j = 0; j < B / 2; ++j) v[c][j] = in.load_nt(off(q, j));
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        fence<L>();
        if (s1) {
            reg_dft_io<-1, B, T, true>([&](int j) { return v[c][j]; }, [&](int i, cpx<T> x) {
                lds[(i * A + q) * TX + t] = i > 0 ? x * tw_at<-1>(tws, q * i) : x;
            });
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < H; ++m) v[c][m] = lds[(k2 * A + (Z::PAIR ? 2 * m + h : m)) * TX + t];
        __syncthreads();
        if constexpr (H == 16)
            reg_dft_io<-1, H, T, false>([&](int j) { return v[c][j]; }, [&](int i, cpx<T> x) { v[c][i] = x; });
        else
            reg_dft_any<-1, H, T>(v[c]);
        if constexpr (Z::PAIR) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                v[c][i] = pair_forward<-1, TX>(v[c][i], i * B, h, sgn, tws);
                if (i % 4 == 3) fence<L>();
            }
        }
    }
    fence<L>();

    const int GP = green_pitch(L1), O2 = L2 / 2 + 1;
    int kx, ky;
    bool fx, fy;
    fold_index(kx0, L1, kx, fx);
    fold_index(y, L2, ky, fy);
    // half-space table: k_x > L1/2 reads the entry at -k
    const bool hneg = kx0 > L1 / 2;
    const int hx = hneg ? L1 - kx0 : kx0, hy = hneg ? (L2 - y) % L2 : y;
    // the table entries of value i + 1 are requested before value i is multiplied; the scheduling fences keep the
    // compiler from requesting more at once, which would cost the registers of a second wave
    cpx<T> g[2][6];
    auto load = [&](int i) __attribute__((always_inline)) {
        const int kz0 = k2 + B * (i + H * h);
        unsigned o;
        if constexpr (HALF) {
            const int hz = hneg ? (L - kz0) % L : kz0;
            o = ((unsigned)hz * (unsigned)L2 + (unsigned)hy) * (unsigned)(kGreenUnits<T> * GP) + (unsigned)hx;
        } else {
            const int kz = kz0 > L / 2 ? L - kz0 : kz0;
            o = ((unsigned)kz * (unsigned)O2 + (unsigned)ky) * (unsigned)(kGreenUnits<T> * GP) + (unsigned)kx;
        }
        load_g6(ghat, o * 16u, GP, g[i & 1]);
    };
    load(0);
#pragma unroll
    for (int i = 0; i < H; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < H) load(i + 1);
        __builtin_amdgcn_sched_barrier(0);
        const cpx<T> g11 = g[i & 1][0], g22 = g[i & 1][1], g33 = g[i & 1][2];
        cpx<T> g23 = g[i & 1][3], g13 = g[i & 1][4], g12 = g[i & 1][5];
        if constexpr (!HALF) {
            const bool fz = k2 + B * (i + H * h) > L / 2;
            if (fy != fz) g23 = T(-1) * g23;
            if (fx != fz) g13 = T(-1) * g13;
            if (fx != fy) g12 = T(-1) * g12;
        }
        const cpx<T> f1 = v[0][i], f2 = v[1][i], f3 = v[2][i];
        v[0][i] = cdot3(g11, f1, g12, f2, g13, f3);
        v[1][i] = cdot3(g12, f1, g22, f2, g23, f3);
        v[2][i] = cdot3(g13, f1, g23, f2, g33, f3);
    }

#pragma unroll
    for (int c = 0; c < 3; ++c) {
        fence<L>();
        if constexpr (Z::PAIR) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                v[c][i] = pair_backward<+1, TX>(v[c][i], i * B, h, sgn, tws);
                if (i % 4 == 3) fence<L>();
            }
        }
        auto put = [&](int m, cpx<T> x) __attribute__((always_inline)) {
            const int n1 = Z::PAIR ? 2 * m + h : m;
            lds[(n1 * B + k2) * TX + t] = x * tw_at<+1>(tws, n1 * k2);
        };
        if constexpr (H == 16) {
            reg_dft_io<+1, H, T, false>([&](int j) { return v[c][j]; }, put);
        } else {
            reg_dft_any<+1, H, T>(v[c]);
#pragma unroll
            for (int m = 0; m < H; ++m) put(m, v[c][m]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < B; ++i) v[c][i] = lds[(qa * B + i) * TX + t];
        if (c < 2) __syncthreads();
        if (s1) {
            const Buffer<T> out(base + c * CS, bytes);
            int qs = q;   // opaque copy: the offsets are computed again, not kept in registers since the loads
            asm volatile("" : "+v"(qs));
            reg_dft_io<+1, B, T, false>([&](int j) { return v[c][j]; }, [&](int j, cpx<T> x) {
                if (j < B / 2) out.store_nt(off(qs, j), x);
            });
        }
    }
}

// LDS z pass for one work-buffer layout (ZBS, compile time), full or half table
template <typename T, int LL, int TX, int ZBS>
void launch_lds_z(Ctx* c, cpx<T>* data, int nrhs, long long CS, long long RS, long long ES, const GreenTabs<T>& ghat,
                  const cpx<T>* tw) {
    const dim3 grid(nrhs * (c->L1 / TX), c->L2, 1);
    if (c->green_half)
        hipLaunchKernelGGL((k_fft_zgreen<T, LL, TX, true, ZBS>), grid, dim3(kThreads), 0, c->stream, data, nrhs,
                           c->L1, c->L2, CS, RS, ES, c->n3, ghat, tw);
    else
        hipLaunchKernelGGL((k_fft_zgreen<T, LL, TX, false, ZBS>), grid, dim3(kThreads), 0, c->stream, data, nrhs,
                           c->L1, c->L2, CS, RS, ES, c->n3, ghat, tw);
}

template <typename T, int LL, int TX, bool HALF>
void launch_reg_z(Ctx* c, cpx<T>* data, int nrhs, long long CS, long long RS, long long ES, const GreenTabs<T>& ghat,
               const cpx<T>* tw) {
    const long long nb = (long long)nrhs * (c->L1 / TX) * c->L2;
    const dim3 g((unsigned)((nb + 7) / 8 * 8)), b(TX * ZLine<LL>::NT);
    if (c->zbs)
        hipLaunchKernelGGL((k_zgreen<T, LL, TX, HALF, 3>), g, b, 0, c->stream, data, nrhs, c->L1, c->L2, CS, RS, ES, c->n3,
                           ghat, tw, nb);
    else
        hipLaunchKernelGGL((k_zgreen<T, LL, TX, HALF, 0>), g, b, 0, c->stream, data, nrhs, c->L1, c->L2, CS, RS, ES, c->n3,
                           ghat, tw, nb);
}

template <typename T>
int launch_zgreen(Ctx* c, cpx<T>* data, int nrhs, const GreenTabs<T>& ghat, const cpx<T>* tw, int variant = 0,
                  int ntab = 1) {
    const int L1 = c->L1, L2 = c->L2, L = c->L3;
    const long long CS = (long long)c->n3 * L2 * L1;
    const long long RS = 3 * CS;
    const long long ES = (long long)L2 * L1;
    // the register kernel addresses a component's line and the table with 32-bit byte offsets (the line's with the top
    // bit free); larger grids (half-space tables of 256^3 in FP64) take the LDS kernel
    const long long table = (c->green_half ? (long long)L * L2 : (long long)(L / 2 + 1) * (L2 / 2 + 1)) * green_pitch(L1);
    const bool off32 = CS * (long long)sizeof(cpx<T>) < (1LL << 31) && L / 2 * ES * (long long)sizeof(cpx<T>) < (1LL << 31) &&
                       table * 6 * (long long)sizeof(cpx<T>) < (1LL << 32);
    c->prof.begin(c->stream, LS_PNAME(T, "fft_z_green"), nrhs, ntab);
    const bool fs = variant == 0 && use_fourstep() && off32;
    switch (L) {
#define CASE(LL)                                                                                              \
    case LL: {                                                                                                \
        if (fs) {                                                                                             \
            constexpr int TX = seg_cols<T>();                                                                 \
            if (L1 % TX) return fail(LS_ERR_ARG, "x length not a multiple of the z-pass tile");               \
            if (c->green_half)                                                                                \
                launch_reg_z<T, LL, TX, true>(c, data, nrhs, CS, RS, ES, ghat, tw);                           \
            else                                                                                              \
                launch_reg_z<T, LL, TX, false>(c, data, nrhs, CS, RS, ES, ghat, tw);                          \
            break;                                                                                            \
        }                                                                                                     \
        constexpr int TX = zpass_cols<T, LL>();                                                               \
        if (L1 % TX) return fail(LS_ERR_ARG, "x length not a multiple of the z-pass tile");                   \
        if (c->zbs)                                                                                           \
            launch_lds_z<T, LL, TX, 3>(c, data, nrhs, CS, RS, ES, ghat, tw);                                  \
        else                                                                                                  \
            launch_lds_z<T, LL, TX, 0>(c, data, nrhs, CS, RS, ES, ghat, tw);                                  \
        break;                                                                                                \
    }
        LS_FOR_LENGTHS(CASE)
#undef CASE
        default:
            return fail(LS_ERR_ARG, "unsupported FFT length");
    }
    c->prof.end(c->stream);
    LS_HIP(hipGetLastError());
    return LS_OK;
}

template <typename T>
const cpx<T>* green_table(const Ctx* c, int i);
template <>
const z128* green_table<double>(const Ctx* c, int i) { return c->ghat[i]; }
template <>
const z64* green_table<float>(const Ctx* c, int i) { return c->ghat32[i]; }

template <typename T>
GreenTabs<T> green_tabs(const Ctx* c, const RhsSet& set) {
    GreenTabs<T> g{};
    for (int r = 0; r < set.n; ++r) g.g[r] = green_table<T>(c, set.freq[r]);
    return g;
}

}  // namespace

template <typename T>
int z_green_pass(Ctx* c, const RhsSet& set, cpx<T>* work, int variant) {
    return launch_zgreen<T>(c, work, set.n, green_tabs<T>(c, set), twiddles<T>(c, c->L3), variant, distinct_freqs(set));
}

template int z_green_pass<double>(Ctx*, const RhsSet&, z128*, int);
template int z_green_pass<float>(Ctx*, const RhsSet&, z64*, int);

}  // namespace ls
